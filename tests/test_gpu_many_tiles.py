"""Kernels whose workgroups loop over row tiles, at sizes where each workgroup takes
several: the staged CSR products on an irregular operator (several chunks of
entries per tile as well, a ragged last tile, odd and even p), and the
Gram-Schmidt update passes (more than eight 16-row steps per workgroup, a ragged
last one).

Tolerances.  Products: 2 (k + 2) u sum |t a_ij x_j| for a row of k entries (each side
sums within (k + 1) u, plus the rounding of t a_ij).  Inner solves: the operators are
diagonally dominant, 1 in the off-diagonal row sum against 3, so cond <= 2 after
scaling and the true residual is within a small multiple of the tolerance.
Whole solves: as in test_gpu_orth_update.py, 1e-10 for a stopping bound of 1e-11.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import workloads as wl
from oracle import inverses
from oracle.cf import r_eval
from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def irregular(n, long_row, every, symmetric):
    """Diagonal 3 and, in every `every`-th row, `long_row` random entries summing to
    1 in modulus (less where the transpose is added)."""
    rng = np.random.default_rng(n)
    rows = np.arange(5, n, every)
    i = np.repeat(rows, long_row)
    j = rng.integers(0, n, i.size)
    v = rng.uniform(-1.0, 1.0, i.size) / long_row
    M = sp.csr_matrix((v, (i, j)), shape=(n, n))
    M = M + M.T if symmetric else M
    M.setdiag(0.0)
    s = np.asarray(abs(M).sum(axis=1)).ravel()
    s = np.maximum(s, np.asarray(abs(M).sum(axis=0)).ravel())
    M = M.multiply(1.0 / max(1.0, s.max()))
    A = -sp.csr_matrix(M + 3.0 * sp.identity(n))
    assert A.nnz <= 8 * n
    return A


# rows per tile: 512 / lanes per row; 512 workgroups
CASES = [(100003, 16), (160001, 3), (20011, 31), (330001, 4), (100003, 12), (90001, 8)]


@pytest.mark.parametrize("n,p", CASES)
def test_products(n, p):
    print(f"[gpu-test] many tiles, product n={n} p={p}", flush=True)
    A = irregular(n, 2500, 601, False)
    pl = Plan.csr(A.indptr, A.indices, A.data, 0.7, device=DEV, inner_precond="jacobi", m=3)
    X = np.random.default_rng(p).standard_normal((n, p))
    for transpose in (False, True):
        M = sp.csr_matrix(A.T if transpose else A) * 0.7
        Y = pl.apply_operator(torch.from_numpy(X), transpose=transpose).cpu().numpy()
        k = np.diff(M.indptr)[:, None]
        assert np.all(np.abs(Y - M @ X) <= 2 * (k + 2) * 2.0 ** -53 * (abs(M) @ abs(X)))


@pytest.mark.parametrize("n,p", CASES)
@pytest.mark.parametrize("symmetric", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_inner_solves(n, p, symmetric, precision):
    print(f"[gpu-test] many tiles, inverse n={n} p={p} sym={symmetric} {precision}", flush=True)
    A = irregular(n, 1000, 601, symmetric)
    tol = 1e-12 if precision == "fp64" else 1e-6
    pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_precond="jacobi", m=3,
                  inner_tol=tol, precision=precision)
    X = np.random.default_rng(p).standard_normal((n, p))
    for transpose in (False,) if symmetric else (False, True):
        Y, _ = pl.apply_inverse(torch.from_numpy(X), transpose=transpose)
        R = (A.T if transpose else A) @ Y.cpu().numpy() - X
        res = np.linalg.norm(R, axis=0) / np.linalg.norm(X, axis=0)
        assert res.max() < 10 * max(tol, 2.0 ** -22 if precision == "mixed" else 0.0)


# n = 76,729 = 512 * 16 * 9.4: the column-block counts 8, 16, 24 and 32 of the update
# passes from both sides (p = 16 is limited to 31 panels, p = 8 to 63)
@pytest.mark.parametrize("p,m", [(16, 8), (16, 9), (16, 17), (16, 25), (16, 31), (8, 16), (8, 17),
                                 (8, 33), (8, 49), (8, 63)])
def test_update_passes(p, m):
    print(f"[gpu-test] many steps, orth update p={p} m={m}", flush=True)
    W = wl.c1(N=277, p=p)
    ref = inverses.dst_laplacian_function(277, 2, W.t, lambda x: r_eval(np.asarray(x, float)), W.B)
    pl = Plan.csr(W.A.rowptr, W.A.colind, W.A.val, W.t, device=DEV, m=m, max_cycles=400)
    Z, _ = pl.execute(torch.from_numpy(W.B), tol=1e-11)
    assert np.linalg.norm(Z.cpu().numpy() - ref) < 1e-10 * np.linalg.norm(ref)
