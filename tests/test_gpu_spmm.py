"""CSR products whose entries are staged through LDS (csr_rows_staged) and
those that are not (rows of more than 8 nonzeros on average), element by
element against scipy.

Tolerance: a row of k products summed in any order is within (k + 1) u of its
exact value relative to sum |a_ij x_j| (u = 2^-53), on both sides, plus the
rounding of t a_ij: 2 (k + 2) u sum |t a_ij x_j|.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def arrow(n):
    """Tridiagonal with a dense first row and column: one row of n entries
    (many chunks), the others of 3 or 4."""
    A = sp.lil_matrix(sp.diags([np.full(n - 1, -1.0), np.full(n, 4.0), np.full(n - 1, -1.5)],
                               [-1, 0, 1]))
    A[0, :] = np.linspace(-1.0, 1.0, n)
    A[:, 0] = np.linspace(1.0, -0.5, n)[:, None]
    A[0, 0] = 2.0 * n
    return sp.csr_matrix(A)


def diagonal_and_long(n):
    """Rows of one entry and, every 97th, of 150."""
    A = sp.lil_matrix(sp.identity(n) * 3.0)
    rng = np.random.default_rng(n)
    for i in range(0, n, 97):
        A[i, rng.choice(n, 150, replace=False)] = rng.standard_normal(150)
        A[i, i] = 5.0
    return sp.csr_matrix(A)


def wide(n):
    """27 nonzeros per row: not staged."""
    return sp.csr_matrix(sp.diags([np.full(n, 30.0 if o == 0 else -1.0) for o in range(-13, 14)],
                                  range(-13, 14), shape=(n, n)))


@pytest.mark.parametrize("make,n", [(arrow, 2500), (arrow, 513), (diagonal_and_long, 4100),
                                    (wide, 1000)])
@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 8, 12, 16, 31, 32])
def test_products(make, n, p):
    print(f"[gpu-test] products {make.__name__} n={n} p={p}", flush=True)
    A = -make(n)
    pl = Plan.csr(A.indptr, A.indices, A.data, 0.7, device=DEV, inner_precond="jacobi", m=3)
    X = np.random.default_rng(p).standard_normal((n, p))
    for transpose in (False, True):
        M = sp.csr_matrix(A.T if transpose else A) * 0.7
        Y = pl.apply_operator(torch.from_numpy(X), transpose=transpose).cpu().numpy()
        k = np.diff(M.indptr)[:, None]
        bound = 2 * (k + 2) * 2.0 ** -53 * (abs(M) @ abs(X))
        assert np.all(np.abs(Y - M @ X) <= bound)


@pytest.mark.parametrize("p", [3, 8, 16, 32])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_inner_solves_with_staged_products(p, precision):
    """The inner CG and BiCGStab (whose products write the dot products'
    partial sums) on staged operators with one long row: Jacobi, residual of
    the result."""
    print(f"[gpu-test] staged inner p={p} {precision}", flush=True)
    n = 5000
    tol = 1e-12 if precision == "fp64" else 1e-6
    T = sp.diags([np.full(n - 1, -1.0), np.full(n, 3.0), np.full(n - 1, -1.0)], [-1, 0, 1])
    S = sp.csr_matrix(T) + sp.csr_matrix(([0.001], ([0], [n - 1])), shape=(n, n))
    for A in (sp.csr_matrix(T), S):
        A = -sp.csr_matrix(A)
        pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_precond="jacobi", m=3,
                      inner_tol=tol, precision=precision)
        X = np.random.default_rng(p).standard_normal((n, p))
        Y, _ = pl.apply_inverse(torch.from_numpy(X))
        res = np.linalg.norm(A @ Y.cpu().numpy() - X, axis=0) / np.linalg.norm(X, axis=0)
        # the recurrence residual stops at tol; cond(K) <= 5, so the true one
        # (and, in FP32, the rounding of Y itself) is within a small multiple
        assert res.max() < 10 * max(tol, 2.0 ** -22 if precision == "mixed" else 0.0)
