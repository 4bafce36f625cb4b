"""Operators small enough for one workgroup per column (csrc/small_solve.hpp),
against a sparse direct solve.

Tolerance of the inverse: the solver stops at a relative residual of 1e-13
(FP64), so the error is at most cond(K) 1e-13; the grids below have
cond(K) < 2e3 (2D Laplacian: at most 4 / pi^2 65^2 for 64 x 64 nodes, less for
the flat grids), hence 1e-9.  The FP32 inner solver (tolerance 1e-6) gives 2e3 x 1e-6.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import workloads as wl
from oracle import inverses
from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def grid2d(nx, ny, skew):
    """5-point operator on nx x ny nodes; skew > 0: upwind (nonsymmetric)."""
    one = lambda m, s: sp.diags([-(1 + s) * np.ones(m - 1), (2 + s) * np.ones(m), -np.ones(m - 1)],  # noqa: E731
                                [-1, 0, 1])
    return -sp.csr_matrix(sp.kron(sp.identity(ny), one(nx, skew)) +
                          sp.kron(one(ny, skew), sp.identity(nx)))


# edges of the row split: 512 threads with 1, 2, 4 and 8 (CG) or 7 (BiCGStab) rows
# each; above 3,584 and 4,096 rows the streaming kernels
SHAPES = [(1, 1), (5, 3), (32, 16), (27, 19), (32, 32), (41, 25), (64, 32), (683, 3), (64, 56),
          (163, 22), (64, 64), (241, 17)]


@pytest.mark.parametrize("nx,ny", SHAPES)
@pytest.mark.parametrize("skew", [0.0, 0.5])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_small_inverse(nx, ny, skew, precision):
    print(f"[gpu-test] small inverse {nx}x{ny} skew={skew} {precision}", flush=True)
    A = grid2d(nx, ny, skew)
    p = min(3, nx * ny)
    tol = 1e-13 if precision == "fp64" else 1e-6
    pl = Plan.csr(A.indptr, A.indices, A.data, 1.7, device=DEV, precision=precision,
                  inner_tol=tol, inner_precond="jacobi")
    for transpose in (False, True):
        X = np.random.default_rng(nx + transpose).standard_normal((nx * ny, p))
        X[:, p - 1] *= 1e150 if precision == "fp64" and p > 1 else 1.0   # columns are independent
        Y, iters = pl.apply_inverse(torch.from_numpy(X), transpose=transpose)
        M = (1.7 * (A.T if transpose else A)).tocsr()
        ref = inverses.splu_inverse(M)(X)
        err = np.linalg.norm(Y.cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)
        assert iters > 0
        assert err.max() < 2e3 * max(tol, 5e-13), err


def test_small_inverse_rows_and_columns():
    """Rows of 7 (in registers) and 8 nonzeros (streaming kernels), 32
    columns of which one is zero, in place."""
    for width in (7, 8):
        print(f"[gpu-test] small inverse width {width}", flush=True)
        n = 700
        offs = list(range(-(width // 2), width - width // 2))
        A = -sp.csr_matrix(sp.diags([np.full(n, 2.5 * width if o == 0 else -1.0) for o in offs],
                                    offs, shape=(n, n)))
        pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_tol=1e-13)
        X = np.random.default_rng(width).standard_normal((n, 32))
        X[:, 7] = 0.0
        Y, _ = pl.apply_inverse(torch.from_numpy(X))
        ref = inverses.splu_inverse(A.tocsr())(X)
        assert np.linalg.norm(Y.cpu().numpy() - ref) < 1e-11 * np.linalg.norm(ref)
        assert not Y[:, 7].any()


@pytest.mark.parametrize("skew", [0.0, 0.5])
def test_small_inverse_cap(skew):
    """The iteration cap stops every column and is reported (EINNER, 7)."""
    A = grid2d(20, 20, skew)
    pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_maxit=3)
    with pytest.raises(Exception, match="status 7"):
        pl.apply_inverse(torch.ones(400, 4, dtype=torch.float64))


# blocks of 1 to 4 columns at the edges of the one-workgroup block step (6,144
# values of W, 81,920 of the basis), and p = 5 and larger blocks past them
@pytest.mark.parametrize("nx,ny,p,m", [(9, 1, 1, 6), (64, 2, 1, 30), (64, 64, 1, 22), (95, 32, 2, 14),
                                       (96, 32, 2, 12), (64, 32, 3, 13), (83, 37, 2, 12),
                                       (48, 32, 4, 9), (48, 33, 4, 9), (30, 30, 5, 8)])
@pytest.mark.parametrize("skew", [0.0, 0.5])
def test_small_block_steps(nx, ny, p, m, skew):
    """e^{tA}B with the one-workgroup kernels against the streaming ones (which
    opts.profile selects).  Both stop at an error bound of 1e-12 relative to
    ||Z||; rounding is about 1e-15 ||B||, and ||Z|| > 1e-3 ||B|| on these grids:
    1e-10."""
    print(f"[gpu-test] small block steps {nx}x{ny} p={p} skew={skew}", flush=True)
    A = grid2d(nx, ny, skew)
    B = np.random.default_rng(p).standard_normal((nx * ny, p))
    Z = []
    for profile in (0, 1000000):
        pl = Plan.csr(A.indptr, A.indices, A.data, 2.0, device=DEV, m=m, profile=profile,
                      inner_precond="jacobi")
        out, info = pl.execute(torch.from_numpy(B), tol=1e-12)
        Z.append(out.cpu().numpy())
    assert np.linalg.norm(Z[0] - Z[1]) < 1e-10 * np.linalg.norm(Z[1])
