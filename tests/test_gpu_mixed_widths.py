"""FP32 inner solves of even widths: two columns per lane at p = 2, 4, 6, 10, four
at 8, 12, 20, with staged (3 nonzeros per row) and long rows, and the time of
four columns.

Tolerance: the recurrence residual stops at 1e-6 and cond(K) <= 5, so the true one,
with the rounding of the FP32 result, is within a small multiple.
"""
import time

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def banded(n, width, skew):
    offs = list(range(-(width // 2), width - width // 2))
    return -sp.csr_matrix(sp.diags([np.full(n, 2.0 * width if o == 0 else -1.0 - skew * (o > 0))
                                    for o in offs], offs, shape=(n, n)))


@pytest.mark.parametrize("p", [2, 4, 6, 8, 10, 12, 20])
@pytest.mark.parametrize("n,width", [(5000, 3), (70001, 3), (9001, 27)])
@pytest.mark.parametrize("skew", [0.0, 0.3])
def test_residuals(p, n, width, skew):
    print(f"[gpu-test] mixed widths p={p} n={n} width={width} skew={skew}", flush=True)
    A = banded(n, width, skew)
    pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_precond="jacobi", m=3,
                  inner_tol=1e-6, precision="mixed")
    X = np.random.default_rng(p).standard_normal((n, p))
    Y, _ = pl.apply_inverse(torch.from_numpy(X))
    res = np.linalg.norm(A @ Y.cpu().numpy() - X, axis=0) / np.linalg.norm(X, axis=0)
    assert res.max() < 1e-5


def test_time_of_four_columns():
    """40,000 rows of 27: an iteration of four columns takes at most 0.85 times one of
    eight (0.78 measured, 0.90 with one lane per row)."""
    print("[gpu-test] mixed width time", flush=True)
    offs = range(-13, 14)
    A = -sp.csr_matrix(sp.diags([np.full(40000, 32.5 if o == 0 else -1.0) for o in offs], offs,
                                shape=(40000, 40000)))
    pl = Plan.csr(A.indptr, A.indices, A.data, 1.0, device=DEV, inner_precond="jacobi", m=3,
                  inner_tol=1e-5, precision="mixed")
    best = {}
    for _ in range(15):
        for p in (4, 8):
            X = torch.ones(40000, p, device=DEV, dtype=torch.float64)
            X[::2] = -0.5
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(4):
                _, iters = pl.apply_inverse(X)
            best[p] = min(best.get(p, np.inf), (time.perf_counter() - t0) / max(iters, 1))
    assert best[4] < 0.85 * best[8], best
