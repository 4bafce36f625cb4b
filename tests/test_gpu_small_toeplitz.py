"""Toeplitz products and inverses at the lengths where one workgroup does a
whole column (csrc/small_fft.hpp) and just past them, against dense
arithmetic.

Tolerances relative to the largest entry: FFTs of length L lose about
log2(L) u per transform (u = 1.1e-16), six transforms and pointwise products in
the inverse: 1e-13 for the product, and 1e-13 times the condition number (at
most (3 + 1.7) / (3 - 1.7) < 4 for the column below, times the ratio 3 of the
largest and smallest d) for the inverse: 1.2e-12.
"""
import numpy as np
import pytest
import scipy.linalg as sla
import torch

from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def vectors(n, symmetric):
    """col, row: c_0 = 3, the rest summing to less than 1.7 in modulus."""
    k = np.arange(1, n)
    rng = np.random.default_rng(n)
    col = np.concatenate([[3.0], -0.8 / np.maximum(k, 1) ** 2 * 0.6 * rng.uniform(0.5, 1.0, n - 1)])
    row = np.concatenate([[3.0], -0.8 / np.maximum(k, 1) ** 2 * rng.uniform(0.2, 0.6, n - 1)])
    return col, (col if symmetric else row)


# inverse: radices 2 3 4 5 8, lengths 3^7, the last one in LDS (3,000) and some past
# it; embedding form below and above n = 1,024;
# product: L = 2,048 at n = 1,024, past it at 1,025
SIZES = [2, 3, 5, 8, 30, 97, 625, 1000, 1009, 1024, 1025, 2048, 2049, 2187, 3000, 3125, 3240, 3375]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["symmetric", "general", "diag"])
def test_small_toeplitz(n, kind):
    print(f"[gpu-test] small toeplitz n={n} {kind}", flush=True)
    col, row = vectors(n, kind == "symmetric")
    d = np.linspace(1.0, 3.0, n) if kind == "diag" else None
    T = sla.toeplitz(col, row)
    t = 0.3
    M = -t * (T if d is None else d[:, None] * T)
    pl = Plan.toeplitz(col, t, device=DEV, m=3,
                       row0=None if kind == "symmetric" else row, diag=d)
    for p in sorted({1, min(2, n), min(5, n)}):
        X = np.random.default_rng(p).standard_normal((n, p))
        for transpose in (False, True):
            A = M.T if transpose else M
            Y = pl.apply_operator(torch.from_numpy(X), transpose=transpose).cpu().numpy()
            assert np.abs(Y - A @ X).max() <= 1e-13 * np.abs(A @ X).max()
            W, _ = pl.apply_inverse(torch.from_numpy(X), transpose=transpose)
            ref = np.linalg.solve(A, X)
            assert np.abs(W.cpu().numpy() - ref).max() <= 1.2e-12 * np.abs(ref).max()
