"""Toeplitz products and inverses whose result overlaps the input (the same block,
and blocks shifted by a few elements, which the streaming passes always took),
against the call on blocks of their own.

Tolerance: in place the same kernels run (the same bits); shifted, the streaming
ones: both within 1e-13 (product) and 1.2e-12 (inverse, condition number below 4
times six transforms) of the exact result relative to its largest entry, so within
twice that of each other.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1405_0707_amd import Plan
from paper_1405_0707_amd._lib import check, lib

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [600, 1000, 1009, 3000])
@pytest.mark.parametrize("p", [1, 5, 32])
@pytest.mark.parametrize("shift", [0, 1, 3, 40])
def test_overlap(n, p, shift):
    print(f"[gpu-test] overlapping blocks n={n} p={p} shift={shift}", flush=True)
    col = np.concatenate([[3.0], -0.5 / np.arange(1.0, n) ** 2])
    pl = Plan.toeplitz(col, 0.3, device=DEV, m=3)
    X = torch.from_numpy(np.random.default_rng(n + p).standard_normal((n, p))).to(DEV)
    buf = torch.zeros(n * p + 64, dtype=torch.float64, device=DEV)
    wp, wb = pl._ws(p)
    it = C.c_longlong()
    for name in ("product", "inverse"):
        for a, b in ((0, shift), (shift, 0)):
            ref = pl.apply_operator(X) if name == "product" else pl.apply_inverse(X)[0]
            x, y = buf[a:a + n * p].view(n, p), buf[b:b + n * p].view(n, p)
            x.copy_(X)
            if name == "product":
                check(lib().expmv_apply_operator(pl._h, 0, x.data_ptr(), p, wp, wb, y.data_ptr()),
                      name)
            else:
                check(lib().expmv_apply_inverse(pl._h, 0, x.data_ptr(), p, wp, wb, y.data_ptr(),
                                                C.byref(it)), name)
            tol = 0.0 if shift == 0 else (2e-13 if name == "product" else 2.4e-12)
            assert (y - ref).abs().max() <= tol * ref.abs().max()
