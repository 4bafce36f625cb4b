"""Blocks that start at an odd FP64 element (views into a larger buffer): the
entry points that read and write a caller's block through the inner solvers'
16-byte accesses, against the same call on an aligned copy.

The products, the Jacobi and AMG solves and the preconditioner run the same
operations per element in the same order on both, so the results agree to the
last bit; e^{tA}B and the time gradient do too.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def odd_view(x):
    n, p = x.shape
    buf = torch.zeros(n * p + 2, dtype=torch.float64, device=DEV)
    v = buf[1:1 + n * p].view(n, p)
    v.copy_(x)
    assert v.data_ptr() % 16 == 8
    return v


@pytest.mark.parametrize("N,precond", [(20, "jacobi"), (75, "jacobi"), (75, "amg")])
@pytest.mark.parametrize("p", [1, 2, 4, 6, 16])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_odd_offsets(N, precond, p, precision):
    print(f"[gpu-test] odd offset N={N} {precond} p={p} {precision}", flush=True)
    W = wl.c1(N=N, p=p)
    pl = Plan.csr(W.A.rowptr, W.A.colind, W.A.val, W.t, device=DEV, m=8, inner_precond=precond,
                  precision=precision)
    X = torch.from_numpy(np.random.default_rng(p).standard_normal((N * N, p))).to(DEV)
    V = odd_view(X)
    tol = 1e-9 if precision == "fp64" else 1e-5
    for call in (pl.apply_operator, lambda x: pl.apply_inverse(x)[0], pl.apply_preconditioner,
                 lambda x: pl.execute(x, tol=tol)[0]):
        assert torch.equal(call(X), call(V))
    assert pl.grad_t(X, X) == pl.grad_t(V, V)
    out = odd_view(torch.zeros_like(X))
    pl.execute(X, tol=tol, out=out)
    assert torch.equal(out, pl.execute(X, tol=tol)[0])
