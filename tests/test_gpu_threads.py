"""Plans of different sizes used by two host threads at once: the kernels with a
varying amount of LDS (small inner solves, block steps, projected solves, short
Toeplitz transforms) must launch and give what each plan gives by itself (same
kernels, same order of operations: the same bits)."""
import threading

import numpy as np
import pytest
import torch

import workloads as wl
from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def jobs():
    out = []
    for N, p, m in [(12, 2, 6), (60, 1, 10), (40, 4, 8), (24, 8, 10)]:
        W = wl.c1(N=N, p=p)
        pl = Plan.csr(W.A.rowptr, W.A.colind, W.A.val, W.t, device=DEV, m=m, inner_precond="jacobi")
        B = torch.from_numpy(W.B).to(DEV)
        out.append(lambda pl=pl, B=B: pl.execute(B, tol=1e-9)[0])
    for n in (30, 600, 1000, 3000):
        col = np.concatenate([[3.0], -0.5 / np.arange(1.0, n) ** 2])
        pl = Plan.toeplitz(col, 0.3, device=DEV, m=3)
        X = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 3))).to(DEV)
        out.append(lambda pl=pl, X=X: pl.apply_inverse(X)[0])
    return out


def test_plans_of_different_sizes_on_two_threads():
    print("[gpu-test] two threads", flush=True)
    work = jobs()
    ref = [f().cpu() for f in work]
    errors = []

    def use(first, step):
        try:
            # a plan belongs to one thread: every other job each
            for _ in range(10):
                for i in range(first, len(work), step):
                    if not torch.equal(work[i]().cpu(), ref[i]):
                        errors.append(f"job {i} differs")
        except Exception as e:  # noqa: BLE001
            errors.append(repr(e))

    threads = [threading.Thread(target=use, args=(k, 2)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[:3]
