"""The Gram-Schmidt update passes of FP64 bases with panels of 8 and 16
columns (k_orth_upd), at the edges of its column-block counts (8, 16, 24 and 32
blocks of 16 columns) and with a ragged last row block, through whole solves
against the closed form of r(tA)B.

Tolerance: the stopping bound is 1e-11 of ||Z|| and the closed form carries
about 1e-15 ||B||, with ||Z|| > 1e-3 ||B||; a panel that is not orthogonal to
the others (or a coefficient that is off) shows at the size of the error it
makes, so 1e-10 as in the other solves.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import inverses
from oracle.cf import r_eval
from paper_1405_0707_amd import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,p,m", [(45, 16, 3), (45, 16, 8), (45, 16, 9), (53, 16, 16), (53, 16, 17),
                                   (53, 16, 24), (53, 16, 25), (53, 16, 31), (45, 8, 2), (45, 8, 16),
                                   (45, 8, 17), (53, 8, 33)])
@pytest.mark.parametrize("precond", [1, 0])
def test_solves(N, p, m, precond):
    print(f"[gpu-test] orth update N={N} p={p} m={m} precond={precond}", flush=True)
    if precond == 0 and m < 3:
        pytest.skip("cycles of two steps of Algorithm 1 do not converge")
    W = wl.c1(N=N, p=p)
    t = W.t * 0.1 if precond == 0 else W.t      # Algorithm 1 needs a smaller ||tA||
    ref = inverses.dst_laplacian_function(N, 2, t, lambda x: r_eval(np.asarray(x, float)), W.B)
    pl = Plan.csr(W.A.rowptr, W.A.colind, W.A.val, t, device=DEV, m=m, preconditioned=precond,
                  max_cycles=400)
    Z, _ = pl.execute(torch.from_numpy(W.B), tol=1e-11)
    assert np.linalg.norm(Z.cpu().numpy() - ref) < 1e-10 * np.linalg.norm(ref)
