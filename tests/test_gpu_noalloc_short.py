"""lqt_solve_noalloc at nx >= 5 over short horizons, where its trees keep four blocks per slot (the solve
with a workspace takes fewer, for more slots): one group, one more block, a root stage of one and of
several nodes per slot, in batches, against the oracle.  Tolerance as for every solve."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import relerr
from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-9, torch.float32: 1e-4}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,T", [(5, 1), (5, 4), (5, 16), (8, 61), (8, 64), (8, 65), (8, 129),
                                  (9, 1), (9, 4), (12, 16), (12, 17), (12, 33), (16, 5), (16, 70),
                                  (16, 257)])
def test_noalloc_short(nx, T, dtype):
    ps = [W.random_stable(5, nx, 2, T, 1, tf=min(2.0, 0.05 * T)) for _ in range(3)]
    for b, p in enumerate(ps):
        p.r, p.x0 = p.r * (1.0 + b), p.x0 - b
    got = lqt.solve_noalloc(lqt.DeviceProblem.from_problems(ps, dtype=dtype))
    torch.cuda.synchronize()
    for b, p in enumerate(ps):
        ref = O.solve(p)
        for k in ("S", "v", "x", "u"):
            e = relerr(got[k][b].cpu().numpy().astype(np.float64), ref[k])
            assert e < TOL[dtype], f"problem {b} {k}: {e:.3e}"


def test_noalloc_takes_a_full_array():
    """The largest batch of the capacity table at nx = 16, T = 4: the first and last problem."""
    p = W.random_stable(5, 16, 1, 4, 1, tf=0.2, time_varying=False)
    dp = lqt.DeviceProblem.from_problems([p])
    B = 5938
    for k in ("t", "Q", "R", "r", "Qf", "rf", "x0"):
        a = getattr(dp, k)
        setattr(dp, k, a.expand(B, *a.shape[1:]).contiguous())
    dp.batch = B
    got = lqt.solve_noalloc(dp)
    torch.cuda.synchronize()
    ref = O.solve(p)
    for b in (0, 1, B // 2, B - 1):
        for k in ("S", "v", "x", "u"):
            assert relerr(got[k][b].cpu().numpy(), ref[k]) < 1e-9, (b, k)
