"""Variants of the value and trajectory scans of the small sizes that depend on how much there is to do,
against the oracle: FP32 scans with and without two waves a SIMD (more than 1024 tiles over all
problems: 64 blocks a tile for short horizons, 256 in the trajectory scan from 2^15 blocks on), and
time-invariant solves whose elements are formed and reduced in one launch or in two (FP32 up to
2^15 blocks), at nx = 3 within the horizons of the three-launch scan (2^13 to 2^15 blocks).
Problems of a batch have scaled references and initial states.  Tolerance as for every solve."""
import pytest
import torch

import oracle as O
from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-9, torch.float32: 1e-4}


def _check(p, batch, dtype, lti=False):
    dp = lqt.DeviceProblem.from_problems([p], dtype=dtype)
    scale = torch.linspace(0.5, 2.0, batch, dtype=dtype, device="cuda")
    for k in ("t", "Q", "R", "r", "Qf", "rf", "x0"):
        a = getattr(dp, k)
        a = a.expand(batch, *a.shape[1:]).contiguous()
        if k in ("r", "x0", "rf"):  # v, x and u follow the inputs linearly, S does not change
            a = a * scale.view(-1, *[1] * (a.dim() - 1))
        setattr(dp, k, a)
    dp.batch, dp.lti = batch, lti
    got = lqt.solve(dp)
    torch.cuda.synchronize()
    ref = O.solve(p)
    for k in ("S", "v", "x", "u"):
        want, x = torch.as_tensor(ref[k], device="cuda"), got[k].double()
        if k != "S":
            x = x / scale.double().view(-1, *[1] * (x.dim() - 1))
        e = float((x - want).abs().max() / want.abs().max())
        assert e < TOL[dtype], f"{k}: {e:.3e}"


@pytest.mark.parametrize("nx", [3, 4])
@pytest.mark.parametrize("T,batch", [(5, 1024), (5, 1025), (129, 341), (129, 342), (512, 129),
                                     (32769, 7), (32769, 8)])
def test_fp32_waves(nx, T, batch):
    _check(W.random_stable(5 + nx, nx, 2, T, 1, tf=min(2.0, 0.05 * T), time_varying=False), batch,
           torch.float32)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,T,batch", [(3, 8193, 1), (3, 9001, 2), (3, 32768, 1), (4, 600, 1),
                                        (4, 5001, 3), (4, 32769, 1), (4, 300001, 1)])
def test_time_invariant_one_or_two_launches(nx, T, batch, dtype):
    _check(W.random_stable(8, nx, 2, T, 2, tf=2.0, time_varying=False), batch, dtype, lti=True)
