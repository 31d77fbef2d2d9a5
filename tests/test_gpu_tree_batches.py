"""Batches on the tree kernels, whose launches go over the groups of all problems: several groups a
problem, whole and broken rounds of the order in which workgroups take them, and short horizons in
large batches, through the solve and the value scan.  The problems of a batch have scaled references and
initial states, which v, x and u follow linearly, so one solve of the oracle serves all of them.
Tolerance as for every solve."""
import pytest
import torch

import oracle as O
from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-9, torch.float32: 1e-4}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nx,T,batch", [(4, 1, 300), (4, 7, 70), (4, 33, 85), (4, 257, 31), (4, 600, 17),
                                        (5, 1, 40), (5, 4, 300), (5, 65, 70), (8, 300, 13), (8, 9, 130),
                                        (9, 1, 70), (9, 5, 300), (9, 257, 5), (16, 4, 130), (16, 70, 21)])
def test_batches(nx, T, batch, dtype):
    p = W.random_stable(5 + nx, nx, 2, T, 1, tf=min(2.0, 0.05 * T), time_varying=False)
    dp = lqt.DeviceProblem.from_problems([p], dtype=dtype)
    scale = torch.linspace(0.5, 2.0, batch, dtype=dtype, device="cuda")
    for k in ("t", "Q", "R", "r", "Qf", "rf", "x0"):
        a = getattr(dp, k)
        a = a.expand(batch, *a.shape[1:]).contiguous()
        if k in ("r", "x0", "rf"):  # v, x and u follow the inputs linearly, S does not change
            a = a * scale.view(-1, *[1] * (a.dim() - 1))
        setattr(dp, k, a)
    dp.batch = batch
    got = lqt.solve(dp, keep_elements=True)
    S, v = lqt.scan_value(dp, got["elts"])
    torch.cuda.synchronize()
    ref = O.solve(p)
    for k, x in (("S", got["S"]), ("v", got["v"]), ("x", got["x"]), ("u", got["u"]), ("S", S), ("v", v)):
        want = torch.as_tensor(ref[k], device="cuda")
        x = x.double()
        if k != "S":
            x = x / scale.double().view(-1, *[1] * (x.dim() - 1))
        e = float((x - want).abs().max() / want.abs().max())
        assert e < TOL[dtype], f"{k}: {e:.3e}"
