"""The scans of the tree kernels give the same bits in every call, also where the last group of a
stage is ragged (nodes without a pair in waves that have some: 10 to 15 slots of 16, and the like of
32), with other work on the device in between."""
import pytest
import torch

from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,T,dtype", [
    (4, 21, torch.float64), (4, 27, torch.float64), (4, 8 * 43 + 3, torch.float64), (5, 11, torch.float64),
    (7, 3001, torch.float32), (7, 3001, torch.float64), (8, 4 * 29, torch.float64),
    (12, 4 * 7, torch.float64), (16, 4 * 11 + 1, torch.float32)])
def test_same_bits_every_call(nx, T, dtype):
    dp = lqt.DeviceProblem.from_problems([W.random_stable(nx + T, nx, 2, T, 2, tf=2.0)], dtype=dtype)
    first = {k: v.clone() for k, v in lqt.solve(dp).items()}
    noise = torch.randn(1 << 20, device="cuda")
    out, ws = lqt.solve(dp), lqt.workspace(dp, lqt.CALL_SOLVE)
    for i in range(30):
        if i % 3 == 0:
            noise = noise.sin()
        lqt.solve(dp, out, ws)
        for k in ("S", "v", "x", "u"):
            assert torch.equal(out[k], first[k]), (i, k)
