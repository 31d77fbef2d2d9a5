"""Tree stages of the value and trajectory scans at their edges, vs the CPU oracle.

A slot of a workgroup takes 1, 2, 4 or 8 blocks, a group 32 (nx <= 4), 16 (nx <= 8) or 4 slots, and the
last stage up to 8 (nx >= 9: 4) nodes per slot: horizons of one group take one launch, longer ones
add stages.  The horizons below are the last of a shape and the first of the next, with ragged
last slots and groups; nx = 4 in FP64 leaves these kernels at 257 groups, the element build of nx = 3
at 8193 blocks and of nx = 4 at 32769.  Tolerances: normwise 1e-9 in FP64 and 1e-4 in FP32 against
the FP64 oracle, as for every other solve."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import relerr
from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-9, torch.float32: 1e-4}


def _check(ps, dtype=torch.float64, check=None):
    out = lqt.solve(lqt.DeviceProblem.from_problems(ps, dtype=dtype))
    torch.cuda.synchronize()
    for b in check if check is not None else range(len(ps)):
        ref = O.solve(ps[b])
        for k in ("S", "v", "x", "u"):
            e = relerr(out[k][b].cpu().numpy().astype(np.float64), ref[k])
            assert e < TOL[dtype], f"problem {b} {k}: {e:.3e}"


@pytest.mark.parametrize("T", [1, 2, 5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513,
                               8191, 8193, 65537])
def test_nx4(T):
    _check([W.point_mass(T, T, 1, 0.0, 0.01 * T if T < 1000 else 10.0)])


@pytest.mark.parametrize("T", [33, 130, 600])
def test_nx4_sampled_with_drift(T):
    p = W.random_stable(T, 4, 3, T, 3, tf=2.0)
    p.c = 0.3 * np.sin(np.linspace(0, 3, p.r.shape[0]))[:, None] * np.arange(1.0, 5.0)
    _check([p])


@pytest.mark.parametrize("T,batch", [(33, 3), (257, 3), (64, 256), (64, 257), (257, 128), (257, 129)])
def test_nx4_batch(T, batch):
    _check([W.point_mass(7 * T + b, T, 1, 0.0, 2.0) for b in range(batch)], check=(0, batch - 1))


@pytest.mark.parametrize("nx,T", [(5, 1), (5, 16), (5, 17), (5, 64), (5, 65), (5, 8192), (5, 8193),
                                  (9, 1), (9, 4), (9, 5), (9, 16), (9, 17), (9, 256), (9, 257),
                                  (9, 4097)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_wave_sizes(nx, T, dtype):
    _check([W.random_stable(nx * T, nx, 2, T, 1, tf=min(2.0, 0.05 * T))], dtype)


@pytest.mark.parametrize("nx,T,dtype", [(3, 8192, torch.float64), (3, 8193, torch.float64),
                                        (3, 8192, torch.float32), (4, 8192, torch.float32),
                                        (4, 8193, torch.float32), (4, 32768, torch.float64),
                                        (4, 32769, torch.float64)])
def test_build_rule(nx, T, dtype):
    _check([W.random_stable(nx + T, nx, 2, T, 1, tf=2.0)], dtype)


# The value scan in three launches (nx = 3, 4; tiles of 64 x 2, 4 or 8 blocks): one block short of and
# past its first horizon (nx = 4; nx = 3 takes it from 8193 to 32768 blocks, see test_build_rule), whole
# and ragged tiles, and the changes of the blocks per lane.
@pytest.mark.parametrize("nx,T,batch,dtype", [
    (3, 512, 1, torch.float64), (3, 513, 1, torch.float64), (3, 640, 2, torch.float32),
    (3, 16385, 1, torch.float64), (3, 32768, 1, torch.float32), (3, 32769, 1, torch.float64),
    (4, 513, 1, torch.float32), (4, 1023, 3, torch.float32), (4, 16384, 1, torch.float32),
    (4, 65537, 1, torch.float64), (4, 131073, 1, torch.float64), (4, 65537, 2, torch.float64)])
def test_split_value_scan(nx, T, batch, dtype):
    if batch == 1:
        ps = [W.random_stable(nx + T, nx, 2, T, 1, tf=2.0)]
    else:
        ps = [W.random_stable(5, nx, 2, T, 1, tf=2.0, time_varying=False) for _ in range(batch)]
        for b, p in enumerate(ps):
            p.r, p.x0 = p.r * (1.0 + b), p.x0 - b
    _check(ps, dtype)


def _grid(T, uneven):
    t = np.linspace(0.0, 10.0, T + 1)
    if uneven is not None:  # one block longer by 1e-6 of its length
        t[uneven + 1:] += 1e-6 * (t[1] - t[0])
    return t


# Constant F and L beyond 2^19 blocks (the elements from tables to first order in the blocks' lengths
# where the grid is even to 2^-27, the general build elsewhere, problem by problem).
@pytest.mark.parametrize("T,n,uneven", [(524289, 1, [None]), (524289, 5, [None]), (524301, 2, [0]),
                                        (524301, 1, [524300]), (262145, 2, [None, 131000])])
def test_even_grid(T, n, uneven):
    _check([W.point_mass(3 + b, T, n, t_grid=_grid(T, u)) for b, u in enumerate(uneven)])


def test_even_grid_nx3():
    ps = [W.random_stable(8, 3, 2, 32768, 1, tf=2.0, time_varying=False) for _ in range(17)]
    for b, p in enumerate(ps):
        p.r = p.r * (1.0 + 0.1 * b)
    _check(ps, check=(0, 16))


@pytest.mark.parametrize("nx,T,n,batch", [(4, 70001, 5, 1), (4, 140001, 2, 1), (4, 300007, 1, 1),
                                          (3, 1025, 4, 2)])
def test_time_invariant_reduction(nx, T, n, batch):
    ps = [W.random_stable(8, nx, 2, T, n, tf=2.0, time_varying=False) for _ in range(batch)]
    for b, p in enumerate(ps):
        p.r = p.r * (1.0 + 0.1 * b)
    dp = lqt.DeviceProblem.from_problems(ps)
    dp.lti = True  # even to rounding, which is more than 1e-12 of such short blocks
    out = lqt.solve(dp)
    for b, p in enumerate(ps):
        ref = O.solve(p)
        for k in ("S", "v", "x", "u"):
            e = relerr(out[k][b].cpu().numpy(), ref[k])
            assert e < TOL[torch.float64], f"problem {b} {k}: {e:.3e}"
