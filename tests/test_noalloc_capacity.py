"""Batches of short horizons at nx >= 5 that lqt_solve_noalloc takes: their scratch fits the fixed array
(on the CPU; the solves themselves are in test_gpu_noalloc_short.py).  Each count is the largest that
fits when a tree record is kept for every fourth block and every fourth node above."""
import ctypes

import pytest

from paper_2212_11744_amd import lqt


@pytest.mark.parametrize("nx,T,dtype,batch", [
    (5, 4, lqt.LQT_F64, 49489), (5, 16, lqt.LQT_F64, 14873), (8, 16, lqt.LQT_F64, 6428),
    (8, 17, lqt.LQT_F32, 7506), (9, 1, lqt.LQT_F64, 17421), (12, 17, lqt.LQT_F32, 3546),
    (16, 4, lqt.LQT_F64, 5938), (16, 17, lqt.LQT_F64, 1030), (16, 70, lqt.LQT_F32, 591)])
def test_short_horizons_fit(nx, T, dtype, batch):
    d = lqt.Dims(nx=nx, nu=1, T=T, n_steps=4, batch=batch, dtype=dtype, F_sampled=0, L_sampled=0,
                 has_c=0, lti=0)
    need = lqt.lib().lqt_noalloc_scratch_size(ctypes.byref(d))
    assert 0 < need <= lqt.NOALLOC_SCRATCH_BYTES
