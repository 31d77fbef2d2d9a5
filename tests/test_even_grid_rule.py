"""Which solves take the tables of the even-grid path, on the CPU: their workspace has room for them.
Without a drift (has_c = 0) and with one, which never takes them, the layouts differ by nothing else."""
import ctypes

import pytest

from paper_2212_11744_amd import lqt


def _size(**kw):
    base = dict(nx=4, nu=2, T=1024, n_steps=4, batch=1, dtype=lqt.LQT_F64, F_sampled=0, L_sampled=0,
                has_c=0, lti=0)
    base.update(kw)
    return lqt.lib().lqt_workspace_size(ctypes.byref(lqt.Dims(**base)), lqt.CALL_SOLVE)


@pytest.mark.parametrize("T,n,batch,tables", [
    (600, 75, 1000, False),      # 2416 block integrations per problem for the tables, 600 for the build
    (2303, 4, 1000, False), (2304, 4, 1000, True),   # 16 times 4 (2 n + 1) nx
    (2 ** 19, 4, 1, False), (2 ** 19 + 1, 4, 1, True), (2 ** 18, 4, 3, True),
    (2 ** 20, 4, 1, True), (2 ** 20, 2047, 1, True), (2 ** 20, 2048, 1, False)])
def test_tables_only_where_they_are_a_sixteenth_of_the_build(T, n, batch, tables):
    assert (_size(T=T, n_steps=n, batch=batch) > _size(T=T, n_steps=n, batch=batch, has_c=1)) == tables
