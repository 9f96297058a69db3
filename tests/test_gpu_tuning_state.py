"""GPU: which calls a change of the work item size leaves a build for.  The
size in force is checked against the one asked for last (512 where none was), also
in a small context, which keeps items of 256 until a size is asked for: asking
for 512 there keeps the build, asking for 256 needs a new one, as in any
context.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _phases(sim, between=None):
    from paper_2605_28525_amd import mpm as M
    a, b = sim.a.view(), sim.b.view()
    M.mpm_sparse_build(sim.ctx, a)
    if between:
        between()
    M.mpm_p2g(sim.ctx, a)
    if between:
        between()
    M.mpm_grid_update(sim.ctx)
    M.mpm_g2p(sim.ctx, a, b)
    rc, f = sim.status()
    assert rc == 0, f
    return dict(sim.b.to_arrays(), id=sim.b.ids())


@pytest.mark.parametrize("asked", [0, 512])
def test_general_size_keeps_a_build(asked):
    from paper_2605_28525_amd import mpm as M
    got = []
    for between in (False, True):
        sim = M.Simulation(wl.collapse_2d(), flags=M.MPM_FLAG_FULL_SORT)
        try:
            if asked:
                M.mpm_set_tuning(sim.ctx, chunk=asked)
            got.append(_phases(sim, (lambda: M.mpm_set_tuning(sim.ctx, chunk=512)) if between else None))
            got.append(_phases(sim))   # the next build takes the new size
        finally:
            sim.close()
    for k in got[0]:   # a stable sort: the particles do not depend on the items
        assert np.array_equal(got[0][k], got[2][k]), k
        assert np.array_equal(got[1][k], got[3][k]), k


@pytest.mark.parametrize("first", [0, 512, 128])
@pytest.mark.parametrize("size", [64, 256, 768])
def test_another_size_needs_a_new_build(first, size):
    from paper_2605_28525_amd import mpm as M
    sim = M.Simulation(wl.collapse_2d())
    try:
        if first:
            M.mpm_set_tuning(sim.ctx, chunk=first)
        M.mpm_sparse_build(sim.ctx, sim.a.view())
        M.mpm_set_tuning(sim.ctx, chunk=size)
        with pytest.raises(M.MPMError):
            M.mpm_p2g(sim.ctx, sim.a.view())
        _phases(sim)
    finally:
        sim.close()
