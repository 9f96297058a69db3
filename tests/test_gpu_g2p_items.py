"""GPU: G2P with one, two and three particles per thread (work items of up to
256, 512 and 768 particles): the step's particles are the same bits whatever
the size of the work items, with a stable sort (the order does not depend on
the items).  Item sizes around a thread's share, blocks around an item."""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import CLOUDS, _announce, _cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("name", list(CLOUDS))
def test_item_size_does_not_change_a_step(name, dim):
    from paper_2605_28525_amd import mpm as M
    x = _cloud(dim, CLOUDS[name], 17)
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt = dim, 0.25, (20, 40, 16)[:dim], 1e-4
    st = wl.rest_state(x)
    st["v"] = np.random.default_rng(2).normal(0, 0.05, st["v"].shape).astype(np.float32)
    for k, a in st.items():
        setattr(w, k, a)
    ref = None
    for chunk in (64, 255, 256, 257, 512, 513, 768):
        _announce("G2P items", name, dim, chunk)
        sim = M.Simulation(w, flags=M.MPM_FLAG_FULL_SORT)
        try:
            M.mpm_set_tuning(sim.ctx, chunk=chunk)
            sim.step(3)
            rc, f = sim.status()
            assert rc == 0, f
            got = dict(sim.a.to_arrays(), id=sim.a.ids())
        finally:
            sim.close()
        ref = ref or got
        for k in ref:
            assert np.array_equal(ref[k], got[k]), (chunk, k)


def test_kept_item_size_is_the_general_default():
    """A workgroup size set alone is checked against work items of 512, also in
    a small context, whose items are of 256."""
    from paper_2605_28525_amd import mpm as M
    sim = M.Simulation(wl.collapse_2d())
    try:
        for blk in (64, 128):
            with pytest.raises(M.MPMError):
                M.mpm_set_tuning(sim.ctx, g2p_block=blk)
        M.mpm_set_tuning(sim.ctx, g2p_block=256)
        M.mpm_set_tuning(sim.ctx, chunk=128, g2p_block=64)
        M.mpm_set_tuning(sim.ctx, g2p_block=128)
        sim.step(2)
        assert sim.status()[0] == 0
    finally:
        sim.close()
