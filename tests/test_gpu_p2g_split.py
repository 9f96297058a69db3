"""GPU: P2G with two waves per block (up to P2G_SPLIT_MAX_N = 393,216 particles
in 3D) against one wave per block (above it): both add the same terms in the
same order, so particles in the same cells give the same grid bit for bit
whichever form runs.  A set of n particles, alone and with a far cloud that
takes the count past the line, for blocks of one particle up to cells of
hundreds, with cell ranges from the sort and counted from the keys."""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import CLOUDS, _announce, _cloud

pytestmark = pytest.mark.gpu

LINE = 3 << 17


def _grid(x, flags, seed, n_near):
    """P2G grid of the near particles' blocks, by block key."""
    import torch
    from paper_2605_28525_amd import mpm as M
    w = wl.tiny_3d(n=48, ties=False)
    w.dx, w.cells = 0.25, (160, 160, 160)
    st = wl.rest_state(x)
    rng = np.random.default_rng(seed)
    for k, sc in (("v", 1.0), ("C", 2.0), ("tau", 100.0)):  # the near particles' values do not depend on the far ones
        st[k][:, :n_near] = rng.normal(0, sc, st[k][:, :n_near].shape).astype(np.float32)
    for k, a in st.items():
        setattr(w, k, a)
    sim = M.Simulation(w, flags=flags, block_capacity=16384)
    try:
        M.mpm_sparse_build(sim.ctx, sim.a.view())  # a stable sort in every mode
        M.mpm_p2g(sim.ctx, sim.a.view())
        nb, _ = M.mpm_active_count(sim.ctx)
        k = torch.empty(nb, dtype=torch.int64, device="cuda")
        m = torch.empty_like(k)
        M.mpm_get_active(sim.ctx, k, m, nb)
        g = torch.empty(nb * 64, 4, dtype=torch.float32, device="cuda")
        M.mpm_get_grid(sim.ctx, g, nb)
        rc, f = sim.status()
        assert rc == 0, f
        return dict(zip(k.cpu().numpy().tolist(), g.reshape(nb, 64, 4).cpu().numpy()))
    finally:
        sim.close()


@pytest.mark.parametrize("flags", ["full", "scan", "ordered"])
@pytest.mark.parametrize("name", list(CLOUDS))
def test_two_waves_equal_one(name, flags):
    from paper_2605_28525_amd import mpm as M
    fl = {"full": M.MPM_FLAG_FULL_SORT, "scan": M.MPM_FLAG_SCAN_BUILD,
          "ordered": M.MPM_FLAG_DETERMINISTIC_ORDER}[flags]
    near = _cloud(3, CLOUDS[name], 3)
    n = near.shape[1]
    far = (np.random.default_rng(8).uniform(80, 140, (3, LINE + 1 - n)) * 0.25).astype(np.float32)
    _announce("P2G two waves", name, flags, n)
    two = _grid(near, fl, 21, n)
    one = _grid(np.concatenate([near, far], axis=1), fl, 21, n)
    assert len(two) > 0
    for k, g in two.items():
        assert np.array_equal(g, one[k]), k
