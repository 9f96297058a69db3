"""GPU: mpm_step of several steps, whose G2P forms the nodes it reads itself up to
65,536 particles (G2P_GATHER_MAX_N), against the same steps one call each, whose
grids are summed and updated by P2G's second pass: particles and the last grid
bit for bit (a stable sort: the particles' order is the same)."""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import CLOUDS, _announce, _cloud

pytestmark = pytest.mark.gpu


def _workload(name):
    if name == "ensemble":
        return wl.ensemble_small(n_instances=3)
    if name == "landslide_crop":
        return wl.landslide_crop()   # terrain boundary
    if name == "collapse_2d":
        return wl.perturbed(wl.collapse_2d(), seed=5)
    cloud, dim = name.rsplit("_", 1)
    w = wl.tiny_3d(n=48, ties=False) if dim == "3d" else wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt = int(dim[0]), 0.25, (20, 40, 16)[:int(dim[0])], 1e-4
    for k, a in wl.rest_state(_cloud(w.dim, CLOUDS[cloud], 23)).items():
        setattr(w, k, a)
    return w


@pytest.mark.parametrize("chunk", [256, 512])
@pytest.mark.parametrize("name", ["ensemble", "landslide_crop", "collapse_2d", "few_2d", "few_3d", "block_1025_2d",
                                  "block_1025_3d"])
def test_steps_together_equal_steps_apart(name, chunk):
    import torch
    from paper_2605_28525_amd import mpm as M
    w = _workload(name)
    _announce("G2P gather", name, chunk, w.n)
    got = []
    for together in (True, False):
        sim = M.Simulation(w, flags=M.MPM_FLAG_FULL_SORT)
        try:
            M.mpm_set_tuning(sim.ctx, chunk=chunk)
            for _ in range(1 if together else 4):
                sim.step(4 if together else 1)
            rc, f = sim.status()
            assert rc == 0, f
            nb, _ = M.mpm_active_count(sim.ctx)
            nodes = 64 if getattr(w, "dim", 3) == 3 else 16
            k = torch.empty(nb, dtype=torch.int64, device="cuda")
            m = torch.empty_like(k)
            M.mpm_get_active(sim.ctx, k, m, nb)
            g = torch.empty(nb * nodes, 4, dtype=torch.float32, device="cuda")
            M.mpm_get_grid(sim.ctx, g, nb)
            o = torch.argsort(k)
            got.append(dict(sim.a.to_arrays(), id=sim.a.ids(), keys=k[o].cpu().numpy(),
                            grid=g.reshape(nb, nodes, 4)[o].cpu().numpy()))
        finally:
            sim.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
