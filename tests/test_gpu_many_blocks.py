"""GPU: steps of contexts with room for many blocks.  Above 2^16 blocks a small step
keeps P2G's second pass, above 2^18 the re-sort keeps its scan as launches of its
own.  The kernels by name, from the profiler's record, and the steps against those
of a context with just enough room (the re-sort may permute a cell's particles:
float32 sums in another order, 1e-5 of a field's largest value); scattered
particles, which have several blocks each, must not pay for the re-sort more
than a sort from scratch does.
"""
import re

import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import _announce, _far_cloud, _state
from test_gpu_tabsort_full import step_times

pytestmark = pytest.mark.gpu

FIELDS = ("x", "v", "C", "F", "tau")


def _workload(x, cells):
    w = wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt = 2, 0.25, cells, 1e-4
    w.p_vol0 = w.dx ** 2 / 4
    w.p_mass = w.rho * w.p_vol0
    for k, a in _state(x, 6).items():
        setattr(w, k, a)
    return w


def _steps(w, capacity):
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2605_28525_amd import mpm as M
    sim = M.Simulation(w, block_capacity=capacity)
    try:
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            sim.step(4)
            torch.cuda.synchronize()
        sim.step(5)
        rc, f = sim.status()
        assert rc == 0, f
        assert np.array_equal(np.sort(sim.a.ids()), np.arange(w.n))
        by = np.argsort(sim.a.ids())
        state = {k: sim.a.to_arrays()[k][:, by] for k in FIELDS}
    finally:
        sim.close()
    return state, {re.sub(r"^void mpmx::|\(.*$", "", e.name) for e in p.events()}


@pytest.mark.parametrize("capacity,gathers,folded", [
    (1 << 16, True, True), ((1 << 16) + 1, False, True), (1 << 18, False, True), ((1 << 18) + 1, False, False)])
def test_forms_by_the_room_for_blocks(capacity, gathers, folded):
    _announce("many blocks", capacity)
    w = _workload(_far_cloud(2, 6000, 11), (2100, 2100))   # 276,676 blocks
    ref, _ = _steps(w, 4096)
    got, names = _steps(w, capacity)
    for k in FIELDS:
        assert np.abs(got[k] - ref[k]).max() <= 1e-5 * np.abs(ref[k]).max(), k
    if not any(n.startswith("k_g2p<") for n in names):
        pytest.skip("the profiler recorded no kernels")
    assert any(re.match(r"k_g2p<2, 256, \d, true>", n) for n in names) == gathers
    assert f"k_rs_place<2, {'false' if folded else 'true'}>" in names
    assert f"k_rs_place<2, {'true' if folded else 'false'}>" not in names


def test_scattered_particles_re_sort_as_fast_as_they_sort():
    """262,144 particles over about 518,000 blocks: 1323 us a step re-sorted, 1339
    sorted from scratch; with the folded scan 1684."""
    from paper_2605_28525_amd import mpm as M
    rng = np.random.default_rng(3)
    w = _workload((0.25 * rng.uniform(4, 5996, (2, 262144))).astype(np.float32), (6000, 6000))
    _announce("scattered particles", w.n)
    sims = [M.Simulation(w, flags=flags, block_capacity=4 * w.n) for flags in (0, M.MPM_FLAG_FULL_SORT)]
    try:
        t = step_times(sims, 10)
    finally:
        for sim in sims:
            sim.close()
    print("us per step", [round(1e6 * v, 1) for v in t])
    assert t[0] < 1.12 * t[1]
