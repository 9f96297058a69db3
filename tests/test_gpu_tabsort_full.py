"""GPU: the counting sort where blocks are full, and where they are small.  Contexts
with up to 96 particles in a block at rest order blocks of up to 128 by a wave each.
Otherwise (and above 128) a workgroup orders a block.  Blocks of up to 1024 particles
pass through registers, larger ones are read twice, up to 3072 or (contexts
whose cells at rest hold more than 32 particles in 3D) 8192 of them in LDS, the rest
by one wave; contexts with more than 110 particles in a cell at rest, or 4608 in a
block (72 in a 3D cell), keep the radix sort.  The order must be the stable one in each, element by element, and a
step that sorts from scratch must not cost a multiple of one that re-sorts.
"""
import math
import time

import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import _announce, _cloud, _state, expected_order

pytestmark = pytest.mark.gpu

# cells of a row (four to a block): particles per cell
ROWS = {
    64: [64, 0, 0, 0, 1, 2, 3, 58, 20, 21, 22],
    127: [100, 27, 0, 0, 128, 0, 0, 0, 1],
    129: [32, 32, 32, 33, 64, 0, 64, 0, 700],
    1023: [300, 300, 300, 123, 5],
    1024: [1, 1000, 23, 0, 5],
    1025: [256, 257, 256, 256, 0, 9],
    2049: [2000, 0, 48, 1, 1026, 3],
    3072: [768, 768, 768, 768, 31],
    3073: [768, 769, 768, 768, 3072],
    8192: [2048, 2048, 2048, 2048, 4097],
    8193: [2048, 2048, 2049, 2048, 100],
}


def _workload(dim, per_cell, x, seed):
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt = dim, 0.25, (20, 40, 16)[:dim], 1e-5
    w.p_vol0 = w.dx ** dim / per_cell
    w.p_mass = w.rho * w.p_vol0
    for k, a in _state(x, seed).items():
        setattr(w, k, a)
    return w


@pytest.mark.parametrize("flags", ["full", "scan", "dense", "adjoint"])
@pytest.mark.parametrize("per_cell", [1, 4, 8, 64, 72, 73, 110, 111])
@pytest.mark.parametrize("dim", [2, 3])
def test_order_of_full_blocks(dim, per_cell, flags):
    import torch
    from paper_2605_28525_amd import mpm as M
    fl = {"full": M.MPM_FLAG_FULL_SORT, "scan": M.MPM_FLAG_SCAN_BUILD, "dense": 0, "adjoint": M.MPM_FLAG_ADJOINT}[flags]
    for block, row in ROWS.items():
        x = _cloud(dim, row, seed=block)
        w = _workload(dim, per_cell, x, 3)
        _announce("full blocks", dim, per_cell, flags, block, w.n)
        sim = M.Simulation(w, flags=fl, grid_mode=M.MPM_GRID_DENSE if flags == "dense" else M.MPM_GRID_SPARSE)
        try:
            for step in range(2):  # the second from the first one's output order
                xin = sim.a.to_arrays()["x"]
                M.mpm_sparse_build(sim.ctx, sim.a.view())
                M.mpm_p2g(sim.ctx, sim.a.view())
                M.mpm_grid_update(sim.ctx)
                M.mpm_g2p(sim.ctx, sim.a.view(), sim.b.view())
                order = torch.empty(w.n, dtype=torch.int32, device="cuda")
                M.mpm_get_order(sim.ctx, order, w.n)
                rc, f = sim.status()
                assert rc == 0, f
                assert np.array_equal(order.cpu().numpy(), expected_order(xin, w.dx, w.cells, dim)), (block, step)
                sim.a, sim.b = sim.b, sim.a
        finally:
            sim.close()


def step_times(sims, steps):
    """Median seconds per step of each simulation, lap by lap in turn."""
    import torch
    laps = [[] for _ in sims]
    for _ in range(7):
        for lap, sim in zip(laps, sims):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sim.step(steps)
            torch.cuda.synchronize()
            lap.append((time.perf_counter() - t0) / steps)
    assert all(sim.status()[0] == 0 for sim in sims)
    return [sorted(lap)[2] for lap in laps]


def _column(dim, side, per_axis):
    rng = np.random.default_rng(3)
    dx, E, rho = 0.01, 1e6, 2000.0
    x = wl.stratified_cells([4] * dim, [4 + side] * dim, dx, per_axis, rng)
    vol = dx ** dim / per_axis ** dim
    w = wl.Workload(name="column", dim=dim, dx=dx, cells=(side + 32,) * dim, steps=20, gravity=(0.0, -9.81, 0.0),
                    dt=0.25 * dx / math.sqrt(E * 0.7 / (1.3 * 0.4) / rho), model="dp", E=E, nu=0.3, rho=rho,
                    friction_deg=30.0, ppc=per_axis ** dim, p_vol0=vol, p_mass=rho * vol)
    for k, a in wl.rest_state(x).items():
        setattr(w, k, a)
    return w


@pytest.mark.parametrize("dim,side,per_axis", [(3, 21, 3), (3, 13, 5), (2, 51, 10)])
def test_a_full_sort_is_not_a_multiple_of_a_step(dim, side, per_axis):
    """About 260,000 particles at 27, 125 and (2D) 100 per cell: a step that sorts
    from scratch takes 1.1 to 1.3 times one that re-sorts; with one wave per full
    block it took 1.7 to 2.4 times."""
    from paper_2605_28525_amd import mpm as M
    w = _column(dim, side, per_axis)
    _announce("cost of a full sort", dim, per_axis, w.n)
    sims = [M.Simulation(w, flags=flags) for flags in (0, M.MPM_FLAG_FULL_SORT)]
    try:
        t = step_times(sims, 20)
    finally:
        for sim in sims:
            sim.close()
    print("ratio", round(t[1] / t[0], 2), "us per step", [round(1e6 * v, 1) for v in t])
    assert t[1] < 1.5 * t[0]
