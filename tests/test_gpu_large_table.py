"""GPU: block hash tables from one tile of the compaction (2048 slots) up to many
times what the blocks need, around 2^21 slots, above which the tiles' running
sums are made by a launch of their own.  The size changes only where blocks lie
in the table: the active set and (with a stable sort) every particle are the
same, and a step may not grow with the square of the table.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_tabsort import _announce, _far_cloud, _state
from test_gpu_tabsort_full import step_times

pytestmark = pytest.mark.gpu


def _workload(dim, n):
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt = dim, 0.25, (40, 48, 44)[:dim], 1e-4
    w.p_vol0 = w.dx ** dim / 2 ** dim
    w.p_mass = w.rho * w.p_vol0
    for k, a in _state(_far_cloud(dim, n, 11), 6).items():
        setattr(w, k, a)
    return w


@pytest.mark.parametrize("flags", ["MPM_FLAG_FULL_SORT", "MPM_FLAG_DETERMINISTIC_ORDER", "MPM_FLAG_ADJOINT", ""])
@pytest.mark.parametrize("dim", [2, 3])
def test_table_size_does_not_change_a_step(dim, flags):
    import torch
    from paper_2605_28525_amd import mpm as M
    w = _workload(dim, 5000)
    ref = None
    for log2 in (11, 12, 21, 22, 23):
        _announce("large table", dim, flags, log2)
        sim = M.Simulation(w, flags=getattr(M, flags) if flags else 0, block_capacity=1024, hash_capacity_log2=log2)
        try:
            sim.step(3)
            rc, f = sim.status()
            assert rc == 0, f
            M.mpm_sparse_build(sim.ctx, sim.a.view())
            nb, touched = M.mpm_active_count(sim.ctx)
            assert nb == touched
            kh = torch.empty(nb, dtype=torch.int64, device="cuda")
            mh = torch.empty_like(kh)
            M.mpm_get_active(sim.ctx, kh, mh, nb)
            act = np.stack([kh.cpu().numpy(), mh.cpu().numpy()])
            if flags != "MPM_FLAG_DETERMINISTIC_ORDER":  # (slot order)
                act = act[:, np.argsort(act[0])]
            by = np.argsort(sim.a.ids())
            got = {k: a[:, by] for k, a in sim.a.to_arrays().items()}
            if flags:
                got["ids"] = sim.a.ids()
        finally:
            sim.close()
        ref = ref or (act, got)
        assert np.array_equal(ref[0], act), log2
        for k in got:
            if flags:
                assert np.array_equal(ref[1][k], got[k]), (log2, k)
            else:  # the re-sort may permute a cell's particles: sums in another order
                scale = np.abs(ref[1][k]).max()
                assert np.abs(ref[1][k] - got[k]).max() <= 1e-5 * scale, (log2, k)


def test_step_does_not_grow_with_the_square_of_the_table():
    """262,144 particles with 2^17 and 2^24 slots: the larger table is read once more
    (16.8 million keys), 71 and 113 us; with every tile adding up all tiles' counts it
    was 321 us."""
    from paper_2605_28525_amd import mpm as M
    w = wl.collapse_3d(seed=2, scale=2)
    _announce("large table, time", w.n)
    sims = [M.Simulation(w, hash_capacity_log2=log2) for log2 in (17, 24)]
    try:
        t = step_times(sims, 20)
    finally:
        for sim in sims:
            sim.close()
    print("us per step", [round(1e6 * v, 1) for v in t])
    assert t[1] < 2.5 * t[0]
