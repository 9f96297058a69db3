"""GPU: an ensemble whose instances together occupy more blocks than one
instance's domain has.  Each instance all but fills its domain of 64 blocks, so three
of them need about 190; with the default capacity, with one asked for, and grown by
the overflow rebuild.  Every instance steps as it does alone (parity bar).
"""
import numpy as np
import pytest

from parity_util import RTOL, assert_field, tau_floor
from paper_2605_28525_amd import workloads as wl
from test_gpu_ensemble import FIELDS, _announce, _by_id

pytestmark = pytest.mark.gpu

N_INST, N_EACH = 3, 1500


def _member(seed):
    """Particles scattered over every block of a 12^3-cell domain, at rest: at
    two per cell, with the confining stretch that keeps them elastic."""
    rng = np.random.default_rng(seed)
    w = wl.tiny_3d(n=48, ties=False)
    w.dx, w.cells, w.dt = 0.25, (12, 12, 12), 1e-4
    x = (0.25 * rng.uniform(0.7, 11.3, (3, N_EACH))).astype(np.float32)
    st = wl.rest_state(x)
    st["F"][[0, 4, 8]] = 0.999
    for k, a in st.items():
        setattr(w, k, a)
    return w


def _blocks(w):
    b = np.floor(w.x.astype(np.float64) / w.dx - 0.5).astype(np.int64)
    assert b.min() >= 0 and b.max() + 2 <= 12
    hit = np.zeros((4, 4, 4), bool)
    for m in range(8):
        q = [(b[a] + (2 if (m >> a) & 1 else 0)) >> 2 for a in range(3)]
        hit[q[0], q[1], q[2]] = True
    return int(hit.sum())


def _ensemble():
    members = [_member(40 + i) for i in range(N_INST)]
    for i, m in enumerate(members):
        m.E *= 1.0 + 0.1 * i
    arr = {k: np.concatenate([getattr(m, k) for m in members], axis=1) for k in FIELDS}
    inst = np.repeat(np.arange(N_INST), N_EACH).astype(np.int32)
    return wl.Ensemble(name="full domains", members=members, steps=1, inst=inst, **arr)


@pytest.mark.parametrize("name,flag,capacity", [
    ("default", None, 0), ("asked", None, 192), ("ordered", "MPM_FLAG_DETERMINISTIC_ORDER", 0),
    ("full", "MPM_FLAG_FULL_SORT", 0), ("grown", "MPM_FLAG_SYNC_REBUILD", 8)])
def test_instances_fill_their_domains(name, flag, capacity):
    from paper_2605_28525_amd import mpm as M
    ens = _ensemble()
    want = sum(_blocks(m) for m in ens.members)
    assert 2 * 64 < want <= 64 * N_INST
    _announce("ensemble capacity", name, ens.n, want)
    flags = getattr(M, flag) if flag else 0
    batch = M.Simulation(ens, flags=flags, block_capacity=capacity)
    singles = [M.Simulation(m, flags=flags, block_capacity=capacity and 64) for m in ens.members]
    try:
        M.mpm_sparse_build(batch.ctx, batch.a.view())
        rc, f = batch.status()
        assert rc == 0, f
        assert M.mpm_active_count(batch.ctx)[0] == want
        for sim in [batch] + singles:
            sim.step(3)
            rc, f = sim.status()
            assert rc == 0, f
        assert np.array_equal(np.sort(batch.a.ids()), np.arange(ens.n))
        for i, (m, sim) in enumerate(zip(ens.members, singles)):
            got, ref = _by_id(batch.a, ens.member_positions(i)), _by_id(sim.a, np.arange(m.n))
            for k in FIELDS:
                assert_field(f"inst {i} {k}", got[k], ref[k], RTOL, atol=tau_floor(m) if k == "tau" else 0.0)
    finally:
        batch.close()
        for s in singles:
            s.close()
