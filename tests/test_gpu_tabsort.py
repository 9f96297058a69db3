"""GPU: the full sort by counting in a table of owner blocks against a stable
argsort on the CPU, element by element: the permutation that mpm_g2p applies
(mpm_get_order) must be the stable order by (owner block, base cell), stored
rank-major inside each block, whatever order the input had.

Sizes are where the sort changes its way: cells of up to and past a wave,
blocks of up to and past 1024 (ordered in LDS, or by radix passes), particle
counts around a workgroup, and domains around a tile of the table.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl

pytestmark = pytest.mark.gpu

IL_ROUNDS = 32


def _announce(*a):
    print("CASE", *a, flush=True)


def expected_order(x, dx, cells, dim, inst=None):
    """Permutation of the stable sort, rank-major per block."""
    b = np.floor(x[:dim].astype(np.float64) * (1.0 / dx) - 0.5).astype(np.int64)
    own, loc = b >> 2, b & 3
    nblk = [(c + 4) // 4 for c in cells]
    lin = own[0] + nblk[0] * (own[1] + (nblk[1] * own[2] if dim == 3 else 0))
    cell = loc[0] + 4 * loc[1] + (16 * loc[2] if dim == 3 else 0)
    if inst is not None:
        lin = lin + inst.astype(np.int64) * int(np.prod(nblk[:dim]))
    order = np.lexsort((np.arange(lin.size), cell, lin))
    # rank of each particle in its cell, then (block, rank, cell) for ranks
    # below IL_ROUNDS and (block, cell, rank) after them
    key = lin[order] * 4 ** dim + cell[order]
    first = np.r_[0, np.nonzero(np.diff(key))[0] + 1]
    rank = np.arange(key.size) - np.repeat(first, np.diff(np.r_[first, key.size]))
    lo, c = lin[order], cell[order]
    late = rank >= IL_ROUNDS
    return order[np.lexsort((np.where(late, rank, c), np.where(late, c, 0), np.where(late, IL_ROUNDS, rank), lo))]


def _state(x, seed):
    st = wl.rest_state(np.ascontiguousarray(x.astype(np.float32)))
    st["v"] = np.random.default_rng(seed).normal(0, 0.05, st["v"].shape).astype(np.float32)
    return st


def _cloud(dim, counts, seed):
    """counts[i] particles in cell i of a row of cells (3 blocks of cells apart
    in y), shuffled."""
    rng = np.random.default_rng(seed)
    pts = []
    for i, k in enumerate(counts):
        base = np.array([4 + i % 8, 4 + 3 * (i // 8), 5][:dim], np.float64)
        pts.append(base + 0.5 + rng.uniform(0.02, 0.98, (k, dim)))
    p = np.concatenate(pts)
    return (p[rng.permutation(len(p))].T * 0.25).astype(np.float32)


CLOUDS = {
    "few": [1, 0, 2, 3, 1, 5],
    "cell_64": [64, 63, 65, 1],
    "cell_200": [200, 1, 300, 64, 65],
    "block_1024": [256, 256, 256, 256, 7],
    "block_1025": [256, 257, 256, 256, 7],
    "block_5000": [5000, 3, 700, 90, 1, 1025],
    "wg_255": [255],
    "wg_257": [100, 157],
}


@pytest.mark.parametrize("flags", ["full", "scan", "dense", "adjoint"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("name", list(CLOUDS))
def test_order_is_the_stable_sort(name, dim, flags):
    import torch
    from paper_2605_28525_amd import mpm as M
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    x = _cloud(dim, CLOUDS[name], seed=len(name))
    w.dim, w.dx, w.cells = dim, 0.25, (20, 40, 16)[:dim]
    for k, a in _state(x, 3).items():
        setattr(w, k, a)
    _announce("table sort", name, dim, flags, w.n)
    fl = {"full": M.MPM_FLAG_FULL_SORT, "scan": M.MPM_FLAG_SCAN_BUILD, "dense": 0, "adjoint": M.MPM_FLAG_ADJOINT}[flags]
    sim = M.Simulation(w, flags=fl, grid_mode=M.MPM_GRID_DENSE if flags == "dense" else M.MPM_GRID_SPARSE)
    try:
        for step in range(2):  # the second from the first one's output order
            xin = sim.a.to_arrays()["x"]
            a, b = sim.a.view(), sim.b.view()
            M.mpm_sparse_build(sim.ctx, a)
            M.mpm_p2g(sim.ctx, a)
            M.mpm_grid_update(sim.ctx)
            M.mpm_g2p(sim.ctx, a, b)
            order = torch.empty(w.n, dtype=torch.int32, device="cuda")
            M.mpm_get_order(sim.ctx, order, w.n)
            rc, f = sim.status()
            assert rc == 0, f
            exp = expected_order(xin, w.dx, w.cells, dim)
            assert np.array_equal(order.cpu().numpy(), exp), step
            sim.a, sim.b = sim.b, sim.a
    finally:
        sim.close()


@pytest.mark.parametrize("cells", [(51, 51, 15), (52, 51, 16), (260, 260, 4)])
def test_order_around_table_tiles(cells):
    """Domains of 676, 910 and 8712 blocks (the table's tiles hold 2048), 3000
    particles everywhere in them in random order."""
    import torch
    from paper_2605_28525_amd import mpm as M
    w = wl.tiny_3d(n=48, ties=False)
    w.cells = cells
    rng = np.random.default_rng(9)
    x = rng.uniform(1.1, np.asarray(cells, np.float64)[:, None] - 1.6, (3, 3000)) * w.dx
    for k, a in _state(x, 4).items():
        setattr(w, k, a)
    _announce("table sort, domain", cells)
    sim = M.Simulation(w, flags=M.MPM_FLAG_FULL_SORT)
    try:
        M.mpm_sparse_build(sim.ctx, sim.a.view())
        M.mpm_p2g(sim.ctx, sim.a.view())
        order = torch.empty(w.n, dtype=torch.int32, device="cuda")
        M.mpm_get_order(sim.ctx, order, w.n)
        rc, f = sim.status()
        assert rc == 0, f
        assert np.array_equal(order.cpu().numpy(), expected_order(w.x, w.dx, cells, 3))
    finally:
        sim.close()


@pytest.mark.parametrize("grid", ["sparse", "dense"])
@pytest.mark.parametrize("cells", [(31, 31, 31), (32, 31, 31), (2047, 2047), (2048, 2047)])
def test_order_around_the_scan_s_sizes(cells, grid):
    """Domains of 512 and 576 blocks (one tile of the short scan, and two) and
    of 2^18 and 262,656 (the last with short tiles, and past it); particles in
    random order everywhere, in the first and in the last block."""
    import torch
    from paper_2605_28525_amd import mpm as M
    dim = len(cells)
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    w.dim, w.dx, w.cells = dim, 0.25, cells
    rng = np.random.default_rng(12)
    top = np.asarray(cells, np.float64)[:, None] - 0.6
    x = np.concatenate([rng.uniform(0.6, top, (dim, 3000)), rng.uniform(0.6, 2.0, (dim, 70)),
                        rng.uniform(top - 1.0, top, (dim, 70))], axis=1)
    x = x[:, rng.permutation(x.shape[1])] * w.dx
    for k, a in _state(x, 4).items():
        setattr(w, k, a)
    _announce("table sort, scan size", cells, grid)
    sim = M.Simulation(w, flags=M.MPM_FLAG_FULL_SORT, block_capacity=1 << 14,  # up to 4 blocks a particle
                       grid_mode=M.MPM_GRID_DENSE if grid == "dense" else M.MPM_GRID_SPARSE)
    try:
        M.mpm_sparse_build(sim.ctx, sim.a.view())
        M.mpm_p2g(sim.ctx, sim.a.view())
        order = torch.empty(w.n, dtype=torch.int32, device="cuda")
        M.mpm_get_order(sim.ctx, order, w.n)
        rc, f = sim.status()
        assert rc == 0, f
        assert np.array_equal(order.cpu().numpy(), expected_order(w.x, w.dx, cells, dim))
    finally:
        sim.close()


def test_order_of_an_ensemble():
    """Instances first, then blocks: the particles shuffled across instances."""
    import torch
    from paper_2605_28525_amd import mpm as M
    ens = wl.ensemble_small(n_instances=3)
    perm = np.random.default_rng(5).permutation(ens.n)
    for k in ("x", "v", "C", "F", "tau"):
        setattr(ens, k, np.ascontiguousarray(getattr(ens, k)[:, perm]))
    ens.inst = np.ascontiguousarray(ens.inst[perm])
    m = ens.members[0]
    _announce("table sort, ensemble", ens.n)
    sim = M.Simulation(ens, flags=M.MPM_FLAG_FULL_SORT)
    try:
        M.mpm_sparse_build(sim.ctx, sim.a.view())
        M.mpm_p2g(sim.ctx, sim.a.view())
        order = torch.empty(ens.n, dtype=torch.int32, device="cuda")
        M.mpm_get_order(sim.ctx, order, ens.n)
        rc, f = sim.status()
        assert rc == 0, f
        assert np.array_equal(order.cpu().numpy(), expected_order(ens.x, m.dx, m.cells, 3, ens.inst))
    finally:
        sim.close()


def _far_cloud(dim, n, seed):
    """n particles around the middle of a 40-cell box, some blocks full, some with one."""
    rng = np.random.default_rng(seed)
    c = np.concatenate([rng.normal(16, 2.5, (dim, n - n // 8)), rng.uniform(7, 30, (dim, n // 8))], axis=1)
    return (np.clip(c, 6.1, 33.9)[:, rng.permutation(n)] * 0.25).astype(np.float32)


@pytest.mark.parametrize("flags", ["full", "scan", "dense", "adjoint"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [1, 700, 6000])
def test_steps_equal_those_of_a_larger_domain(n, dim, flags):
    """The same particles in a domain within the table and in one of more than
    4.2 million blocks, which keeps the radix sort and the builds from sorted
    keys: the same active blocks in the same order, particles bit for bit (on a
    dense grid, whose P2G adds with atomics, to the parity tolerance)."""
    from paper_2605_28525_amd import mpm as M
    from parity_util import RTOL, assert_field, tau_floor
    fl = {"full": M.MPM_FLAG_FULL_SORT, "scan": M.MPM_FLAG_SCAN_BUILD, "dense": 0, "adjoint": M.MPM_FLAG_ADJOINT}[flags]
    _announce("table against radix", n, dim, flags)
    x = _far_cloud(dim, n, 11)
    got = []
    for cells in [(40, 48, 44)[:dim], (660, 656, 652)[:dim] if dim == 3 else (8300, 8260)]:
        w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
        w.dim, w.dx, w.cells, w.dt = dim, 0.25, cells, 1e-3
        for k, a in _state(x, 6).items():
            setattr(w, k, a)
        sim = M.Simulation(w, flags=fl, block_capacity=4096,
                           grid_mode=M.MPM_GRID_DENSE if flags == "dense" else M.MPM_GRID_SPARSE)
        try:
            sim.step(3)
            rc, f = sim.status()
            assert rc == 0, f
            act = None
            if flags != "dense":
                import torch
                M.mpm_sparse_build(sim.ctx, sim.a.view())
                nb, _ = M.mpm_active_count(sim.ctx)
                kh = torch.empty(nb, dtype=torch.int64, device="cuda")
                mh = torch.empty_like(kh)
                M.mpm_get_active(sim.ctx, kh, mh, nb)
                act = np.stack([kh.cpu().numpy(), mh.cpu().numpy()])
                if flags != "scan":  # (slot order)
                    act = act[:, np.argsort(act[0])]
            got.append((sim.a.to_arrays(), sim.a.ids(), act))
        finally:
            sim.close()
    (sa, ia, aa), (sb, ib, ab) = got
    assert np.array_equal(ia, ib)
    if aa is not None:
        assert np.array_equal(aa, ab)
    for k in sa:
        if flags == "dense":
            assert_field(k, sa[k], sb[k], RTOL, atol=tau_floor(w) if k == "tau" else 0.0)
        else:
            assert np.array_equal(sa[k], sb[k]), k


def test_scan_build_past_its_capacity():
    """More active blocks than the capacity: the overflow is raised, the count
    is the whole one, and the context works again with fewer particles."""
    from paper_2605_28525_amd import mpm as M
    x = _far_cloud(3, 3000, 5)
    w = wl.tiny_3d(n=48, ties=False)
    w.dx, w.cells, w.dt = 0.25, (40, 48, 44), 1e-3
    for k, a in _state(x, 6).items():
        setattr(w, k, a)
    _announce("scan build past its capacity")
    big = M.Simulation(w, flags=M.MPM_FLAG_SCAN_BUILD, block_capacity=4096)
    small = M.Simulation(w, flags=M.MPM_FLAG_SCAN_BUILD, block_capacity=40)
    try:
        M.mpm_sparse_build(big.ctx, big.a.view())
        nb, touched = M.mpm_active_count(big.ctx)
        assert nb == touched > 40
        M.mpm_sparse_build(small.ctx, small.a.view())
        assert M.mpm_active_count(small.ctx) == (40, touched)
        assert small.status()[0] != 0
        M.mpm_clear_status(small.ctx)
        few = M.ParticleSet(3, 4)
        few.x[:] = small.a.x[:, :1]
        M.mpm_sparse_build(small.ctx, few.view())
        nb, touched = M.mpm_active_count(small.ctx)
        assert 0 < nb == touched <= 8 and small.status()[0] == 0
    finally:
        big.close()
        small.close()
