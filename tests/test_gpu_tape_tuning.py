"""GPU: the work item size changed between mpm_tape_forward and
mpm_tape_adjoint.  The reverse sweep walks the items as they were recorded, so
the adjoints are those of a context left alone, bit for bit (the same kernels
over the same items).  Blocks of more than 512 particles: items of 128, 256
and 512 are all several parts of the reverse kernels' workgroups.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl

pytestmark = pytest.mark.gpu

FIELDS = ("x", "v", "C", "F", "tau")
STEPS = 3


def _cloud(dim):
    """700 particles in one block of cells and 300 in the next."""
    rng = np.random.default_rng(4)
    lo = np.array([4, 4, 4][:dim], np.float64)
    x = np.concatenate([lo + rng.uniform(0.7, 3.8, (700, dim)), lo + rng.uniform(4.7, 7.8, (300, dim))])
    w = wl.tiny_3d(n=48, ties=False) if dim == 3 else wl.collapse_2d()
    w.dim, w.dx, w.cells, w.dt, w.E = dim, 0.25, (16, 16, 16)[:dim], 1e-4, 5e4
    st = wl.rest_state((x.T * 0.25).astype(np.float32))
    st["v"] = rng.normal(0, 0.05, st["v"].shape).astype(np.float32)
    for k, a in st.items():
        setattr(w, k, a)
    return w


def _sweep(w, recorded, change):
    import torch
    from paper_2605_28525_amd import mpm as M
    ctx = M.mpm_create(M.params_from_workload(w, flags=M.MPM_FLAG_ADJOINT))
    try:
        M.mpm_set_tuning(ctx, chunk=recorded)
        M.mpm_tape_reserve(ctx, STEPS)
        sets = [M.ParticleSet(w.dim, w.n) for _ in range(STEPS + 1)]
        sets[0].copy_(M.ParticleSet.from_arrays(w.state()))
        views = [s.view() for s in sets]
        M.mpm_tape_forward(ctx, views)
        serial = M.mpm_tape_serial(ctx)
        if change == "autotune":
            b = M.ParticleSet(w.dim, w.n)
            M.mpm_autotune(ctx, sets[0].view(), b.view())
        elif change:
            M.mpm_set_tuning(ctx, chunk=change)
        assert M.mpm_tape_serial(ctx) == serial   # the slots are what they were
        rng = np.random.default_rng(11)
        bar, spare = M.ParticleSet(w.dim, w.n), M.ParticleSet(w.dim, w.n)
        for f, sc in (("x", 1.0), ("v", 1.0), ("C", 1e-2), ("F", 1.0), ("tau", 1e-5)):
            t = getattr(bar, f)
            t.copy_(torch.from_numpy((rng.normal(size=tuple(t.shape)) * sc).astype(np.float32)))
            getattr(spare, f).fill_(1e3)   # what a position left out would be taken from
        pb = torch.zeros(2, dtype=torch.float32, device="cuda")
        M.mpm_tape_adjoint(ctx, views, bar.view(), spare.view(), pb)
        rc, flags = M.mpm_get_status(ctx)
        assert rc == 0, flags
        return dict(bar.to_arrays(), params=pb.cpu().numpy())
    finally:
        M.mpm_destroy(ctx)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("recorded,change", [(512, 128), (512, 64), (256, 64), (128, 768), (512, "autotune")])
def test_adjoint_walks_the_recorded_items(dim, recorded, change):
    w = _cloud(dim)
    print("CASE tape tuning", dim, recorded, change, flush=True)
    ref, got = _sweep(w, recorded, None), _sweep(w, recorded, change)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


@pytest.mark.parametrize("dim", [2, 3])
def test_adjoint_over_radix_sorted_steps(dim):
    """The same particles in a domain of more than 4.2 million blocks, whose steps
    keep the radix sort: the same recording in the same order, so the same bits."""
    ref = _sweep(_cloud(dim), 512, None)
    w = _cloud(dim)
    w.cells = (660, 656, 652) if dim == 3 else (8300, 8260)
    print("CASE tape, radix sort", dim, flush=True)
    got = _sweep(w, 512, None)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k
