"""GPU: two contexts on two streams that accumulate their parameter gradients
into one param_bar, as a program that sums a loss over simulations does: no
context's share is lost.  (The sums differ from the separate ones by float32
additions in another order: 2^-24 of the running total for each addition.)
"""
import numpy as np
import pytest

from test_gpu_tape import FIELDS, _announce, _workload

pytestmark = pytest.mark.gpu

REPS = 100


def test_contexts_share_an_accumulator():
    import torch
    from paper_2605_28525_amd import mpm as M
    w, st = _workload("fd_copy_3d")
    d, n = w.dim, w.n
    _announce("shared param_bar", n, REPS)
    rng = np.random.default_rng(5)
    ctxs, sets, streams = [], [], [torch.cuda.Stream() for _ in range(2)]
    try:
        for _ in range(2):
            ctxs.append(M.mpm_create(M.params_from_workload(w, flags=M.MPM_FLAG_ADJOINT)))
            a, ob, ib = M.ParticleSet.from_arrays(st), M.ParticleSet(d, n), M.ParticleSet(d, n)
            for f, sc in (("x", 1.0), ("v", 1.0), ("C", 1e-2), ("F", 1.0), ("tau", 1e-5)):
                t = getattr(ob, f)
                t.copy_(torch.from_numpy((rng.normal(size=tuple(t.shape)) * sc).astype(np.float32)))
            sets.append((a, ob, ib))
        one = []
        for ctx, (a, ob, ib) in zip(ctxs, sets):
            pb = torch.zeros(2, dtype=torch.float32, device="cuda")
            M.mpm_step_adj(ctx, a.view(), ob.view(), ib.view(), pb)
            one.append(pb.cpu().numpy().astype(np.float64))
        shared = torch.zeros(2, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        for _ in range(REPS):
            for ctx, (a, ob, ib), s in zip(ctxs, sets, streams):
                M.mpm_step_adj(ctx, a.view(), ob.view(), ib.view(), shared, stream=s)
        torch.cuda.synchronize()
        got, want = shared.cpu().numpy().astype(np.float64), REPS * (one[0] + one[1])
        # each addition rounds a total of at most REPS (|a| + |b|)
        bound = 2 * REPS * 2.0 ** -24 * REPS * (np.abs(one[0]) + np.abs(one[1]))
        # and a context's own share repeats to the float32 sums inside it
        bound += 1e-5 * REPS * (np.abs(one[0]) + np.abs(one[1]))
        assert np.all(np.abs(got - want) <= bound), (got, want, bound)
        # (a lost share is far above it)
        assert np.all(bound < 0.5 * np.minimum(np.abs(one[0]), np.abs(one[1]))), (bound, one)
    finally:
        for c in ctxs:
            M.mpm_destroy(c)
