"""GPU: a differentiable rollout whose forward pass recorded its last segment on
the tape, against the same rollout with every segment recomputed: the
gradients are equal bit for bit (the same kernels on the same inputs), also
where something else used the tape in between and the recording is gone."""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_adjoint import _announce, _rollout_inputs

pytestmark = pytest.mark.gpu


def _gradients(roll, w, v0, tgt, between=None, recompute=False):
    import torch
    from paper_2605_28525_amd import autograd as AG
    E, phi = (torch.tensor(q, dtype=torch.float64, requires_grad=True) for q in (2.0e5, 30.0))
    v = torch.from_numpy(v0).cuda().requires_grad_(True)
    x = AG._RolloutFn.apply(E, phi, v, roll) if recompute else AG.rollout(E, phi, v, roll)
    loss = 0.5 * torch.sum((x.double() - tgt) ** 2) / w.n
    if between:
        between()
    out = []
    for _ in range(2):  # the second backward pass of one forward pass
        out += [g.cpu().numpy() for g in torch.autograd.grad(loss, (E, phi, v), retain_graph=True)]
    return [x.detach().cpu().numpy()] + out


@pytest.mark.parametrize("steps,K", [(1, 1), (7, 10), (10, 5), (11, 4)])
@pytest.mark.parametrize("between", ["nothing", "tape", "forward", "tuning"])
def test_recorded_equals_recomputed(steps, K, between):
    import torch
    from paper_2605_28525_amd import autograd as AG
    from paper_2605_28525_amd import mpm as M
    w = wl.differentiable_fd_copy()
    w.E, w.dt = 2.0e5, 2.0e-4
    v0, target = _rollout_inputs(w, w.n)
    tgt = torch.from_numpy(target.astype(np.float64)).cuda()
    _announce("rollout recorded", steps, K, between)
    roll = AG.Rollout(w, steps=steps, checkpoint=K)
    try:
        ref = _gradients(roll, w, v0, tgt, recompute=True)

        def other():
            if between == "tape":
                sets = [M.ParticleSet(w.dim, w.n) for _ in range(2)]
                sets[0].copy_(roll.init)
                M.mpm_tape_forward(roll.ctx, [s.view() for s in sets])
            elif between == "forward":
                roll.run_forward(torch.from_numpy(v0).cuda() * 0.5, 3.0e5, 25.0)
            elif between == "tuning":
                M.mpm_set_tuning(roll.ctx, 128, 0, 0, 0)

        got = _gradients(roll, w, v0, tgt, other)
        rc, flags = M.mpm_get_status(roll.ctx)
        assert rc == 0, flags
    finally:
        roll.close()
    for k, (a, b) in enumerate(zip(ref, got)):
        if between == "tuning" and k in (1, 2, 4, 5):
            # other work items: the parameter sums are grouped another way
            assert abs(a - b) <= 1e-5 * abs(a), k
        else:
            assert np.array_equal(a, b), k
