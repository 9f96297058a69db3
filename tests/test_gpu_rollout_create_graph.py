"""GPU: gradients of a rollout asked for with create_graph, as a program that logs
or penalises them does (they are constants to a second derivative): the same
bits as without it, over one segment and over several, recorded or recomputed,
and the rollout's buffers keep no graph.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_adjoint import _announce, _rollout_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,K", [(3, 5), (6, 3), (7, 3)])
@pytest.mark.parametrize("recorded", [True, False])
def test_create_graph_changes_nothing(steps, K, recorded):
    import torch
    from paper_2605_28525_amd import autograd as AG
    w = wl.differentiable_fd_copy()
    w.E, w.dt = 2.0e5, 2.0e-4
    v0, target = _rollout_inputs(w, w.n)
    tgt = torch.from_numpy(target.astype(np.float64)).cuda()
    _announce("rollout create_graph", steps, K, recorded)
    roll = AG.Rollout(w, steps=steps, checkpoint=K)
    try:
        out = []
        for create in (False, True, False):
            E, phi = (torch.tensor(q, dtype=torch.float64, requires_grad=True) for q in (2.0e5, 30.0))
            v = torch.from_numpy(v0).cuda().requires_grad_(True)
            x = AG.rollout(E, phi, v, roll) if recorded else AG._RolloutFn.apply(E, phi, v, roll)
            loss = 0.5 * torch.sum((x.double() - tgt) ** 2) / w.n
            out.append([g.detach().cpu().numpy() for g in torch.autograd.grad(loss, (E, phi, v), create_graph=create)])
            assert not any(getattr(s, k).requires_grad for s in roll._bars for k in ("x", "v", "C", "F", "tau"))
    finally:
        roll.close()
    for got in out[1:]:
        for a, b in zip(out[0], got):
            assert np.array_equal(a, b)
