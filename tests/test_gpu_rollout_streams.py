"""GPU: one Rollout on two streams.  A forward pass keeps a buffer as its last
checkpoint that an earlier pass, on another stream, may have allocated; dropped
while the pass still runs, it must not be handed out on that other stream
before the pass has finished with it.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_adjoint import _announce, _rollout_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,K", [(4, 5), (7, 3)])
def test_dropped_pass_on_a_side_stream(steps, K):
    import torch
    from paper_2605_28525_amd import autograd as AG
    w = wl.differentiable_fd_copy()
    w.E, w.dt = 2.0e5, 2.0e-4
    v0, _ = _rollout_inputs(w, w.n)
    E, phi = (torch.tensor(q, dtype=torch.float64, requires_grad=True) for q in (2.0e5, 30.0))
    v = torch.from_numpy(v0).cuda().requires_grad_(True)
    _announce("rollout on two streams", steps, K)
    roll = AG.Rollout(w, steps=steps, checkpoint=K)
    side = torch.cuda.Stream()
    try:
        for _ in range(2):
            ref = AG.rollout(E, phi, v, roll).detach().clone()   # buffers of the current stream
        for _ in range(3):
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                torch.cuda._sleep(20_000_000)
                x = AG.rollout(E, phi, v, roll).detach()   # the pass is dropped here, before it has run
            # what the current stream allocates meanwhile must not be its buffers
            junk = [torch.full_like(getattr(roll.init, k), float("nan")) for k in ("x", "v", "C", "F", "tau")
                    for _ in range(8)]
            torch.cuda.synchronize()
            assert np.array_equal(x.cpu().numpy(), ref.cpu().numpy())
            del junk
    finally:
        torch.cuda.synchronize()
        roll.close()
