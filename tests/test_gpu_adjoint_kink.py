"""GPU: reverse mode of particles within rounding of a kink of the return map
(elastic just inside the cone's tip, plastic just past it), which settle their
branch by another evaluation than the rest, against the FP64 oracle: strains
of one or two units in the last place of 1, where the branch is certain but
near, mixed with ordinary strains.  Bar as in test_gpu_adjoint.
"""
import numpy as np
import pytest

from oracle import mpm as om
from paper_2605_28525_amd import workloads as wl
from test_gpu_adjoint import _announce, _check_step_adjoint, _consistent_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("share", [1, 3, 64])
@pytest.mark.parametrize("dim", [2, 3])
def test_step_adjoint_at_the_kink(dim, share):
    """Every `share`-th particle is at the kink, inside and outside in turn.
    Uniform motion away from the walls and no stress: F_trial is F."""
    if dim == 3:
        w = wl.tiny_3d(n=48, ties=False)
        w.cells = (32, 32, 32)
    else:
        w = wl.collapse_2d()
        sel = (w.x[0] < 0.15) & (w.x[1] < 0.15)
        for k in ("x", "v", "C", "F", "tau"):
            setattr(w, k, getattr(w, k)[:, sel].copy())
    w.E = 5e4
    w.gravity = (0.0, 0.0, 0.0)
    w.x = w.x + np.float32(8 * w.dx if dim == 3 else 32 * w.dx)
    st = _consistent_state(w, 7)
    st["v"][:] = np.float32(0.01)
    st["C"][:] = 0.0
    st["tau"][:] = 0.0
    out = om.step(om.state_from_soa(dict(st, F=np.tile(np.eye(dim).reshape(-1, 1), w.n)), dim), om.Params.from_workload(w))
    assert np.abs(out["F"] - np.eye(dim)).max() < 1e-12  # no velocity gradient: strains below stay what they are
    at = np.arange(0, w.n, share)
    one = np.float32(1.0)
    for j, (lo, hi) in enumerate([(np.nextafter(one, np.float32(0)),) * 2, (np.nextafter(one, np.float32(2)), one)]):
        F = np.zeros((dim * dim, 1), np.float32)
        F[0] = lo
        F[[a * (dim + 1) for a in range(1, dim)]] = hi
        st["F"][:, at[j::2]] = F
    _announce("step adjoint at the kink", dim, share, w.n)
    print(_check_step_adjoint(w, st, 8))
