"""GPU: the autotuner runs the kernels that mpm_step runs.  Small steps leave
P2G's second pass to a form of G2P that only some launch shapes have; the
trials of those shapes must run that form (and no second pass), the trials of
the others the second pass with the grid update in it.  Kernels by name, from the
profiler's record of the call.
"""
import re

import pytest

from paper_2605_28525_amd import workloads as wl

pytestmark = pytest.mark.gpu

# trials: 4 workgroup counts x (a warm-up and 5 timed steps) per launch shape
TRIALS = 24


def _kernels(w, grid_mode=0):
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2605_28525_amd import mpm as M
    sim = M.Simulation(w, grid_mode=grid_mode)
    try:
        sim.step(1)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            M.mpm_autotune(sim.ctx, sim.a.view(), sim.b.view())
            torch.cuda.synchronize()
        assert sim.status()[0] == 0
    finally:
        sim.close()
    count = {}
    for e in p.events():
        name = re.sub(r"^void mpmx::|\(.*$", "", e.name)
        count[name] = count.get(name, 0) + 1
    if not any(k.startswith("k_g2p<") for k in count):
        pytest.skip("the profiler recorded no kernels")
    return count


@pytest.mark.parametrize("case", ["2d", "3d", "3d large", "2d dense"])
def test_trials_run_the_steps_kernels(case):
    from paper_2605_28525_amd import mpm as M
    print("CASE autotune", case, flush=True)
    w = {"2d": wl.collapse_2d, "3d": wl.differentiable_fd_copy, "3d large": lambda: wl.collapse_3d(seed=2, scale=2),
         "2d dense": wl.collapse_2d}[case]()
    dense = case == "2d dense"
    k = _kernels(w, M.MPM_GRID_DENSE if dense else M.MPM_GRID_SPARSE)
    d = w.dim
    gathers = not dense and w.n <= 65536
    form = "true" if gathers else "false"
    got = {n: c for n, c in k.items() if n.startswith(("k_g2p", "k_p2g_gather", "k_grid_update"))}
    want = {f"k_g2p<{d}, 64, 2, false>": 2 * TRIALS, f"k_g2p<{d}, 128, 2, false>": 2 * TRIALS,
            f"k_g2p<{d}, 256, 1, {form}>": TRIALS, f"k_g2p<{d}, 256, 2, {form}>": TRIALS,
            f"k_g2p<{d}, 256, 3, false>": TRIALS}
    if dense:
        want[f"k_grid_update<{d}>"] = 7 * TRIALS
    else:
        want[f"k_p2g_gather<{d}, true>"] = (5 if gathers else 7) * TRIALS
    assert got == want
