"""GPU: the incremental re-sort where its particle counts are summed over several
groups of previous blocks (256 blocks each), at the edges of a group and past
it, with blocks of one particle and blocks split over several work items, and
after displacements that leave most blocks for new ones.

The oracle is the full radix sort on the same states (as in test_gpu_resort):
active blocks and node masks equal, particle layout as specified, grids and
particles at the parity bar.
"""
import numpy as np
import pytest

from paper_2605_28525_amd import workloads as wl
from test_gpu_resort import _announce, _run_pair, _run_pair_continue

pytestmark = pytest.mark.gpu


def _clusters(k, sizes, seed):
    """k separate clusters, one inside each of k owner blocks two blocks apart
    (8 active blocks each), with sizes[i % len(sizes)] particles."""
    w = wl.tiny_3d(n=48, ties=False)
    rng = np.random.default_rng(seed)
    per = 16
    w.cells = (per * 8 + 16, per * 8 + 16, 8 * (k // (per * per) + 1) + 16)
    pts = []
    for i in range(k):
        lo = 8 * np.array([i % per, (i // per) % per, i // (per * per)]) + 4
        pts.append(lo + rng.uniform(0.6, 3.4, size=(sizes[i % len(sizes)], 3)))
    x = (np.concatenate(pts).T * w.dx).astype(np.float32)
    for key, a in wl.rest_state(np.ascontiguousarray(x)).items():
        setattr(w, key, a)
    return wl.perturbed(w, seed=seed + 1, v_scale=0.5, C_scale=0.2)


# 8 active blocks per cluster: 31, 32 and 33 clusters end below, at and past
# the first group of 256; 130 clusters fill four groups and start a fifth
@pytest.mark.parametrize("k", [31, 32, 33, 130])
@pytest.mark.parametrize("sizes", [(1, 3, 2), (1, 700, 40)])
def test_counts_over_groups_of_blocks(k, sizes):
    w = _clusters(k, sizes, seed=61 + k)
    _announce("resort groups", k, sizes, w.n)
    inc, full = _run_pair(w, 3, "groups")
    try:
        # every particle moved by up to 6 cells: most blocks empty, most
        # particles in blocks without a previous slot
        rng = np.random.default_rng(7 * k)
        st = inc.a.to_arrays()
        ids = inc.a.ids()
        lo, hi = 3.0 * w.dx, np.asarray(w.cells, np.float64)[:, None] * w.dx - 3.0 * w.dx
        shift = rng.uniform(-6.0, 6.0, size=st["x"].shape) * w.dx
        st["x"] = np.clip(st["x"].astype(np.float64) + shift, lo, hi).astype(np.float32)
        inc.set_state(st, ids=ids)
        full.set_state(st, ids=ids)
        _run_pair_continue(w, inc, full, 3, "groups displaced")
    finally:
        inc.close()
        full.close()
