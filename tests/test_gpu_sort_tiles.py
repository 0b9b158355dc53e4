"""GPU test of the radix sort's order of tiles (4,096 pairs each, dealt to the
XCDs in contiguous eighths): fewer tiles than XCDs, a few more, many, and a
grid sized for a capacity that the pairs do not fill."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("capacity", [0, 1, 5])
@pytest.mark.parametrize("n", [3, 200, 700, 1100, 20000])
def test_lists_are_stably_sorted(n, capacity):
    import paper_2604_01844_amd as fgs
    from paper_2604_01844_amd.ops import binning_dump
    gs = si.gaussians(n, 81)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in ("mean", "log_scale", "quat", "density")]
    grid = fgs.Grid.from_dict(si.grid(104))  # 2,197 tiles of some 50 each per Gaussian
    ws = fgs.Workspace(DEV)
    fgs.voxelize(*args, grid, ws=ws)
    k = ws.n_pairs
    if capacity:
        ws = fgs.Workspace(DEV)
        ws.set_capacity(capacity * k)
        fgs.voxelize(*args, grid, ws=ws)
    d = binning_dump(ws)
    keys, vals = (d[a].cpu().numpy()[:k].astype(np.int64) for a in ("sorted_keys", "sorted_vals"))
    start = d["tile_start"].cpu().numpy()
    assert (np.diff(keys) >= 0).all() and (np.diff(vals)[np.diff(keys) == 0] > 0).all()
    np.testing.assert_array_equal(np.sort(vals), np.arange(k))
    np.testing.assert_array_equal(np.bincount(keys, minlength=start.size - 1), np.diff(start))
