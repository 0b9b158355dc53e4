"""GPU test of the voxelizer's binning on both sides of the line (16,384) from
which a wave takes four Gaussians: a Gaussian's tiles do not depend on it."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAMES = ("mean", "log_scale", "quat", "density")


@pytest.mark.parametrize("n,voxels,sd", [
    (16384, 2.0, 0.3),    # rectangles of up to 64 tiles
    (16387, 8.0, 0.6),    # both kinds, the last wave with three Gaussians
    (20001, 20.0, 0.3),   # all large, some of more than 512 tiles
])
def test_tiles_do_not_depend_on_the_split(n, voxels, sd):
    import paper_2604_01844_amd as fgs
    gs = si.gaussians(n, 97, log_scale_mean=float(np.log(voxels / 128)), log_scale_sd=sd)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in NAMES]
    grid = fgs.Grid((-0.5,) * 3, (1.0 / 128,) * 3, (127, 128, 125))

    def binning(p):
        ws = fgs.Workspace(DEV)
        fgs.voxelize(*p, grid, ws=ws)
        d = fgs.binning_dump(ws)
        tile = torch.repeat_interleave(torch.arange(ws.s.n_tiles, device=DEV), d["tile_start"].diff())
        own = torch.empty(ws.n_pairs, dtype=torch.int64, device=DEV)
        own[d["sorted_vals"].long()] = tile  # every slot's tile: Gaussian by Gaussian, row-major in each
        return d["offset"].diff().clone(), own

    half = 9000
    count, own = binning(args)
    parts = [binning([t[..., a:b].contiguous() for t in args]) for a, b in ((0, half), (half, n))]
    assert half < 16384 and n - half < 16384 <= n
    assert torch.equal(count, torch.cat([c for c, _ in parts]))
    assert torch.equal(own, torch.cat([o for _, o in parts]))
