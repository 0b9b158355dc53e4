"""GPU tests of Gaussians hundreds of times longer than wide, whose quadratic
form's terms cancel: the culling of quarters and quadrants must not change the
decision that the per-voxel and per-pixel cutoff makes in FP32, so paths that
cull and paths that do not agree."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _needles(n, length, width, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    gs = si.gaussians(n, seed)
    ls = np.log(np.array([[length], [width], [width]])) + 0.2 * r.normal(size=(3, n))
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)
            for a in (gs["mean"], ls, gs["quat"], gs["density"])]


@pytest.mark.parametrize("length,width,kappa,n", [
    (2000, 0.2, 3.0, 1500),
    (5000, 0.5, 3.0, 1500),
    (2000, 0.2, 1.0, 1500),
    (40, 1.0, 3.0, 200),
])
def test_quarters_keep_every_decision(length, width, kappa, n):
    """The same Gaussians on a grid of 8,000 tiles, whose kernel tests every
    voxel of a tile, and on one of 8,400 with the same voxels and some more, whose
    kernel first skips quarters: where lists hold at most one batch, the same
    sums in the same order."""
    import paper_2604_01844_amd as fgs
    h = 1.0 / 160
    args = _needles(n, length * h, width * h, 17)
    ws = fgs.Workspace(DEV)
    small = fgs.voxelize(*args, fgs.Grid((-0.5,) * 3, (h,) * 3, (160, 160, 160)), kappa=kappa, ws=ws)
    lists = fgs.binning_dump(ws)["tile_start"].diff()
    assert ws.s.n_tiles == 8000 and 0 < int(lists.max()) <= 64
    large = fgs.voxelize(*args, fgs.Grid((-0.5,) * 3, (h,) * 3, (168, 160, 160)), kappa=kappa, ws=ws)
    assert ws.s.n_tiles == 8400 and ws.n_pairs < 64 * 8400
    assert (small > 0).sum() > 1000
    assert torch.equal(small, large[..., :160].contiguous())


@pytest.mark.parametrize("length,width,kappa", [(10.0, 0.0005, 3.0), (10.0, 0.0005, 1.0), (0.2, 0.002, 3.0)])
def test_quadrants_keep_every_decision(length, width, kappa):
    """A call that splits its pairs by quadrant (32 tiles per Gaussian) and one
    with the culling switched off. A pair at the cutoff adds w exp(-kappa^2 / 2),
    1e-2 w and more; the sums, of some tens of pairs per pixel, differ by their order and
    by interior pairs' products, 1e-6 of the largest. Of the gradients the density's is a
    plain sum over pixels (the others' moments cancel)."""
    import paper_2604_01844_amd as fgs
    args = _needles(150, length, width, 18)
    geom = fgs.Geometry.from_dict(si.geometry(512, 500), si.angles(3), DEV)
    c = torch.from_numpy(si.normals((3, 500, 512), 19)).to(DEV)
    ws = fgs.Workspace(DEV)
    img = fgs.project_views(*args, geom, kappa=kappa, ws=ws)
    assert ws.n_pairs >= 32 * 3 * 150
    ref = fgs.project_views(*args, geom, kappa=kappa, ablate=fgs.ops.ABLATE_QUADRANT_CULL)
    assert float((img - ref).abs().max()) < 1e-5 * float(ref.max())
    got = fgs.project_views_backward(*args, geom, c, kappa=kappa)
    ref = fgs.project_views_backward(*args, geom, c, kappa=kappa, ablate=fgs.ops.ABLATE_QUADRANT_CULL)
    assert float((got[3] - ref[3]).norm() / ref[3].norm()) < 1e-4
