"""GPU tests of the splat kernels where four waves share a tile's list (8,192
tiles or more, lists long enough on average) and where they do not: both sides
of that line, lists shorter than a batch of 64 and longer than a round of four,
ragged detectors, the split of interior pairs, and a fixed key capacity, where
the line is drawn on the device."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
BAND = 1e-5   # pairs this near the cutoff d^2 = kappa^2 have no unique answer

CASES = [
    # n, sigma, det_w, det_h, views
    (60, 0.02, 256, 256, 33),     # a few keys per tile: a wave per tile
    (1500, 0.03, 256, 256, 33),   # shared, lists of none to some 500
    (700, 0.1, 250, 130, 60),     # ragged, shared, split
    (3000, 0.05, 128, 128, 130),  # shared, several rounds of four batches
]


@pytest.mark.parametrize("n,sigma,det_w,det_h,views", CASES)
def test_shared_lists(n, sigma, det_w, det_h, views):
    import paper_2604_01844_amd as fgs
    gs = si.gaussians(n, 61, log_scale_mean=float(np.log(sigma)))
    gd = si.geometry(det_w, det_h)
    ang = si.angles(views)
    geom = fgs.Geometry.from_dict(gd, ang, DEV)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in ("mean", "log_scale", "quat", "density")]
    ws = fgs.Workspace(DEV)
    img = fgs.project_views(*args, geom, ws=ws)
    assert oracle.rel_l2(img.cpu().numpy(), oracle.project(gs, gd, ang)) < TOL
    c = si.normals((views, det_h, det_w), 62)
    cd = torch.from_numpy(c).to(DEV)
    got = fgs.project_views_backward(*args, geom, cd, recompute=False, ws=ws)
    ref = oracle.project_bwd(gs, gd, ang, c.astype(np.float64), band=BAND)
    names = ("mean", "log_scale", "quat", "density")
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(names, got)}, ref)
    assert max(errs.values()) < TOL, errs
    # the same pairs at a fixed capacity give the same bits, whatever the capacity
    for margin in (1.0, 4.0):
        wf = fgs.Workspace(DEV)
        wf.set_capacity(int(margin * ws.n_pairs) + 64)
        assert torch.equal(img, fgs.project_views(*args, geom, ws=wf))
        for x, y in zip(got, fgs.project_views_backward(*args, geom, cd, recompute=False, ws=wf)):
            assert torch.equal(x, y)
