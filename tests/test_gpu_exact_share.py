"""GPU tests of the ray-exact kernels on both sides of the line from which four
waves share a tile's list (8,192 tiles or more), ragged detectors among them,
and at a fixed key capacity, where the line is drawn on the device."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
BAND = 1e-5   # pairs this near the cutoff have no unique answer
NAMES = ("mean", "log_scale", "quat", "density")


@pytest.mark.parametrize("n,sigma,det_w,det_h,views,shared", [
    (60, 0.02, 256, 256, 33, False),   # a few keys per tile
    (150, 0.03, 250, 250, 33, False),  # ragged
    (400, 0.1, 250, 130, 60, True),    # ragged, lists of several batches
])
def test_share_line(n, sigma, det_w, det_h, views, shared):
    import paper_2604_01844_amd as fgs
    gs = si.gaussians(n, 53, log_scale_mean=float(np.log(sigma)))
    gd = si.geometry(det_w, det_h)
    ang = si.angles(views)
    geom = fgs.Geometry.from_dict(gd, ang, DEV)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in NAMES]
    ws = fgs.Workspace(DEV)
    img = fgs.project_views(*args, geom, model="exact", ws=ws)
    tiles = ws.s.n_tiles
    assert tiles >= 8192 and (ws.n_pairs >= tiles * min(tiles, 65536) // 512) == shared
    assert oracle.rel_l2(img.cpu().numpy(), oracle.exact_project(gs, gd, ang)) < TOL
    c = si.normals((views, det_h, det_w), 54)
    cd = torch.from_numpy(c).to(DEV)
    got = fgs.project_views_backward(*args, geom, cd, recompute=False, ws=ws, model="exact")
    ref = oracle.exact_bwd(gs, gd, ang, c.astype(np.float64), band=BAND)
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(NAMES, got)}, ref)
    assert max(errs.values()) < TOL, errs
    support = fgs.project_views_support(*args, geom, model="exact")
    # the same pairs at a fixed capacity give the same bits, whatever the capacity
    for cap in (ws.n_pairs, 4 * max(ws.n_pairs, tiles * tiles // 512)):
        wf = fgs.Workspace(DEV)
        wf.set_capacity(cap)
        assert torch.equal(img, fgs.project_views(*args, geom, model="exact", ws=wf))
        again = fgs.project_views_backward(*args, geom, cd, recompute=False, ws=wf, model="exact")
        assert all(torch.equal(a, b) for a, b in zip(got, again))
        assert fgs.project_views_support(*args, geom, model="exact", ws=wf) == support
