"""GPU tests of the ray-exact kernels where four waves share a tile's list:
lists shorter than a batch of 64, lists that leave some of the waves (or of the
chunks that calls with few tiles add) empty, lists of several rounds, ragged
detectors, and calls with many tiles, which have no chunks."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
BAND = 1e-5   # pairs this near the cutoff have no unique answer


@pytest.fixture(scope="module")
def fgs():
    import paper_2604_01844_amd as m
    return m


@pytest.mark.parametrize("n,sigma,det_w,det_h,views", [
    (1, 0.03, 16, 16, 1),       # one tile, one Gaussian
    (65, 0.2, 16, 16, 1),       # one tile, a second batch of one
    (6000, 0.1, 16, 16, 1),     # more than one round of 16 chunks of 4 batches
    (700, 0.1, 75, 41, 3),      # ragged
    (300, 0.1, 256, 256, 33),   # 8,448 tiles: no chunks, lists of zero to five batches
])
def test_shared_lists(fgs, n, sigma, det_w, det_h, views):
    gs = si.gaussians(n, 51, log_scale_mean=float(np.log(sigma)))
    gd = si.geometry(det_w, det_h)
    ang = si.angles(views)
    geom = fgs.Geometry.from_dict(gd, ang, DEV)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in ("mean", "log_scale", "quat", "density")]
    ws = fgs.Workspace(DEV)
    img = fgs.project_views(*args, geom, model="exact", ws=ws).cpu().numpy()
    assert oracle.rel_l2(img, oracle.exact_project(gs, gd, ang)) < TOL
    c = si.normals((views, det_h, det_w), 52)
    got = fgs.project_views_backward(*args, geom, torch.from_numpy(c).to(DEV), recompute=False, ws=ws, model="exact")
    ref = oracle.exact_bwd(gs, gd, ang, c.astype(np.float64), band=BAND)
    names = ("mean", "log_scale", "quat", "density")
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(names, got)}, ref)
    assert max(errs.values()) < TOL, errs
