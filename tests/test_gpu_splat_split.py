"""GPU tests of the rasterizer's split of (quadrant, Gaussian) pairs into
interior and boundary ones, taken by calls that average 16 (forward) or 32
(backward) tiles or more per
Gaussian: both sides of that line, detector edges that cut tiles, single and
few views (work units) and many, thresholds of large kappa and of the
density-aware support, and a fixed key capacity."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
BAND = 1e-5   # pairs this near the cutoff d^2 = kappa^2 have no unique answer


@pytest.fixture(scope="module")
def fgs():
    import paper_2604_01844_amd as m
    return m


CASES = [
    # n, sigma, spread, det_w, det_h, views, mode, kappa, tau
    (300, 0.06, 0.3, 203, 150, 2, "cone", 3.0, 0.0),      # sigma 7-8 pixels, ragged edges, work units
    (300, 0.02, 0.3, 203, 150, 2, "cone", 3.0, 0.0),      # below the line: whole lists
    (40, 0.2, 0.3, 256, 256, 40, "cone", 3.0, 0.0),       # 10,240 tiles: a wave per tile; all but a rim interior
    (60, 0.08, 1.0, 250, 130, 3, "cone", 3.0, 0.0),       # elongated
    (100, 0.06, 0.3, 203, 150, 2, "parallel", 3.0, 0.0),
    (60, 0.15, 0.3, 203, 150, 2, "cone", 3.0, 0.0),       # 60 tiles each: split in the backward too
    (30, 0.03, 0.2, 256, 256, 1, "cone", 8.0, 0.0),       # threshold -46 in the exponent
    (20, 0.02, 0.2, 512, 512, 1, "cone", 10.0, 0.0),      # threshold -72: never interior
    (300, 0.08, 0.3, 203, 150, 2, "cone", 3.0, 2e-3),
    (200, 0.3, 0.1, 16, 16, 1, "cone", 3.0, 0.0),         # one tile
]


@pytest.mark.parametrize("n,sigma,sd,det_w,det_h,views,mode,kappa,tau", CASES)
def test_split_pairs(fgs, n, sigma, sd, det_w, det_h, views, mode, kappa, tau):
    gs = si.gaussians(n, 41, log_scale_mean=float(np.log(sigma)), log_scale_sd=sd)
    gd = si.geometry(det_w, det_h, mode=mode)
    ang = si.angles(views)
    geom = fgs.Geometry.from_dict(gd, ang, DEV)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in ("mean", "log_scale", "quat", "density")]
    ws = fgs.Workspace(DEV)
    img = fgs.project_views(*args, geom, kappa=kappa, tau=tau, ws=ws)
    ref = oracle.project(gs, gd, ang, kappa=kappa, tau=tau)
    assert oracle.rel_l2(img.cpu().numpy(), ref) < TOL
    c = si.normals((views, det_h, det_w), 42)
    cd = torch.from_numpy(c).to(DEV)
    got = fgs.project_views_backward(*args, geom, cd, kappa=kappa, tau=tau, recompute=False, ws=ws)
    bref = oracle.project_bwd(gs, gd, ang, c.astype(np.float64), kappa=kappa, tau=tau, band=BAND)
    names = ("mean", "log_scale", "quat", "density")
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(names, got)}, bref)
    assert max(errs.values()) < TOL, errs
    # the same pairs at a fixed capacity give the same bits, whatever the capacity
    for margin in (1.0, 4.0):
        wc = fgs.Workspace(DEV)
        wc.set_capacity(int(margin * ws.n_pairs) + 64)
        assert torch.equal(img, fgs.project_views(*args, geom, kappa=kappa, tau=tau, ws=wc))
        again = fgs.project_views_backward(*args, geom, cd, kappa=kappa, tau=tau, recompute=False, ws=wc)
        assert all(torch.equal(a, b) for a, b in zip(got, again))
        assert not wc.overflowed()[0]
