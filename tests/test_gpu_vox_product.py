"""GPU tests of the voxelizer's product kernels (8,192 tiles or more, 96 tiles
per Gaussian and 64 pairs per tile on average) over what their tests of
interior quarters and pairs depend on: thresholds of a large kappa and of the
density-aware support, Gaussians past the grid."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
BAND = 1e-5   # pairs this near the cutoff d^2 = kappa^2 have no unique answer
NAMES = ("mean", "log_scale", "quat", "density")

CASES = [
    # n, sigma, spread, dims, kappa, tau
    (3000, 0.06, 0.3, (161, 163, 165), 3.0, 0.0),
    (600, 0.05, 0.2, (161, 163, 165), 8.0, 0.0),     # thresholds far below FP32's usual: -46
    (700, 0.04, 0.2, (161, 163, 165), 10.0, 0.0),    # -72: nothing counts as interior
    (4000, 0.06, 0.3, (161, 163, 165), 3.0, 2e-2),   # density-aware thresholds
    (300, 0.2, 0.3, (161, 163, 165), 3.0, 0.0),      # Gaussians larger than the grid
    (3000, 0.06, 0.3, (2049, 513, 8), 3.0, 0.0),     # a slab of one tile layer
]


@pytest.mark.parametrize("n,sigma,sd,dims,kappa,tau", CASES)
def test_products(n, sigma, sd, dims, kappa, tau):
    import paper_2604_01844_amd as fgs
    gs = si.gaussians(n, 95, log_scale_mean=float(np.log(sigma)), log_scale_sd=sd)
    h = 1.0 / max(dims)
    gr = dict(origin=tuple(float(np.float32(-0.5 * d * h)) for d in dims), spacing=(float(np.float32(h)),) * 3, dims=dims)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in NAMES]
    grid = fgs.Grid.from_dict(gr)
    ws = fgs.Workspace(DEV)
    vol = fgs.voxelize(*args, grid, kappa=kappa, tau=tau, ws=ws)
    assert ws.n_pairs >= max(96 * n, 64 * ws.s.n_tiles)
    assert oracle.rel_l2(vol.cpu().numpy(), oracle.voxelize(gs, gr, kappa=kappa, tau=tau)) < TOL
    c = si.normals(grid.shape, 96)
    got = fgs.voxelize_backward(*args, grid, torch.from_numpy(c).to(DEV), kappa=kappa, tau=tau, recompute=False, ws=ws)
    ref = oracle.voxelize_bwd(gs, gr, c, kappa=kappa, tau=tau, band=BAND)
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(NAMES, got)}, ref)
    assert max(errs.values()) < TOL, errs
