"""GPU tests of the voxelizer kernels of grids with a wave per tile (8,192
tiles or more): quarters skipped, interior and on the boundary, in list order
(few tiles per Gaussian) and by products along the row (many)."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4    # FP32 kernels against the FP64 oracle, the bar of all parity tests
# Pairs this near the cutoff d^2 = kappa^2 have no unique answer. In needles (standard deviations 30 times apart) the
# form's terms cancel, and d^2 carries ten times the rounding.
BAND, BAND_NEEDLES = 1e-5, 1e-4


@pytest.fixture(scope="module")
def fgs():
    import paper_2604_01844_amd as m
    return m


CASES = [
    # n, log of sigma, spread, dims (8,192 tiles at least, ragged), kappa, tau
    (400, np.log(0.012), 0.3, (161, 163, 165), 3.0, 0.0),   # sigma 2 voxels: list order
    (60, np.log(0.06), 0.3, (161, 163, 165), 3.0, 0.0),     # sigma 10: products, skipped and boundary quarters
    (40, np.log(0.02), 1.2, (168, 160, 161), 3.0, 0.0),     # very elongated
    (30, np.log(0.05), 0.2, (161, 163, 165), 8.0, 0.0),     # thresholds far below FP32's usual: -46
    (60, np.log(0.06), 0.3, (161, 163, 165), 3.0, 2e-2),    # density-aware thresholds
    (200, np.log(0.004), 0.3, (161, 163, 165), 3.0, 0.0),   # below a voxel
    (30, np.log(0.03), 0.3, (2049, 513, 8), 3.0, 0.0),      # a slab of one tile layer
]


@pytest.mark.parametrize("n,mu,sd,dims,kappa,tau", CASES)
def test_large_grids(fgs, n, mu, sd, dims, kappa, tau):
    gs = si.gaussians(n, 31, log_scale_mean=mu, log_scale_sd=sd)
    h = 1.0 / max(dims)
    gr = dict(origin=tuple(float(np.float32(-0.5 * d * h)) for d in dims), spacing=(float(np.float32(h)),) * 3, dims=dims)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in ("mean", "log_scale", "quat", "density")]
    grid = fgs.Grid.from_dict(gr)
    ws = fgs.Workspace(DEV)
    vol = fgs.voxelize(*args, grid, kappa=kappa, tau=tau, ws=ws)
    ref = oracle.voxelize(gs, gr, kappa=kappa, tau=tau)
    assert oracle.rel_l2(vol.cpu().numpy(), ref) < TOL
    assert torch.equal(vol, fgs.voxelize(*args, grid, kappa=kappa, tau=tau))
    c = si.normals(grid.shape, 32)
    got = fgs.voxelize_backward(*args, grid, torch.from_numpy(c).to(DEV), kappa=kappa, tau=tau, recompute=False, ws=ws)
    ref = oracle.voxelize_bwd(gs, gr, c, kappa=kappa, tau=tau, band=BAND_NEEDLES if sd > 1 else BAND)
    got = {k: t.cpu().numpy() for k, t in zip(("mean", "log_scale", "quat", "density"), got)}
    errs = oracle.banded_grad_error(got, ref)
    assert max(errs.values()) < TOL, errs
