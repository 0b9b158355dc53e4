"""GPU tests of the voxelizer on grids of 8,192 tiles or more with a fixed key
capacity, where the kernel (list order, or products along the row) is picked
on the device: the bits are those of a call that reads its count back, on both
sides of the line and whatever the capacity, also where that call takes short
lists by whole tiles. The lists of the product cases
span several batches of 64, of interior and boundary pairs."""
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
    # n, sigma, spread, half-width of the body, dims, tau, product
    (3500, 0.06, 0.3, 0.15, (161, 163, 165), 0.0, True),   # lists of up to 1,000 and more
    (4500, 0.06, 0.3, 0.15, (161, 163, 165), 2e-2, True),
    (500, 0.08, 0.6, 0.2, (2049, 513, 8), 0.0, True),      # one layer of tiles
    (9000, 0.015, 0.3, 0.3, (161, 163, 165), 0.0, False),
    (3000, 0.015, 0.3, 0.2, (161, 163, 165), 0.0, False),  # fewer than 16 pairs per tile: whole tiles
    (3000, 0.015, 0.3, 0.2, (209, 208, 211), 0.0, False),  # and 16 tiles per workgroup
]


@pytest.mark.parametrize("n,sigma,sd,half,dims,tau,product", CASES)
def test_capacity_keeps_bits(n, sigma, sd, half, dims, tau, product):
    import paper_2604_01844_amd as fgs
    gs = si.gaussians(n, 91, log_scale_mean=float(np.log(sigma)), log_scale_sd=sd, lo=-half, hi=half)
    h = 1.0 / max(dims)
    gr = dict(origin=tuple(float(np.float32(-0.5 * d * h)) for d in dims), spacing=(float(np.float32(h)),) * 3, dims=dims)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in NAMES]
    grid = fgs.Grid.from_dict(gr)
    ws = fgs.Workspace(DEV)
    vol = fgs.voxelize(*args, grid, tau=tau, ws=ws)
    assert (ws.n_pairs >= max(96 * n, 64 * ws.s.n_tiles)) == product
    lists = fgs.binning_dump(ws)["tile_start"].diff()
    assert int(lists.max()) > (200 if product else 20)
    c = si.normals(grid.shape, 92)
    cd = torch.from_numpy(c).to(DEV)
    got = fgs.voxelize_backward(*args, grid, cd, tau=tau, recompute=False, ws=ws)
    # a capacity just enough, and one that reaches the line whatever the count
    for cap in (ws.n_pairs, max(4 * ws.n_pairs, 128 * n, 128 * ws.s.n_tiles)):
        wc = fgs.Workspace(DEV)
        wc.set_capacity(cap)
        assert torch.equal(vol, fgs.voxelize(*args, grid, tau=tau, ws=wc))
        again = fgs.voxelize_backward(*args, grid, cd, tau=tau, recompute=False, ws=wc)
        assert all(torch.equal(a, b) for a, b in zip(got, again))
        assert not wc.overflowed()[0]
    assert oracle.rel_l2(vol.cpu().numpy(), oracle.voxelize(gs, gr, tau=tau)) < TOL
    ref = oracle.voxelize_bwd(gs, gr, c, tau=tau, band=BAND)
    errs = oracle.banded_grad_error({k: t.cpu().numpy() for k, t in zip(NAMES, got)}, ref)
    assert max(errs.values()) < TOL, errs


def test_capacity_too_small_bins_nothing():
    import paper_2604_01844_amd as fgs
    n, dims = 4000, (161, 163, 165)
    gs = si.gaussians(n, 93, log_scale_mean=float(np.log(0.06)), lo=-0.15, hi=0.15)
    args = [torch.from_numpy(gs[k]).to(DEV) for k in NAMES]
    grid = fgs.Grid((-0.5,) * 3, (1.0 / 165,) * 3, dims)
    wc = fgs.Workspace(DEV)
    wc.set_capacity(600000)  # past the line (592,704), below the call's pairs
    vol = fgs.voxelize(*args, grid, ws=wc)
    got = fgs.voxelize_backward(*args, grid, torch.ones(grid.shape, device=DEV), recompute=False, ws=wc)
    assert (vol == 0).all() and all((t == 0).all() for t in got)
    over, need = wc.overflowed()
    assert over and need > 600000
