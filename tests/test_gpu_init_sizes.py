"""GPU tests of the initialisation kernels at the sizes where their tiling can
go wrong: FDK's filter (rows of 32, segments of 512 samples, both parities) and
backprojection (staged detector pieces, views sampled from global memory, runs
of 4 and of 16 voxels)."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# FP32 against FP64: a sample's coordinate on a detector of up to 640 pixels is off by a few ulps of 640 (1e-4 pixel),
# and neighbouring filtered samples differ by about their own size.
TOL = 1e-4


@pytest.fixture(scope="module")
def fgs():
    import paper_2604_01844_amd as m
    return m


@pytest.mark.parametrize("det_w,det_h,views,dims,extent", [
    (33, 17, 5, (7, 9, 5), 1.0),          # one short odd segment, a last row group of 21
    (1, 3, 2, (3, 2, 1), 1.0),            # a single column: only the centre tap
    (65, 32, 3, (17, 33, 6), 0.5),        # patches cut by the grid's ends
    (513, 9, 4, (20, 18, 9), 0.1),        # a second segment of one sample
    (640, 24, 6, (24, 20, 16), 1.2),      # pieces too wide for the buffer, voxels past the detector
    (1100, 5, 2, (16, 16, 4), 0.05),      # three segments
    (96, 96, 3, (163, 161, 165), 1.0),    # runs of 16 voxels, the last one ragged
])
def test_fdk_sizes(fgs, det_w, det_h, views, dims, extent):
    ph = si.phantom(10, 100)
    gd = si.geometry(det_w, det_h)
    ang = si.angles(views)
    img = oracle.phantom_project(ph, gd, ang).astype(np.float32)
    img += 0.05 * si.normals(img.shape, 3)
    gr = dict(origin=tuple(float(np.float32(-0.5 * extent + 0.01 * a)) for a in range(3)),
              spacing=tuple(float(np.float32(extent / d)) for d in dims), dims=dims)
    vol = fgs.fdk(torch.from_numpy(img).to(DEV), fgs.Geometry.from_dict(gd, ang), fgs.Grid.from_dict(gr))
    ref = oracle.fdk(img, gd, ang, gr)
    assert np.isfinite(ref).all() and oracle.rel_l2(vol.cpu().numpy(), ref) < TOL


def _blob(dims, centre, width):
    z, y, x = np.meshgrid(*(np.arange(d) for d in dims[::-1]), indexing="ij")
    d2 = sum(((c - o) / w) ** 2 for c, o, w in zip((x, y, z), centre, width))
    return (d2 < 1.0).astype(np.float32)


@pytest.mark.parametrize("n,dims,origin,blobs", [
    (1, (16, 16, 16), -0.5, [((8, 8, 8), (4, 4, 4))]),                      # no neighbour at all
    (2, (16, 16, 16), -0.5, [((2, 2, 2), (1.2, 1.2, 1.2)), ((13, 13, 13), (1.2, 1.2, 1.2))]),  # far apart: many rings
    (5000, (40, 36, 33), -0.5, [((20, 18, 16), (12, 9, 11))]),
    (5000, (96, 96, 96), -0.5, [((3, 3, 3), (1.2, 1.2, 1.2)), ((92, 90, 91), (1.2, 1.2, 1.2))]),  # two dense clusters
    (3000, (200, 1, 1), -0.5, [((100, 0, 0), (50, 1, 1))]),                 # a row of cells
    (4000, (8, 8, 8), -0.5, [((4, 4, 4), (3, 3, 3))]),                      # too small a grid for the cells: brute force
    (3000, (64, 64, 64), 100.0, [((32, 32, 32), (20, 20, 20))]),            # coordinates large against the cells
])
def test_nearest_neighbour_scales(fgs, n, dims, origin, blobs):
    """The log-scales are those of the nearest other mean, found by a k-d tree
    over the means that the call returned, their logarithm taken in FP32 on
    the GPU too (its own rounding is an ulp or two of up to 9). A squared
    distance is within a few FP32 ulps, 2e-7 relative; with one ulp of the
    logarithm that stays within 1e-6."""
    from scipy.spatial import cKDTree
    vol = sum(_blob(dims, c, w) for c, w in blobs)
    vol = vol * (1.0 + 0.1 * si.normals(vol.shape, 4))
    u = np.random.Generator(np.random.PCG64(5)).random((4, n))
    grid = fgs.Grid((origin,) * 3, (1.0 / 64,) * 3, dims)
    mean, ls, _, _ = fgs.gradient_init(torch.from_numpy(vol.astype(np.float32)).to(DEV), grid,
                                       torch.from_numpy(u).to(DEV), min_scale=1e-12, weighting="intensity")
    m = mean.cpu().numpy().astype(np.float64).T
    d = cKDTree(m).query(m, k=2)[0][:, 1]
    ref = torch.log(torch.from_numpy(np.maximum(d, 1e-12).astype(np.float32)).to(DEV)).cpu().numpy()
    got = ls.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got, np.broadcast_to(got[0], got.shape))
    if n == 1:
        assert np.isinf(got).all()
    else:
        np.testing.assert_allclose(got[0], ref, rtol=0, atol=1e-6)
