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
