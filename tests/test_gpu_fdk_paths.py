"""GPU tests of FDK's backprojection on both sides of the line between a voxel
per thread and pieces of the detector staged in LDS (2^19 voxels and little
padding), with pieces that fit the buffer and pieces that don't, in runs of 4
and of 16 voxels; and of the filter's rows that end inside a segment."""
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


@pytest.mark.parametrize("det_w,det_h,views,dims,extent", [
    (96, 90, 3, (96, 95, 63), 1.0),      # 574,560 voxels: pieces, runs of 4, ragged
    (96, 90, 3, (96, 95, 54), 1.0),      # 492,480: a voxel per thread
    (40, 44, 3, (96, 95, 63), 0.5),      # less than a pixel per voxel, past the detector
    (640, 24, 4, (96, 95, 63), 1.2),     # pieces too wide for the buffer
    (640, 24, 2, (163, 161, 165), 1.2),  # the same in runs of 16
    (96, 90, 2, (520, 510, 3), 1.0),     # a slab of three slices: padded by a third, a voxel per thread
    (96, 90, 2, (520, 510, 4), 1.0),     # of four: pieces
    (31, 40, 3, (20, 17, 5), 1.0),       # a row ends in the first piece of a segment,
    (63, 33, 3, (20, 17, 5), 1.0),       # at its end,
    (66, 33, 3, (20, 17, 5), 1.0),       # in the second,
    (545, 9, 2, (20, 17, 5), 0.5),       # and in the second segment
])
def test_fdk_paths(det_w, det_h, views, dims, extent):
    import paper_2604_01844_amd as fgs
    ph = si.phantom(10, 100)
    gd = si.geometry(det_w, det_h)
    ang = si.angles(views)
    img = oracle.phantom_project(ph, gd, ang).astype(np.float32)
    img += 0.05 * si.normals(img.shape, 3)
    gr = dict(origin=tuple(float(np.float32(-0.5 * extent + 0.01 * a)) for a in range(3)),
              spacing=tuple(float(np.float32(extent / max(d, 20))) for d in dims), dims=dims)
    vol = fgs.fdk(torch.from_numpy(img).to(DEV), fgs.Geometry.from_dict(gd, ang), fgs.Grid.from_dict(gr))
    ref = oracle.fdk(img, gd, ang, gr)
    assert np.isfinite(ref).all() and oracle.rel_l2(vol.cpu().numpy(), ref) < TOL
