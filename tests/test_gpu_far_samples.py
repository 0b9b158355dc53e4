"""GPU tests of the samplers of a volume for points far outside it or at
infinity, whose voxel index is past the range of an int: such a point takes
nothing from the volume."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FAR = [1e9, -1e9, 3e12, -3e12, 1e30, float("inf"), float("-inf")]  # a voxel is 1/24: index 2^31 is at 9e7


def test_patch_of_a_far_mean_is_zero():
    """One axis far outside, the other two inside the grid."""
    import paper_2604_01844_amd as fgs
    from paper_2604_01844_amd.mlp import K_IN
    grid = fgs.Grid((-0.5,) * 3, (1.0 / 24,) * 3, (24, 24, 24))
    vol = torch.from_numpy(1.0 + si.normals(grid.shape, 81).astype(np.float32) ** 2).to(DEV)
    near = torch.from_numpy(0.2 * si.normals((3, 50), 82).astype(np.float32)).to(DEV)
    mean = near.clone()
    far = []
    for k, v in enumerate(FAR):
        for a in range(3):
            far.append(2 * (3 * k + a))  # among others in the same workgroup and wave
            mean[a, far[-1]] = v
    net = fgs.InitMLP(fgs.InitMLP.init_weights(1))
    x, xt, rows = net.features(vol, grid, 1.0, mean, transposed=True)
    ref, _, _ = net.features(vol, grid, 1.0, near)
    assert torch.equal(x, xt.T)
    x = x.view(torch.bfloat16)[:50]
    ref = ref.view(torch.bfloat16)[:50]
    rest = [i for i in range(50) if i not in far]
    assert torch.equal(x[rest], ref[rest])
    assert (x[far][:, :512] == 0).all() and x.shape[1] == K_IN
    assert torch.equal(x[:, 512:515], (2 * mean.T).to(torch.bfloat16))


@pytest.mark.parametrize("dims", [(17, 17, 17), (96, 97, 63), (165, 161, 161)])  # one voxel, runs of 4, of 16
def test_fdk_voxels_beside_the_source(dims):
    """A plane of voxels 2^-25 in front of the source, whose rays meet the
    detector's plane up to 2^31 pixels away, and voxels behind the source. A
    pixel coordinate is 5,120 t0 at most in front of that plane, a few ulps of
    which are 1e-3 pixel, and neighbouring samples differ by about their own size."""
    import paper_2604_01844_amd as fgs
    h = 1.0 / 16
    at = 8  # this plane's x is 1/2 - 2^-25, exactly
    gr = dict(origin=(0.5 - 2.0 ** -25 - (at + 0.5) * h, -0.5 * dims[1] * h, -0.5 * dims[2] * h), spacing=(h,) * 3, dims=dims)
    gd = dict(mode="cone", sod=0.5, sdd=2.0, det_w=64, det_h=48, pitch_u=2.0 / 160, pitch_v=2.0 / 160, off_u=0.0, off_v=0.0)
    ang = np.zeros(1, dtype=np.float32)
    img = (1.0 + 0.1 * si.normals((1, 48, 64), 83)).astype(np.float32)
    vol = fgs.fdk(torch.from_numpy(img).to(DEV), fgs.Geometry.from_dict(gd, ang), fgs.Grid.from_dict(gr)).cpu().numpy()
    ref = oracle.fdk(img, gd, ang, gr)
    assert np.abs(ref[..., :at]).max() > 0 and np.abs(ref[..., at]).max() > 1e12
    assert (vol[..., at + 1:] == 0).all() and ((ref == 0) <= (vol == 0)).all()
    assert oracle.rel_l2(vol[..., :at], ref[..., :at]) < 1e-3
    np.testing.assert_allclose(vol[..., at], ref[..., at], rtol=1e-3)
