"""GPU tests of the samplers of a volume for points far outside it or at
infinity, whose voxel index is past the range of an int: such a point takes
nothing from the volume."""
import numpy as np
import pytest
import torch

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
