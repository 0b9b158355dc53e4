"""GPU tests of the 3D SSIM loss and gradient at the edges of its kernels'
work: tiles of 16 x 16, filtered four outputs at a time, chunks of 64 slices
with a halo of 5, several columns per XCD."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 17, 13), (65, 15, 33), (130, 16, 16), (6, 64, 63), (64, 49, 50)])
def test_sizes(shape):
    import paper_2604_01844_amd as fgs
    rng = np.random.default_rng(sum(shape))
    x = rng.random(shape).astype(np.float32)
    y = (0.7 * x + 0.3 * rng.random(shape)).astype(np.float32)
    loss, g = fgs.ssim3d_loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), scale=0.2)
    rl, rg = oracle.ssim3d_loss_grad(x, y, scale=0.2)
    # FP32 kernels against the FP64 oracle, the bar of all parity tests
    assert abs(float(loss) - rl) < 1e-4 * max(abs(rl), 1e-3)
    assert oracle.rel_l2(g.cpu().numpy(), rg) < 1e-4


def test_outside_the_grid_counts_as_zero():
    """A value that only the clamped loads of a ragged column see stays out: voxels more than a window away from an
    infinity are finite."""
    import paper_2604_01844_amd as fgs
    x = torch.rand((20, 20, 40), generator=torch.Generator().manual_seed(1)).cuda()
    y = torch.rand((20, 20, 40), generator=torch.Generator().manual_seed(2)).cuda()
    x[0, 0, 0] = float("inf")
    _, g = fgs.ssim3d_loss_grad(x, y)
    assert torch.isfinite(g[11:]).all() and torch.isfinite(g[:, 11:]).all() and torch.isfinite(g[:, :, 11:]).all()
