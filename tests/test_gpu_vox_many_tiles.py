"""GPU test of the voxelizer's backward on the largest grids: 2^24 tiles whose
lists average a batch of 64, where four waves per tile would pass the
work-items that a launch holds."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_backward_of_2_24_tiles():
    """A sheet of voxels one thick. The gradients of the Gaussians near the
    first corner are those of a small grid there, whose voxels have the same
    coordinates (same origin and spacing): the same pairs, sums of the same
    terms in FP32."""
    import paper_2604_01844_amd as fgs
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 110 GB of device memory")
    dims, near = (65535 * 8, 257 * 8, 1), (512, 512, 1)
    n, n_near = 22_000_000, 400
    r = torch.Generator(device=DEV).manual_seed(5)
    mean = torch.rand(3, n, device=DEV, generator=r) * torch.tensor([[float(dims[0])], [float(dims[1])], [0.0]], device=DEV)
    mean[:2, :n_near] = 48.0 + 416.0 * torch.rand(2, n_near, device=DEV, generator=r)  # whole in the small grid
    mean[2] = 0.5
    args = [mean, torch.full((3, n), 2.3, device=DEV), torch.zeros(4, n, device=DEV), torch.ones(n, device=DEV)]
    args[2][0] = 1.0
    grid = fgs.Grid((0.0,) * 3, (1.0,) * 3, dims)
    g = torch.randn(grid.shape, device=DEV, generator=r)
    ws = fgs.Workspace(DEV)
    got = fgs.voxelize_backward(*args, grid, g, ws=ws)
    tiles = 65535 * 257
    assert tiles >= 1 << 24 and 64 * tiles <= ws.n_pairs < 96 * n
    small = [t[..., :n_near].contiguous() for t in args]
    ref = fgs.voxelize_backward(*small, fgs.Grid((0.0,) * 3, (1.0,) * 3, near), g[:, :512, :512].contiguous())
    for a, b in zip(got, ref):
        torch.testing.assert_close(a[..., :n_near], b, rtol=1e-5, atol=1e-5 * float(b.abs().max() + 1e-30))
