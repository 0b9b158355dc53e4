"""GPU tests of the nearest-neighbour scales where the search over cells hands
points on: isolated points, many points in few cells, and both sides of the
sizes that take the brute force."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _volume(dims, cubes, specks, seed):
    v = np.zeros(dims[::-1], dtype=np.float32)
    for c, w, a in cubes:
        v[c[2] - w:c[2] + w + 1, c[1] - w:c[1] + w + 1, c[0] - w:c[0] + w + 1] = a
    r = np.random.Generator(np.random.PCG64(seed))
    for _ in range(specks):
        x, y, z = (r.integers(0, d) for d in dims)
        v[z, y, x] = max(v[z, y, x], 0.2)
    return v


@pytest.mark.parametrize("n,dims,cubes,specks", [
    (1024, (48, 48, 48), [((24, 24, 24), 12, 1.0)], 0),                               # brute force
    (1025, (48, 48, 48), [((24, 24, 24), 12, 1.0)], 0),
    (50000, (96, 96, 96), [((60, 60, 60), 20, 1.0), ((3, 4, 5), 0, 2.0)], 0),         # one voxel far away: one or a few samples
    (50000, (96, 96, 96), [((48, 48, 48), 10, 1.0)], 60),                             # specks all over the margin
    (6000, (128, 128, 128), [((64, 64, 64), 0, 1.0)], 0),                             # all in one voxel
    (20000, (128, 128, 128), [((20, 20, 20), 2, 1.0), ((100, 100, 100), 2, 1.0)], 0), # two cells' worth
    (3000, (64, 64, 64), [], 3000),                                                   # nothing but isolated voxels
])
def test_scales(n, dims, cubes, specks):
    """The log-scales are those of the nearest other mean, found by a k-d tree
    over the means that the call returned, their logarithm taken in FP32 on
    the GPU too. A squared distance is within a few FP32 ulps, 2e-7 relative; with an
    ulp or two of the logarithm (of up to 28) that stays within 4e-6."""
    import paper_2604_01844_amd as fgs
    from scipy.spatial import cKDTree
    vol = torch.from_numpy(_volume(dims, cubes, specks, 7)).to(DEV)
    u = torch.from_numpy(np.random.Generator(np.random.PCG64(8)).random((4, n))).to(DEV)
    grid = fgs.Grid((-0.5,) * 3, (1.0 / max(dims),) * 3, dims)
    mean, ls, _, _ = fgs.gradient_init(vol, grid, u, min_scale=1e-12, weighting="intensity")
    m = mean.cpu().numpy().astype(np.float64).T
    d = cKDTree(m).query(m, k=2)[0][:, 1]
    ref = torch.log(torch.from_numpy(np.maximum(d, 1e-12).astype(np.float32)).to(DEV)).cpu().numpy()
    got = ls.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got, np.broadcast_to(got[0], got.shape))
    np.testing.assert_allclose(got[0], ref, rtol=0, atol=4e-6)
    again = fgs.gradient_init(vol, grid, u, min_scale=1e-12, weighting="intensity")[1]
    assert torch.equal(ls, again)
