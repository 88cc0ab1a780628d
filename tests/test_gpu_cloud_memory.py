"""The point-cloud pass's workspace stays within what the header states."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# just above a power of two, where the hash table has four slots a point
@pytest.mark.parametrize("m,voxels", [((1 << 19) + 1, (0.01,)), ((1 << 19) + 1, (0.05, 0.01)), (1 << 20, (0.01, 0.1)),
                                      (3000, (0.01,))])
def test_workspace_per_point(m, voxels):
    import torch
    import paper_2605_29663_amd as pkg
    ctx = pkg.Context(0)
    rng = np.random.default_rng(1)
    xyz = torch.tensor(rng.uniform(-1, 1, (m, 3)).astype(np.float32) * np.float32([36, 36, 1]), device="cuda")
    # the outputs' allocation and the kernels' code come before the measurement
    other = pkg.Context(0)
    for v in voxels:
        other.cloud_downsample(xyz, (0.0, 0.0), -1.0, 1.0, 36.0, v, 8192)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for v in voxels:
        ctx.cloud_downsample(xyz, (0.0, 0.0), -1.0, 1.0, 36.0, v, 8192)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    print(m, voxels, used, used / m)
    # allocations come in pieces of 2 MB, four buffers
    assert used <= max(57 * m, 4 << 20) + (8 << 20)
    other.close()
    ctx.close()
