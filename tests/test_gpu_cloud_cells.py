"""Voxel tables and budget cuts of the point-cloud pass at their edges, bit for
bit against the oracle: ranges whose voxels are a plain grid or a hash table,
the robot far from the origin, bins that the budget cuts with few, one
thousand and many more candidates (equal ranges included), budgets around the
number of representatives, and point counts around whole words and
workgroups."""
import numpy as np
import pytest

from test_gpu_cloud import _check, _cloud, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [31, 32, 33, 127, 129, 8191, 8193, 16385])
def test_word_and_block_edges(ctx, m):
    p = _cloud(np.random.default_rng(m), m, spread=6.0)
    kept = _check(ctx, p, (0.1, 0.2), -0.5, 1.5, 5.0, 0.1, 1 << 15)
    for n_out in (1, kept - 1, kept, kept + 1, kept // 2):
        _check(ctx, p, (0.1, 0.2), -0.5, 1.5, 5.0, 0.1, max(n_out, 0))


@pytest.mark.parametrize("voxel", [0.5, 0.0156, 0.0155, 0.01, 0.001])
@pytest.mark.parametrize("center", [(0.0, 0.0), (-3000.3, 77.7), (2.5e5, -1.0e5)])
def test_grid_and_hash_voxels(ctx, voxel, center):
    rng = np.random.default_rng(5)
    p = _cloud(rng, 20000, spread=4.5)
    p[:, :2] += np.float32(center)
    for n_out in (100, 5000, 30000):
        _check(ctx, p, center, -0.5, 1.5, 4.0, voxel, n_out)


@pytest.mark.parametrize("voxel", [0.02, 0.002])
@pytest.mark.parametrize("n", [900, 1024, 1025, 5000, 40000])
def test_many_candidates_in_the_cut_bin(ctx, voxel, n):
    # points on a circle (ranges equal to rounding) and on the axes' mirror
    # images (ranges equal exactly), with some near and far ones around them
    rng = np.random.default_rng(n)
    ang = rng.uniform(0, 2 * np.pi, n // 4 + 1)
    q = np.stack([3 * np.cos(ang), 3 * np.sin(ang)], 1).astype(np.float32)
    ring = np.concatenate([q, q * [-1, 1], q * [1, -1], -q])[:n].astype(np.float32)
    near = rng.uniform(-1, 1, (300, 2)).astype(np.float32)
    far = rng.uniform(3.2, 3.4, (300, 2)).astype(np.float32)
    p = np.concatenate([ring, near, far])
    p = np.concatenate([p, np.zeros((len(p), 1), np.float32)], 1)[rng.permutation(len(p))]
    total = _check(ctx, p, (0.0, 0.0), -1, 1, 6.0, voxel, 1 << 17)
    for n_out in (total // 3, total // 2, total - 400):
        _check(ctx, p, (0.0, 0.0), -1, 1, 6.0, voxel, n_out)


def test_ranges_that_overflow_or_vanish(ctx):
    p = np.float32([[0, 0, 0], [1e19, 0, 0], [3e19, 1e19, 0], [-2e19, 5, 0], [1e-24, 0, 0], [4e-24, 1e-25, 0]])
    _check(ctx, p, (0.0, 0.0), -1, 1, 2.5e19, 1e18, 4)
    _check(ctx, p, (0.0, 0.0), -1, 1, 1e-16, 1e-18, 4)
