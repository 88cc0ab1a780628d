"""Range limits far above the points' ranges, and budgets that cut a crowded bin:
bit for bit the oracle, and as fast as a close limit."""
import numpy as np
import pytest

from test_gpu_cloud import _check, ctx  # noqa: F401
from test_gpu_search_scaled import _us

pytestmark = pytest.mark.gpu


def _disc(rng, n, r):
    a, q = rng.uniform(0, 2 * np.pi, n), r * np.sqrt(rng.random(n))
    return np.stack([q * np.cos(a), q * np.sin(a), np.zeros(n)], 1).astype(np.float32)


# limits at the edges of the bins' 8 and 32 octaves below the largest range
@pytest.mark.parametrize("r_max", [41.0, 640.0, 641.0, 1e4, 4e6, 1e9])
@pytest.mark.parametrize("n_out", [1, 700, 5000, 9000, 40000])
def test_range_limit_far_above_the_points(ctx, r_max, n_out):
    rng = np.random.default_rng(n_out)
    p = np.concatenate([_disc(rng, 20000, 40.0), _disc(rng, 2000, 0.3), _disc(rng, 100, 1e-3)])
    p = p[rng.permutation(len(p))]
    p[3, :2] = 0.7 * min(r_max, 1e6)  # one far from the others
    _check(ctx, p, (0.0, 0.0), -1, 1, r_max, 0.05 if r_max < 1e6 else 50.0, n_out)
    if r_max < 1e6:
        _check(ctx, p + np.float32([3.3, -1.7, 0]), (3.3, -1.7), -1, 1, r_max, 0.01, n_out)


# one bin with far more candidates than the selection counts at once: ranges that
# differ in their lowest bits only, all equal (the index decides), and in between
@pytest.mark.parametrize("spread", [0.0, 1e-6, 1e-4, 1e-2])
@pytest.mark.parametrize("share", [0.001, 0.3, 0.77, 0.999])
def test_crowded_bin(ctx, spread, share):
    rng = np.random.default_rng(int(1e6 * spread) + int(100 * share))
    n = 60000
    k = np.arange(n)
    x = (k % 245 + 1).astype(np.float32)  # 245 x 245 voxels of 1 m
    y = (k // 245 + 1).astype(np.float32)
    if spread == 0.0:  # the axes' mirror images: ranges equal exactly, four by four
        x, y = np.where(k % 2, x, -x), np.where(k % 4 < 2, y, -y)
        c = (0.0, 0.0)
    else:  # a thin ring
        a = 2 * np.pi * k / n
        r = 500.0 * (1 + spread * rng.uniform(-1, 1, n))
        x, y, c = r * np.cos(a), r * np.sin(a), (0.0, 0.0)
    p = np.stack([x, y, 0 * x], 1).astype(np.float32)[rng.permutation(n)]
    total = _check(ctx, p, c, -1, 1, 1000.0, 0.01, 1 << 17)
    _check(ctx, p, c, -1, 1, 1000.0, 0.01, max(int(share * total), 1))


def test_no_slower_without_a_limit(ctx):
    """2^20 points within 40 m, budget 8192: the limit at 60 m and at 1e4 m take the
    same table and the same selection."""
    import torch
    rng = np.random.default_rng(0)
    xyz = torch.tensor(_disc(rng, 1 << 20, 40.0), device="cuda")
    us = [_us(lambda: ctx.cloud_downsample(xyz, (0.0, 0.0), -1.0, 1.0, r, 0.05, 8192)) for r in (60.0, 1e4)]
    print(us)
    assert us[1] < 1.6 * us[0], us
