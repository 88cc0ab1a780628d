"""Leaves of moving points, bounded at the middle of the latest horizon: bit for
bit the minimum over pieces that are evaluated point by point, for horizons
from none to long, slow, fast and overflowing velocities, and sets on both
sides of the sorting paths' limits."""
import numpy as np
import pytest

from paper_2605_29663_amd import scenes
from test_gpu_search import _poses

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [600, 4097, 8193, 33000])
@pytest.mark.parametrize("T,dt,speed", [(1, 1e-6, 1.0), (8, 0.05, 2.0), (60, 0.15, 1.0), (60, 2.0, 50.0), (40, 0.1, 3e38)])
def test_moving_leaves_equal_every_point(n, T, dt, speed):
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(n + T)
    ctx = pkg.Context(0)
    poly = scenes.star_polygon(rng, 9).astype(np.float32)
    ctx.set_footprint(0, poly)
    x, y = rng.uniform(-8, 8, (2, n)).astype(np.float32)
    v = rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.5)
    if speed > 1e30:  # a few equal velocities whose way overflows, the others slow
        v[:, rng.random(n) < 0.03] = speed
    else:
        v *= speed
    vx, vy = v.astype(np.float32)
    # a plan over this horizon, as a controller makes before the next scan
    ctx.set_points(x[:100], y[:100])
    U = torch.zeros((T, 2), device="cuda")
    ctx.mppi_step(scenes.params("c1", K=64, T=T, dt=dt), np.zeros(3, np.float32), U, 1, 0)
    poses = torch.tensor(_poses(rng, 19, 7, 1.5), device="cuda")

    def run(sl, offset):
        ctx.set_points(x[sl], y[sl], vx[sl], vy[sl])
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=dt * T / 7, state_offset=offset, argmin=True)]

    for offset in (0, 1):
        d, a = run(slice(0, n), offset)
        ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
        for i in range(0, n, 500):
            di, ai = run(slice(i, min(i + 500, n)), offset)
            less = di < ref
            ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
        np.testing.assert_array_equal(d, ref)
        np.testing.assert_array_equal(a, arg)
