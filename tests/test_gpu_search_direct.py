"""Sets of at most 512 points that are searched without a hierarchy, and moving
sets with one, against pieces so small that every point of them is evaluated."""
import numpy as np
import pytest

from paper_2605_29663_amd import scenes
from test_gpu_search import _footprint, _poses

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2605_29663_amd as pkg
    return pkg


def _against_pieces(ctx, run, n, prims):
    """d_min and argmin of the whole set against its pieces: points times
    primitives far below where a set is searched."""
    d, a = run(slice(0, n))
    ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
    step = int(20000 / (10.75 * abs(prims) + 6))
    for i in range(0, n, step):
        di, ai = run(slice(i, min(i + step, n)))
        less = di < ref  # pieces in index order: the first of equal distances stays
        ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
    np.testing.assert_array_equal(d, ref)
    np.testing.assert_array_equal(a, arg)


@pytest.mark.parametrize("n,prims", [(512, 9), (511, 16), (512, 17), (300, 33), (512, 64), (505, -12), (512, -32)])
@pytest.mark.parametrize("moving", [False, True])
def test_direct_equals_every_point(pkg, n, prims, moving):
    import torch
    rng = np.random.default_rng(n + abs(prims))
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    x, y = rng.uniform(-4, 4, (2, n)).astype(np.float32)
    x[:9], y[:9] = x[n // 2:n // 2 + 9], y[n // 2:n // 2 + 9]  # ties
    vx, vy = (rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.4)).astype(np.float32)
    vx[:9], vy[:9] = vx[n // 2:n // 2 + 9], vy[n // 2:n // 2 + 9]
    valid = (rng.random(n) < 0.9).astype(np.uint8)
    poses = torch.tensor(_poses(rng, 41, 5, 1.0), device="cuda")

    def run(sl):
        ctx.set_points(x[sl], y[sl], vx[sl] if moving else None, vy[sl] if moving else None, valid[sl])
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, kind=kind, argmin=True)]

    _against_pieces(ctx, run, n, prims)
    ctx.close()


@pytest.mark.parametrize("n", [600, 4097, 8193, 33000])
@pytest.mark.parametrize("T,dt,speed", [(1, 1e-6, 1.0), (60, 0.15, 1.0), (60, 2.0, 50.0), (40, 0.1, 3e38)])
def test_moving_leaves_equal_every_point(pkg, n, T, dt, speed):
    import torch
    rng = np.random.default_rng(n + T)
    ctx = pkg.Context(0)
    ctx.set_footprint(0, scenes.star_polygon(rng, 9).astype(np.float32))
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

    def run(sl):
        ctx.set_points(x[sl], y[sl], vx[sl], vy[sl])
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=dt * T / 7, state_offset=1, argmin=True)]

    _against_pieces(ctx, run, n, 9)
    ctx.close()
