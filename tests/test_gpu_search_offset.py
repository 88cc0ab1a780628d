"""The bounded search with the poses and the points far from the origin, where
a coordinate's rounding exceeds the footprint's own: bit for bit the minimum
of the every-point pass."""
import numpy as np
import pytest

from test_gpu_search import _footprint, _poses

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2605_29663_amd as pkg
    return pkg


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("offset", [1e4, 3e4, 1e5])
def test_side_against_corner(pkg, kind, offset):
    """One pose, a 2 x 0.8 m box beside the body origin: a point off the long side's middle, where the
    group's upper bound is attained, and one off a corner, where its lower bound
    is, nearer by up to two units in the last place of the coordinates; leaves
    of one repeated point each (radius 0)."""
    import torch
    rng = np.random.default_rng(int(offset) + kind)
    ctx = pkg.Context(0)
    mid = np.array([0.37, 0.21])
    corners = np.array([[-1, -.4], [1, -.4], [1, .4], [-1, .4]]) + mid
    ctx.set_footprint(kind, np.float32([[*mid, 1, 0.4]]) if kind else corners.astype(np.float32))
    ulp = float(np.spacing(np.float32(offset)))
    wrong = []
    for trial in range(200):
        th, s = rng.uniform(-3.1, 3.1), rng.uniform(0.02, 0.5)
        c, sn = np.cos(th), np.sin(th)
        q = np.float32([offset * rng.uniform(0.8, 1.0), -offset * rng.uniform(0.8, 1.0), c, sn])
        half = np.hypot(1.0, 0.4)
        body = [(0.0, 0.4 + s)]
        body.append((half + s - rng.uniform(0, 2) * ulp) / half * np.array([1.0, 0.4]) * rng.choice([-1, 1], 2))
        ang, far = 2 * np.pi * np.arange(126) / 126, rng.uniform(3.0, 3.4, 126)
        body = np.concatenate([body, np.stack([far * np.cos(ang), far * np.sin(ang)], 1)]) + mid
        x = (q[0] + c * body[:, 0] - sn * body[:, 1]).astype(np.float32)
        y = (q[1] + sn * body[:, 0] + c * body[:, 1]).astype(np.float32)
        pose = torch.tensor(q.reshape(1, 1, 4), device="cuda")
        ctx.set_points(x, y)  # 128 points: evaluated one by one
        ref = float(ctx.sdf_min_poses(pose, kind=kind))
        ctx.set_points(np.repeat(x, 8), np.repeat(y, 8))
        d = float(ctx.sdf_min_poses(pose, kind=kind))
        if d != ref:
            wrong.append((trial, d, ref))
    assert not wrong, wrong[:5]
    ctx.close()


@pytest.mark.parametrize("prims", [4, 27, -3])
@pytest.mark.parametrize("offset", [2e3, 1e4, 1e5, 1e6])
@pytest.mark.parametrize("moving", [False, True])
def test_search_far_from_origin(pkg, prims, offset, moving):
    """Many poses and a field of repeated points (the grid of the coordinates is
    coarse there), d_min and argmin, static and moving."""
    import torch
    rng = np.random.default_rng(int(offset) + abs(prims))
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    n = 3000
    x, y = (rng.uniform(-6, 6, (2, n)) + [[offset], [-offset]]).astype(np.float32)
    vx, vy = (rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.4)).astype(np.float32)
    p = _poses(rng, 29, 5, 1.0)
    p[..., 0] += np.float32(offset)
    p[..., 1] -= np.float32(offset)
    poses = torch.tensor(p, device="cuda")

    def run(sl):
        ctx.set_points(x[sl], y[sl], vx[sl] if moving else None, vy[sl] if moving else None)
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, kind=kind, argmin=True)]

    d, a = run(slice(0, n))
    ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
    for i in range(0, n, 100):
        di, ai = run(slice(i, i + 100))
        less = di < ref
        ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
    np.testing.assert_array_equal(d, ref)
    np.testing.assert_array_equal(a, arg)
    ctx.close()
