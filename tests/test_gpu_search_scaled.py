"""Poses whose (cos, sin) is no rotation: rounded to 16 bits, scaled, mixed with
rotations; bit for bit as every point evaluated, and bounded like rotations."""
import numpy as np
import pytest

from test_gpu_search import _footprint, _poses

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2605_29663_amd as pkg
    return pkg


def _scaled(rng, p, how):
    p = p.copy()
    if how == "half":
        p[..., 2:] = p[..., 2:].astype(np.float16)
    elif how == "any":
        p[..., 2:] *= np.exp(rng.uniform(-4, 4, p.shape[:2] + (1,)))
    elif how == "few":
        p[::7, 1, 2:] *= np.float32(1.7)
    else:  # lengths around those that have no bounds, and none
        p[..., 2:] *= rng.choice([0.0, 1e-30, 0.9e-3, 1.1e-3, 0.9e3, 1.1e3, 1e18], p.shape[:2] + (1,))
    return p.astype(np.float32)


@pytest.mark.parametrize("prims", [3, 16, 40, -1, -4, -20])
@pytest.mark.parametrize("how", ["half", "any", "few", "ends"])
@pytest.mark.parametrize("n,moving", [(2500, False), (2500, True), (9000, False)])
def test_scaled_poses_equal_every_point(pkg, prims, how, n, moving):
    import torch
    rng = np.random.default_rng(n + 10 * abs(prims) + len(how))
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    x, y = rng.uniform(-6, 6, (2, n)).astype(np.float32)
    vx, vy = (rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.4)).astype(np.float32)
    poses = torch.tensor(_scaled(rng, _poses(rng, 31, 3, 1.0), how), device="cuda")

    def run(sl):
        ctx.set_points(x[sl], y[sl], vx[sl] if moving else None, vy[sl] if moving else None)
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, kind=kind, argmin=True)]

    d, a = run(slice(0, n))
    ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
    step = int(20000 / (10.75 * abs(prims) + 6))
    for i in range(0, n, step):
        di, ai = run(slice(i, min(i + step, n)))
        less = di < ref
        ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
    np.testing.assert_array_equal(d, ref)
    np.testing.assert_array_equal(a, arg)
    ctx.close()


def _us(f, n=3):
    """Fastest of a few GPU times of f."""
    import torch
    f()
    best = np.inf
    for _ in range(n):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        f()
        e[1].record()
        e[1].synchronize()
        best = min(best, 1e3 * e[0].elapsed_time(e[1]))
    return best


@pytest.mark.parametrize("prims", [16, -4])
def test_scaled_poses_are_bounded(pkg, prims):
    """20480 poses against 8192 points take a few times what rotations take (25
    to 40 times where every point of every pose is evaluated)."""
    import torch
    rng = np.random.default_rng(1)
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    ctx.set_points(*rng.uniform(-8, 8, (2, 8192)).astype(np.float32))
    p = _poses(rng, 20480, 1, 0.5)
    us = []
    for how in (None, "half", "few"):
        poses = torch.tensor(p if how is None else _scaled(rng, np.tile(p, (1, 2, 1)), how)[:, 1:], device="cuda")
        us.append(_us(lambda: ctx.sdf_min_poses(poses, kind=kind)))
    print(us)
    assert max(us[1:]) < 8 * us[0], us
    ctx.close()
