"""Sets whose points are nearly equally near: walls, a ring, one place, all far
away.  Bit for bit as every point evaluated; and bounded, not evaluated one by
one, where the nearest points are far from the footprint."""
import numpy as np
import pytest

from test_gpu_search import _footprint, _poses
from test_gpu_search_scaled import _us

pytestmark = pytest.mark.gpu
SETS = ["wall", "ring", "far wall", "very far", "one place", "two places", "edge of the table"]


def _set(rng, name, n):
    x, y = rng.uniform(-8, 8, (2, n))
    a = rng.uniform(0, 2 * np.pi, n)
    if name == "wall":
        y[:] = 3
    elif name == "ring":
        x, y = 5 * np.cos(a), 5 * np.sin(a)
    elif name == "far wall":
        y = 20 + 0.02 * rng.normal(0, 1, n)
    elif name == "very far":
        x, y = 3e4 * np.cos(a), 3e4 * np.sin(a)
    elif name == "one place":
        x[:], y[:] = 1.7, -0.4
    elif name == "two places":
        x[:], y[:] = 1.7, -0.4
        x[::3], y[::3] = -1.9, 0.8
    elif name == "edge of the table":  # around the grid that bounds the near points
        r = rng.uniform(0.6, 2.2, n)
        x, y = r * np.cos(a), r * np.sin(a)
    return x.astype(np.float32), y.astype(np.float32)


@pytest.mark.parametrize("prims", [3, 16, 33, 64, -1, -4, -20])
@pytest.mark.parametrize("name", SETS)
@pytest.mark.parametrize("n,moving", [(400, False), (3000, False), (3000, True), (9000, False)])
def test_sets_equal_every_point(prims, name, n, moving):
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(n + 7 * abs(prims) + len(name))
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    x, y = _set(rng, name, n)
    vx, vy = (rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.4)).astype(np.float32)
    poses = torch.tensor(_poses(rng, 23, 3, 0.5), device="cuda")

    def run(sl, argmin=True):
        ctx.set_points(x[sl], y[sl], vx[sl] if moving else None, vy[sl] if moving else None)
        if not argmin:
            return ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, kind=kind).cpu().numpy()
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, kind=kind, argmin=True)]

    d, a = run(slice(0, n))
    np.testing.assert_array_equal(run(slice(0, n), False), d)
    ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
    step = int(40000 / (10.75 * abs(prims) + 6))
    for i in range(0, n, step):
        di, ai = run(slice(i, min(i + step, n)))
        less = di < ref
        ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
    np.testing.assert_array_equal(d, ref)
    # the minimum is taken over squares: several of them may round to the
    # pieces' equal distances, and then any of those points attains it
    for g in np.argwhere(a != arg):
        at = a[tuple(g)]
        assert run(slice(at, at + 1), False)[tuple(g)] == d[tuple(g)], (name, g)
    if "place" in name and not moving:
        np.testing.assert_array_equal(a, arg)  # repeated points: the lowest index
    ctx.close()


@pytest.mark.parametrize("prims", [16, -4])
def test_far_sets_are_bounded(prims):
    """20480 poses against 8192 points at nearly one distance: a few times what a
    field of as many takes (30 to 40 times with the bounds of the near table)."""
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(3)
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    poses = torch.tensor(_poses(rng, 20480, 1, 0.5), device="cuda")
    us = {}
    for name in ("field", "ring", "far wall"):
        ctx.set_points(*_set(rng, name, 8192))
        us[name] = _us(lambda: ctx.sdf_min_poses(poses, kind=kind))
    print(us)
    assert max(us.values()) < 16 * us["field"], us
    ctx.close()
