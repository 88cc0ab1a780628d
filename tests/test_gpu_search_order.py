"""The spatial order behind the search: sets that alternate between two sources,
thin sets along an axis, and sets with most points in one place."""
import numpy as np
import pytest

from test_gpu_search import _footprint, _poses
from test_gpu_search_scaled import _us

pytestmark = pytest.mark.gpu


def _set(rng, name, n):
    x, y = rng.uniform(-8, 8, (2, n))
    if name == "alternating":
        y[::2] = 3.0
        x[1::2] *= 4
        y[1::2] *= 4
    elif name == "thin":
        x, y = 4.0 + 0.001 * y, 2.0 * x
    elif name == "mostly one place":
        x[: n - n // 20], y[: n - n // 20] = 3.0, -2.5
    return x.astype(np.float32), y.astype(np.float32)


@pytest.mark.parametrize("n", [600, 4097, 9000, 33000])
@pytest.mark.parametrize("name", ["field", "alternating", "thin", "mostly one place"])
@pytest.mark.parametrize("moving", [False, True])
def test_ordered_sets_equal_every_point(n, name, moving):
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(n + len(name))
    kind, geom = _footprint(rng, 7)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    x, y = _set(rng, name, n)
    vx, vy = (rng.uniform(-1, 1, (2, n)) * (rng.random(n) < 0.4)).astype(np.float32)
    poses = torch.tensor(_poses(rng, 19, 3, 1.0), device="cuda")

    def run(sl):
        ctx.set_points(x[sl], y[sl], vx[sl] if moving else None, vy[sl] if moving else None)
        return [t.cpu().numpy() for t in ctx.sdf_min_poses(poses, dt=0.2, state_offset=1, argmin=True)]

    d, a = run(slice(0, n))
    ref, arg = np.full(d.shape, np.inf, np.float32), np.full(d.shape, -1)
    for i in range(0, n, 240):
        di, ai = run(slice(i, min(i + 240, n)))
        less = di < ref
        ref, arg = np.where(less, di, ref), np.where(less, ai + i, arg)
    np.testing.assert_array_equal(d, ref)
    np.testing.assert_array_equal(a, arg)
    ctx.close()


@pytest.mark.parametrize("prims", [16, -4])
def test_alternating_sources_are_ordered(prims):
    """20480 poses against 8192 points of which every other one lies on a wall: as
    fast as a field of as many (7 times slower where a sample at regular places
    takes the wall for the whole set)."""
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(3)
    kind, geom = _footprint(rng, prims)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    poses = torch.tensor(_poses(rng, 20480, 1, 0.5), device="cuda")
    us = {}
    for name in ("field", "alternating"):
        ctx.set_points(*_set(rng, name, 8192))
        us[name] = _us(lambda: ctx.sdf_min_poses(poses, kind=kind))
    print(us)
    assert us["alternating"] < 3 * us["field"], us
    ctx.close()
