"""The horizon that moving sets are sorted for is not spoiled by a call whose time
step is no number (mppi_rollout takes any)."""
import numpy as np
import pytest

from paper_2605_29663_amd import scenes
from test_gpu_search import _footprint, _poses
from test_gpu_search_scaled import _us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [float("nan"), float("inf"), -float("inf")])
def test_rollout_without_a_time_step(dt):
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(2)
    kind, geom = _footprint(rng, 8)
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    pts = [a.astype(np.float32) for a in rng.uniform(-8, 8, (2, 8192))]
    vel = [a.astype(np.float32) for a in rng.uniform(-1, 1, (2, 8192)) * (rng.random(8192) < 0.3)]
    poses = torch.tensor(_poses(rng, 20480, 1, 0.5), device="cuda")
    out, us = [], []
    for _ in range(2):
        ctx.set_points(*pts, *vel)
        out.append(ctx.sdf_min_poses(poses, dt=0.1, state_offset=1))
        us.append(_us(lambda: ctx.sdf_min_poses(poses, dt=0.1, state_offset=1)))
        ctx.mppi_rollout(scenes.params("c1", K=64, T=20, dt=dt), np.zeros(3, np.float32),
                         torch.zeros((20, 2), device="cuda"), 1, 0)
    print(us)
    assert torch.equal(out[0], out[1])
    assert us[1] < 2.5 * us[0], us
    ctx.close()
