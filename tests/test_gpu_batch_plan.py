"""The batch's autotuner and its default plan: tuning never leaves a batch with a
slower plan than the default one, whatever the scenes' sizes."""
import time

import numpy as np
import pytest

from paper_2605_29663_amd import scenes

pytestmark = pytest.mark.gpu


def _step_us(b, U, n):
    q0, ids = np.zeros((n, 3), np.float32), np.arange(n, dtype=np.uint64)
    best = np.inf
    for _ in range(8):
        U.zero_()
        t = time.perf_counter()
        b.mppi_step_batched(q0, U, ids, ids, use_graph=True)
        best = min(best, 1e6 * (time.perf_counter() - t))
    return best


def test_tuned_plan_no_slower_than_default():
    """One scene of 300000 sparse points and 64 edges: no target in pairs that the tuner
    tries (2^26 at most) gives an item more than 8 poses, the default gives 128."""
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(5)
    ctx = pkg.Context(0)
    ctx.set_footprint(0, scenes.star_polygon(rng, 64).astype(np.float32))
    ctx.set_points(*rng.uniform(-200, 200, (2, 300000)).astype(np.float32))
    b = pkg.Batch([ctx], [scenes.params("c1", K=4096, T=60)])
    U = b.new_nominals()
    default, items = _step_us(b, U, 1), b.mppi_batch_info()[0]
    U0 = U.clone()
    work = b.mppi_batch_autotune(reps=2)
    tuned = _step_us(b, U, 1)
    print(default, tuned, items, b.mppi_batch_info())
    assert torch.equal(U, U0)
    assert b.mppi_batch_info()[2] == work
    assert tuned < 1.25 * default
    b.close()
    ctx.close()
