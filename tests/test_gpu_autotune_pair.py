"""What mppi_autotune returns is what it keeps: the pair is the context's entry
for the shape, and gives the same plan through mppi_set_tiles and a saved table."""
import numpy as np
import pytest

from paper_2605_29663_amd import scenes

pytestmark = pytest.mark.gpu


# evaluated point by point; searched; searched in ranges
@pytest.mark.parametrize("n", [300, 5000, 70000])
def test_pair_is_the_entry(n):
    import torch
    import paper_2605_29663_amd as pkg
    rng = np.random.default_rng(n)
    ctx = pkg.Context(0)
    ctx.set_footprint(0, scenes.star_polygon(rng, 8).astype(np.float32))
    ctx.set_points(*rng.uniform(-6, 6, (2, n)).astype(np.float32))
    prm = scenes.params("c1", K=256, T=20, validate=0)
    kept = f"0 8 0 20 {n} 128 1"  # an entry of the validation shape, which is not tuned here
    ctx.mppi_tune_set(kept + "\n")

    def step():
        U = torch.zeros((20, 2), device="cuda")
        ctx.mppi_step(prm, np.zeros(3, np.float32), U, 3, 0)
        return U

    U = step()
    blk, nc = ctx.mppi_autotune(prm, reps=1)
    lines = ctx.mppi_tune_get().split("\n")
    assert blk in (64, 128, 256) and nc >= 1
    assert kept in lines
    assert f"0 8 0 {256 * 20} {n} {blk} {nc}" in lines, lines
    assert torch.equal(step(), U)
    ctx.mppi_set_tiles(blk, nc)
    assert torch.equal(step(), U)
    ctx.close()
