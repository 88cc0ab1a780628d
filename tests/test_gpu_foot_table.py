"""The footprint's bound table at its hard places (corners, medial axes, thin and
curved outlines, boxes that meet): a wrong bound drops the nearest point, so
the search must give the oracle's minimum, and the bits of a point by point
evaluation, for polygons with sharp, blunt and reflex corners, thin ones, boxes
that overlap, touch and lie apart, and points from inside to far outside."""
import numpy as np
import pytest

from paper_2605_29663_amd import scenes

pytestmark = pytest.mark.gpu
TOL_D = 1e-5  # the distance contract (metres)

THIN = np.float32([[-2, -0.01], [2, -0.01], [2, 0.01], [-2, 0.01]])
NEEDLE = np.float32([[0, -0.2], [3, 0], [0, 0.2]])
COMB = np.float32([[0, 0], [3, 0], [3, 1], [2.5, 1], [2.5, 0.2], [1.75, 0.2], [1.75, 1], [1.25, 1], [1.25, 0.2],
                   [0.5, 0.2], [0.5, 1], [0, 1]])
TURN = np.float32([[0.2 * np.cos(a), 0.2 * np.sin(a)] for a in np.arange(48) * (2 * np.pi / 48)])
CROSS = np.float32([[0, 0, 1.0, 0.1], [0, 0, 0.1, 1.0]])
APART = np.float32([[-1, 0, 0.3, 0.2], [1, 0.1, 0.2, 0.4], [0.2, 1.0, 0.05, 0.05]])
TOUCH = np.float32([[0, 0, 0.5, 0.5], [1.0, 0, 0.5, 0.25], [1.0, 0.5, 0.5, 0.25]])


@pytest.mark.parametrize("kind,geom", [(0, THIN), (0, NEEDLE), (0, COMB), (0, TURN), (0, scenes.FOOTPRINT_TOWED16),
                                       (0, scenes.FOOTPRINT_L8), (1, CROSS), (1, APART), (1, TOUCH)])
@pytest.mark.parametrize("spread", [0.3, 1.0, 4.0])
def test_bounds_decide_the_exact_minimum(kind, geom, spread):
    import torch
    import paper_2605_29663_amd as pkg
    from oracle import oracle as orc
    geom = np.asarray(geom, np.float32)
    rng = np.random.default_rng(len(geom) + int(10 * spread))
    ctx = pkg.Context(0)
    ctx.set_footprint(kind, geom)
    K, T = 61, 4
    # points away from a disc of the poses' spread, so that the minima are of
    # either sign, and a grid of equal distances along the axes
    n = 1500
    r = rng.uniform(0.0, 2.5 * spread, n)
    a = rng.uniform(0, 2 * np.pi, n)
    x, y = (r * np.cos(a)).astype(np.float32), (r * np.sin(a)).astype(np.float32)
    x[:200], y[:200] = np.linspace(-3, 3, 200), spread
    far = rng.random(n) < 0.5
    x[far] += np.float32(2.0)
    ctx.set_points(x, y)
    th = rng.uniform(-3.2, 3.2, (K, T))
    th[:20] = np.round(th[:20] / (np.pi / 2)) * (np.pi / 2)
    p = np.stack([rng.normal(0, spread, (K, T)), rng.normal(0, spread, (K, T)), np.cos(th), np.sin(th)], -1)
    p = p.astype(np.float32)
    d, arg = ctx.sdf_min_poses(torch.tensor(p, device="cuda"), kind=kind, argmin=True)
    flat = p.reshape(-1, 4)
    ref = orc.dmin(flat, np.zeros(len(flat), np.float32), x, y, None, None, None, kind, geom)
    np.testing.assert_allclose(d.cpu().numpy().ravel(), ref, atol=TOL_D)
    # and the same bits as over pieces that are evaluated point by point
    best = np.full((K, T), np.inf, np.float32)
    for i in range(0, n, 60):
        ctx.set_points(x[i:i + 60], y[i:i + 60])
        best = np.minimum(best, ctx.sdf_min_poses(torch.tensor(p, device="cuda"), kind=kind).cpu().numpy())
    np.testing.assert_array_equal(d.cpu().numpy(), best)
