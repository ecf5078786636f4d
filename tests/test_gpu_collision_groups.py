"""The collision check's grouping of points at its edges: group (64 points), batch
(4,096), slab (44 groups) and launch (2^20 points) remainders, points in no
order, non-finite points, one Gaussian, and the flags without clearances.
Flags: the oracle's, bit for bit outside a 1e-12 relative tie band.  Clearance:
binary32 evaluation of sqrt(d^2) - w from exact inputs, |error| <= 2e-6 (1 +
|clearance| + 2 max w) (three roundings of d^2 and one each of the root, w and
the difference stay below 5e-7 of dist + w)."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_collision import check, tie_bands, w_max

pytestmark = pytest.mark.gpu


def run(means, ls, pts, clearance=True, no_alloc=False):
    from paper_2409_18122_amd import raster
    ctx = raster.Context(0)
    g = {"means": torch.as_tensor(means).cuda(), "log_scales": torch.as_tensor(ls).cuda()}
    hit, clr = raster.collision_check(ctx, g, torch.as_tensor(pts).cuda(), 0.25, 3.0, clearance=clearance,
                                      no_alloc=no_alloc)
    torch.cuda.synchronize()
    ctx.close()
    return hit.cpu().numpy(), None if clr is None else clr.cpu().numpy()


@pytest.mark.parametrize("n,p", [(1, 1), (63, 64), (64, 65), (1025, 63), (777, 4096), (3000, 4097), (2000, 2816),
                                 (2000, 2817), (200_000, 300), (5, (1 << 20) + 5)])
def test_groups(n, p):
    print(f"collision groups n={n} p={p}", flush=True)
    rng = np.random.default_rng(n + p)
    size = 4.0 * max(n, 64) ** (1 / 3)
    means = rng.uniform(-size, size, (3, n)).astype(np.float32)
    ls = rng.normal(-2.5, 0.6, (3, n)).astype(np.float32)
    # half near Gaussians, half anywhere, in no order
    near = means[:, rng.integers(0, n, p)] + rng.uniform(-0.6, 0.6, (3, p))
    pts = np.where(rng.random(p) < 0.5, near, rng.uniform(-2 * size, 2 * size, (3, p))).astype(np.float32)
    if p > 200:
        pts[0, 7], pts[1, 70], pts[2, 130] = np.nan, np.inf, -np.inf
    fin = np.isfinite(pts).all(0)
    hit, clr = run(means, ls, pts)
    ref_hit, ref_clr = oracle.collision(means, ls, np.ascontiguousarray(pts[:, fin]), 0.25, 3.0)
    sure, maybe = tie_bands(means, ls, pts[:, fin], 0.25, 3.0)
    check(hit[fin], clr[fin], ref_hit, ref_clr, sure, maybe, w_max(ls, 3.0))
    # a point that is nowhere meets nothing
    assert not hit[~fin].any() and np.all(np.isinf(clr[~fin]))
    hit2, none = run(means, ls, pts, clearance=False, no_alloc=True)
    assert none is None and np.array_equal(hit, hit2)
