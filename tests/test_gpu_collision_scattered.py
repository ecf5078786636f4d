"""The collision check where the grouping of points cannot help: small maps (all pairs in one launch) and points scattered
wider than the map.  Flags and clearances are the oracle's, with the tolerances of the other collision tests, around the sizes
where the form changes; and the time stays within that of a loop over all pairs, 100 us and 2.5e12 pairs a second (such a
loop makes 3.3e12; the grouping alone took two to ten times as long)."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_collision import check, tie_bands, w_max
from test_gpu_collision_enclosed import _best_us
from test_gpu_collision_groups import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(0, 65), (1, 1), (3, 64), (5, 65), (4, 32_767), (7, 32_768), (9, 262_143), (2, 262_145),
                                 (63, 1025), (1023, 1000), (1024, 4097), (1025, 300), (2048, 131), (2049, 8000),
                                 (8192, 500), (8193, 500), (8192, 16_383), (8192, 16_385), (2047, 66_000), (2049, 133_000),
                                 (12_288, 8192), (12_289, 8192), (40_000, 6000)])
def test_all_pairs(n, p):
    print(f"collision all pairs n={n} p={p}", flush=True)
    rng = np.random.default_rng(n + p)
    size = 4.0 * max(n, 64) ** (1 / 3)
    means = rng.uniform(-size, size, (3, n)).astype(np.float32)
    ls = rng.normal(-2.5, 0.6, (3, n)).astype(np.float32)
    if n > 20:
        means[0, 5], ls[1, 6], ls[2, 7] = np.nan, np.inf, -np.inf
    pts = rng.uniform(-1.5 * size, 1.5 * size, (3, p)).astype(np.float32)
    if n:
        near = means[:, rng.integers(8, n, p) if n > 20 else rng.integers(0, n, p)] + rng.uniform(-0.6, 0.6, (3, p))
        pts = np.where(rng.random(p) < 0.4, near, pts).astype(np.float32)
    if p > 200:
        pts[0, 7], pts[1, 70], pts[2, 130] = np.nan, np.inf, -np.inf
    fin = np.isfinite(pts).all(0)
    hit, clr = run(means, ls, pts)
    hit2, none = run(means, ls, pts, clearance=False, no_alloc=True)
    assert none is None and np.array_equal(hit, hit2)
    assert not hit[~fin].any() and np.all(np.isinf(clr[~fin]))
    some = np.flatnonzero(fin)
    if n * p > 50_000_000:
        some = rng.choice(some, 50_000_000 // n, replace=False)
    sub = np.ascontiguousarray(pts[:, some])
    ref_hit, ref_clr = oracle.collision(means, ls, sub, 0.25, 3.0)
    sure, maybe = tie_bands(means, ls, sub, 0.25, 3.0) if n else (None, None)
    check(hit[some], clr[some], ref_hit, ref_clr, sure, maybe, w_max(ls, 3.0))


@pytest.mark.parametrize("n,p", [(1, 1 << 20), (100, 1000), (100, 100_000), (2000, 30_000), (8000, 8192), (30_000, 4096),
                                 (100_000, 8256), (3_000_000, 8256)])
def test_scattered_points_cost_no_more_than_all_pairs(n, p):
    from paper_2409_18122_amd import raster
    rng = np.random.default_rng(n)
    m = np.stack([rng.uniform(-20, 20, n), rng.uniform(-20, 20, n), rng.uniform(0, 2, n)]).astype(np.float32)
    g = {"means": torch.as_tensor(m).cuda(), "log_scales": torch.as_tensor(rng.normal(-3.5, 0.3, (3, n)).astype(np.float32)).cuda()}
    x = torch.as_tensor(rng.uniform(-200, 200, (3, p)).astype(np.float32)).cuda()
    ctx = raster.Context(0)
    us = _best_us(lambda: raster.collision_check(ctx, g, x, 0.25, 3.0))
    print(f"collision scattered n={n} p={p}: {us:.0f} us", flush=True)
    assert us < 100.0 + n * p / 2.5e6
    ctx.close()


@pytest.mark.parametrize("n,p,spread", [(9000, 3000, 300.0), (20_000, 2817, 300.0), (100_000, 500, 1000.0), (70_000, 700, 60.0)])
def test_scattered_points(n, p, spread):
    """Blocks whose balls sort nothing out, and such ones beside others."""
    print(f"collision scattered parity n={n} p={p}", flush=True)
    rng = np.random.default_rng(n + p)
    means = rng.uniform(-20, 20, (3, n)).astype(np.float32)
    ls = rng.normal(-2.5, 0.6, (3, n)).astype(np.float32)
    means[0, 5], ls[1, 6], ls[2, 7] = np.nan, np.inf, -np.inf
    pts = rng.uniform(-spread, spread, (3, p)).astype(np.float32)
    pts[:, :p // 3] = means[:, 10:10 + p // 3] + rng.uniform(-0.6, 0.6, (3, p // 3)).astype(np.float32)
    pts[0, 7], pts[1, 70], pts[2, 130] = np.nan, np.inf, -np.inf
    fin = np.isfinite(pts).all(0)
    hit, clr = run(means, ls, pts)
    hit2, _ = run(means, ls, pts, clearance=False, no_alloc=True)
    assert np.array_equal(hit, hit2) and not hit[~fin].any() and np.all(np.isinf(clr[~fin]))
    sub = np.ascontiguousarray(pts[:, fin])
    ref_hit, ref_clr = oracle.collision(means, ls, sub, 0.25, 3.0)
    sure, maybe = tie_bands(means, ls, sub, 0.25, 3.0)
    check(hit[fin], clr[fin], ref_hit, ref_clr, sure, maybe, w_max(ls, 3.0))
