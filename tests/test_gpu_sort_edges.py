"""The depth and tile sorts at the sizes where their form changes: a tile of items and one
more or less, the limits of 4, 8 and 16 items per lane, and of offsets that the
blocks form themselves; records of more pairs than fit the spare bits that carry the
counts through the depth sort.  The sorted pairs are the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


# about one record per Gaussian, and one pair per record but for the big ones
@pytest.mark.parametrize("n", [1, 255, 1023, 1025, 4096, 4097, 16_384, 16_385, 32_700, 32_900, 262_100, 262_300, 1_048_500, 1_048_700, 2_097_300])
def test_sorted_pairs(n):
    from paper_2409_18122_amd import raster
    print(f"sort n={n}", flush=True)
    rng = np.random.default_rng(n)
    w, h = 640, 480
    c = scenes.make_camera(w, h, 500.0, 500.0, 319.5, 239.5)
    z = rng.choice(np.linspace(1.0, 3.0, 1 + n // 3), n)  # equal depths: the sort is stable
    u, v = rng.uniform(0, w - 1, n), rng.uniform(0, h - 1, n)
    means = np.stack([(u - 319.5) / 500.0 * z, (v - 239.5) / 500.0 * z, z]).astype(np.float32)
    ls = np.full((3, n), -6.5, np.float32)
    big = rng.permutation(n)[:max(1, min(n // 50, 40))]
    ls[:, big] = rng.uniform(-3.0, -0.5, len(big)).astype(np.float32)
    q = np.zeros((4, n), np.float32)
    q[0] = 1.0
    g = {"means": means, "log_scales": ls, "quats": q, "opacity": np.full(n, 0.8, np.float32),
         "colors": rng.random((3, n)).astype(np.float32), "uncert": rng.random(n).astype(np.float32)}
    s = dict(scenes.DEFAULT_SETTINGS)
    f = raster.Frame(raster.Context(0), raster.to_device(g), [c], s)
    f.bin_sort()
    keys, vals, _ = f.export()
    keys, vals = keys.cpu().numpy().view(np.uint64), vals.cpu().numpy().view(np.uint32)
    k_box, v_box = oracle.keys(g, [c], s, (16, 16))
    ids = lambda k, v: (k >> np.uint64(32)) << np.uint64(32) | v.astype(np.uint64)
    keep = np.isin(ids(k_box, v_box), ids(keys, vals))
    assert keep.sum() == len(keys) >= len(np.unique(v_box))
    assert np.array_equal(keys, k_box[keep]) and np.array_equal(vals, v_box[keep])


@pytest.mark.parametrize("n", [3, 2047, 2049, 16_386, 70_001])
def test_scanned_offsets(n):
    """Records of sparse visibility: the scan's ragged ends and long runs of zero counts."""
    from paper_2409_18122_amd import raster
    print(f"scan n={n}", flush=True)
    rng = np.random.default_rng(n)
    g = {k: v.copy() for k, v in scenes.config1(n=n, seed=2)[0].items()}
    cams = scenes.config1(n=2)[1] * 3
    g["means"][2, rng.random(n) < 0.7] *= -1.0
    f = raster.Frame(raster.Context(0), raster.to_device(g), cams, dict(scenes.DEFAULT_SETTINGS))
    f.bin_sort()
    keys, vals, _ = f.export()
    keys, vals = keys.cpu().numpy().view(np.uint64), vals.cpu().numpy().view(np.uint32)
    k_box, v_box = oracle.keys(g, cams, dict(scenes.DEFAULT_SETTINGS), (16, 16))
    ids = lambda k, v: (k >> np.uint64(32)) << np.uint64(32) | v.astype(np.uint64)
    keep = np.isin(ids(k_box, v_box), ids(keys, vals))
    assert keep.sum() == len(keys)
    assert np.array_equal(keys, k_box[keep]) and np.array_equal(vals, v_box[keep])
