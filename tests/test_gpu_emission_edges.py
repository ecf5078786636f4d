"""Pair counting and emission at their edges: one record of thousands of pairs (most
waves start inside it), rows wider than a window of 128 pairs, more than 64 rows
of a wave's records, supports that leave rows of their boxes empty, boxes of
a single tile, batches of 63 to 65 records, and several views.  The pairs are those
of the oracle's boxes, in its order, and hold every pair of its supports."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("n,kind,w,h", [(1, "huge", 1999, 701), (1, "needle", 1501, 1203), (63, "mixed", 333, 251),
                                        (64, "tiny", 641, 479), (65, "huge", 130, 1100), (700, "mixed", 1027, 389),
                                        (3000, "tiny", 97, 1025)])
def test_pairs(tile, n, kind, w, h):
    from paper_2409_18122_amd import raster
    print(f"emission tile={tile} n={n} {kind} {w}x{h}", flush=True)
    rng = np.random.default_rng(n)
    g, cams = scenes.tiny_scene(n, n, w, h)
    c = cams[0]
    cams = [c, scenes.make_camera(h, w, c["fx"], c["fy"], h / 2.0, w / 2.0)]
    g = {k: v.copy() for k, v in g.items()}
    ls = g["log_scales"]
    if kind in ("huge", "mixed"):
        ls[:, ::5] = rng.uniform(-0.5, 1.0, ls[:, ::5].shape)
    if kind in ("needle", "mixed"):
        ls[:, ::3] = np.array([[0.0], [-5.0], [-5.0]], np.float32)
    if kind == "tiny":
        ls[:] = rng.uniform(-7.5, -4.0, ls.shape)
    s = dict(scenes.DEFAULT_SETTINGS, tile_w=tile[0], tile_h=tile[1])
    f = raster.Frame(raster.Context(0), raster.to_device(g), cams, s)
    f.bin_sort()
    keys, vals, _ = f.export()
    ids = lambda k, v: (k >> np.uint64(32)) << np.uint64(32) | v.astype(np.uint64)
    keys, vals = keys.cpu().numpy().view(np.uint64), vals.cpu().numpy().view(np.uint32)
    k_box, v_box = oracle.keys(g, cams, s, tile)
    k_sup, v_sup = oracle.keys(g, cams, s, tile, support=True)
    got = ids(keys, vals)
    keep = np.isin(ids(k_box, v_box), got)
    print(f"box {len(k_box)} support {len(k_sup)} here {len(keys)}", flush=True)
    assert keep.sum() == len(got) and len(np.unique(got)) == len(got)
    assert np.array_equal(keys, k_box[keep]) and np.array_equal(vals, v_box[keep])
    assert np.isin(ids(k_sup, v_sup), got).all()
    # every record owns a pair, and the margins of the support add few
    assert len(keys) <= len(k_sup) + len(np.unique(v_box)) * 2 + max(8, len(k_sup) // 20)
