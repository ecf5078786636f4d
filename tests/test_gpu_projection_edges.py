"""Batches of more than 32 views decide most (Gaussian, view) pairs by a binary32 screen;
batches of at most 32 decide every candidate in binary64.  The pairs have to be
the same, bit for bit, whatever the screen cannot vouch for: splats smaller
than a pixel and needles, means on image borders and behind cameras, cameras
whose matrix is no rotation or whose field of view is extreme, maps far from
the origin, inputs that are not finite, and more views than are staged at once."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def _pairs(raster, ctx, dev, cams, s):
    f = raster.Frame(ctx, dev, cams, s)
    f.bin_sort()
    keys, vals, _ = f.export()
    keys, vals = keys.cpu().numpy().view(np.uint64).copy(), vals.cpu().numpy().view(np.uint32).copy()
    f.close()
    return keys, vals


def _cams(rng, nv, far):
    cams = []
    for v in range(nv):
        w, h = ((1, 9), (64, 1), (48, 32), (161, 119))[v % 4 if v % 5 == 0 else 2 + v % 2]
        f = max(w, h) * (rng.uniform(0.05, 0.2) if v % 11 == 3 else rng.uniform(0.6, 3.0))
        R = scenes.random_rotation(rng) * (1.02 if v % 13 == 5 else 1.0)
        cams.append(scenes.make_camera(w, h, f, f * (3.0 if v % 17 == 6 else 1.0), w * rng.uniform(-0.5, 1.5), h * rng.uniform(0, 1),
                                       R, far + rng.uniform(-3, 3, 3)))
    return cams


@pytest.mark.parametrize("n,nv,far,eps2d,iso", [(1, 33, 0.0, 0.0, False), (63, 64, 0.0, 0.3, False), (65, 65, 0.0, 0.0, True),
                                                (511, 255, 0.0, 0.0, False), (513, 257, 30.0, 0.0, False),
                                                (3000, 300, 0.0, 0.0, True), (3000, 100, 1000.0, 0.0, False),
                                                (20000, 70, 0.0, 0.0, False)])
def test_screened_pairs(n, nv, far, eps2d, iso):
    from paper_2409_18122_amd import raster
    print(f"screened pairs n={n} views={nv} far={far} eps2d={eps2d} iso={iso}", flush=True)
    rng = np.random.default_rng(n + nv)
    g = {k: v.copy() for k, v in scenes.subset(scenes.config1(n=max(n, 2), seed=5)[0], np.arange(n)).items()}
    g["means"] = (np.array([far, -far, 0.5 * far])[:, None] + rng.uniform(-4, 4, (3, n))).astype(np.float32)
    g["log_scales"] = rng.uniform(-7.0, 0.5, (3, n)).astype(np.float32)
    g["log_scales"][:, ::9] = -30.0
    g["log_scales"][0, ::7] = 3.0
    g["opacity"][::4] = np.float32(1 / 255) * np.float32(1.0000005)
    cams = _cams(rng, nv, np.array([far, -far, 0.5 * far]))
    if n > 60:
        # on the corners and half a pixel beyond the edges of view 2, and inputs that are not ordinary numbers
        c = cams[2]
        uv = [(0, 0), (c["width"] - 1, c["height"] - 1), (-0.5, 3), (c["width"] - 0.5, 3), (5, -0.5), (5, c["height"] - 0.5), (3, 3)]
        d = np.array([[(u - c["cx"]) / c["fx"], (v - c["cy"]) / c["fy"], 1.0] for u, v in uv]) * 2.0
        R, T = np.asarray(c["R"], np.float64).reshape(3, 3), np.asarray(c["T"], np.float64).reshape(3)
        g["means"][:, :len(uv)] = (R @ d.T + T[:, None]).astype(np.float32)
        g["means"][0, 20], g["log_scales"][1, 21], g["quats"][2, 22], g["opacity"][23] = np.nan, np.inf, -np.inf, np.nan
        g["quats"][:, 24], g["log_scales"][:, 25], g["means"][:, 26] = 0.0, 200.0, 3e38
    if iso:
        g = scenes.isotropic_scene(g)
    s = dict(scenes.DEFAULT_SETTINGS, eps2d=eps2d, isotropic=iso)
    ctx = raster.Context(0)
    dev = raster.to_device(g)
    keys, vals = _pairs(raster, ctx, dev, cams, s)
    kk, vv, tiles = [], [], 0
    for b in range(0, nv, 20):
        part = cams[b:b + 20]
        k, v = _pairs(raster, ctx, dev, part, s)
        kk.append(k + (np.uint64(tiles) << np.uint64(32)))
        vv.append(v)
        tiles += sum(-(-c["width"] // 16) * -(-c["height"] // 16) for c in part)
    kk, vv = np.concatenate(kk), np.concatenate(vv)
    assert len(keys) == len(kk) and np.array_equal(keys, kk) and np.array_equal(vals, vv)
    assert n < 60 or len(kk) > n
