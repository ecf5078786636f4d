"""The compositing kernels at their edges: bands of one, two and four per tile with
and without alpha gradients, tiles that the frame cuts, splats more opaque than
alpha_max, long needles and other alpha thresholds (the width of the
binary64 re-decision follows the splat), and uncertainties that are not finite.
Bars are those of gpu_util; a sum that an infinite or NaN uncertainty
reaches is infinite or NaN, and no other is."""
import numpy as np
import pytest
import torch

import oracle
import scenes
from gpu_util import (GRAD_REL_TOL, SCORE_TOL_PER_PIXEL, assert_elementwise, assert_images_close, gpu_stack,
                      grad_rel_errors, grads_to_numpy)

pytestmark = pytest.mark.gpu


def _settings(tile, amin):
    return dict(scenes.DEFAULT_SETTINGS, tile_w=tile[0], tile_h=tile[1], alpha_min=amin)


def _scene(n, seed, w, h):
    g, cams = scenes.tiny_scene(n, seed, w, h)
    rng = np.random.default_rng(seed)
    g = {k: v.copy() for k, v in g.items()}
    g["opacity"][::3] = rng.uniform(0.992, 1.0, len(g["opacity"][::3])).astype(np.float32)  # above alpha_max
    ls = g["log_scales"]
    ls[:, 1::7] = np.array([[-0.5], [-4.5], [-4.5]], np.float32)  # needles over a good part of the frame
    return g, cams


# on 256 CUs: 2 bands below 4,096 tiles (isotropic maps: 4 below 896), then 1; 8x8 tiles have one band
@pytest.mark.parametrize("au", [False, True])
@pytest.mark.parametrize("iso,tile,w,h,views,n,amin", [(0, (16, 16), 33, 17, 1, 60, 1 / 255), (0, (16, 16), 567, 441, 1, 400, 0.02),
                                                       (0, (32, 8), 289, 130, 2, 300, 1 / 255), (0, (32, 8), 573, 433, 1, 400, 1e-4),
                                                       (0, (16, 16), 477, 381, 6, 400, 1 / 255), (0, (32, 8), 477, 381, 6, 400, 0.02),
                                                       (0, (8, 8), 61, 47, 2, 200, 0.1), (1, (16, 16), 33, 17, 1, 60, 1 / 255),
                                                       (1, (32, 8), 289, 130, 2, 300, 0.02), (1, (16, 16), 567, 441, 1, 400, 1 / 255)])
def test_backward_bands(au, iso, tile, w, h, views, n, amin):
    from paper_2409_18122_amd import raster
    print(f"bands au={au} iso={iso} tile={tile} {w}x{h} views={views} n={n} alpha_min={amin:.4g}", flush=True)
    g, cams = _scene(n, n + w, w, h)
    if iso:
        g = scenes.isotropic_scene(g)
    cams = [scenes.make_camera(w, h, cams[0]["fx"], cams[0]["fy"], cams[0]["cx"] + 3.0 * v, cams[0]["cy"] - 2.0 * v)
            for v in range(views)]
    s = dict(_settings(tile, amin), isotropic=iso)
    f = raster.Frame(raster.Context(0), raster.to_device(g), cams, s)
    f.bin_sort()
    imgs = raster.unpack_images(f.render(), cams)
    rng = np.random.default_rng(3)
    ref = {k: np.zeros((rows, n)) for k, rows in (("means", 3), ("log_scales", 3), ("quats", 4), ("colors", 3))}
    ref["opacity"] = np.zeros(n)
    touched = np.zeros(n, bool)
    planes = [[], [], [], []]
    pairs = slack = 0
    for v, c in enumerate(cams):
        r = oracle.render(g, c, s)
        assert_images_close(gpu_stack(imgs[v], c), r, label=f"view {v}")
        pairs += int(r["ncontrib"].sum())
        slack += n * int((r["nevents"] > 0).sum())  # a decision may end or prolong a pixel's walk
        gs = [rng.standard_normal(sh).astype(np.float32) for sh in ((3, h, w), (h, w), (h, w), (h, w))]
        a = oracle.adjoint(g, c, s, g_rgb=gs[0], g_depth=gs[1], g_alpha=gs[2] if au else None,
                           g_unc=gs[3] if au else None, tile=tile)
        for k in ref:
            ref[k] += a[k]
        touched |= a["touched"]
        for p, x in zip(planes, gs):
            p.append(x.reshape(-1))
    assert abs(f.stats()["contrib_pairs"] - pairs) <= slack
    p = [torch.as_tensor(np.concatenate(x)).cuda() for x in planes]
    got = grads_to_numpy(f.backward(p[0], p[1], p[2] if au else None, p[3] if au else None))
    if iso:  # one log-radius (the oracle leaves its gradient in the first row), no quaternion
        assert "quats" not in got
        ref["log_scales"], ref["quats"], got["quats"] = ref["log_scales"][:1], np.zeros((4, n)), np.zeros((4, n))
        got["log_scales"] = got["log_scales"].reshape(1, n)
    ok = {k: np.where(touched, 0.0, x) for k, x in got.items()}
    rel = grad_rel_errors(ok, {k: np.where(touched, 0.0, x) for k, x in ref.items()})
    assert all(e <= GRAD_REL_TOL for e in rel.values()), rel
    assert assert_elementwise(got, ref, touched) < n


@pytest.mark.parametrize("mode", ["rendered", "binary"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
def test_scores_of_unfinite_uncertainty(tile, mode):
    from paper_2409_18122_amd import raster
    s = _settings(tile, 1 / 255)
    m = ("rendered", "binary").index(mode)
    g, cams = _scene(150, 9, 70, 50)
    c = cams[0]
    # cameras that look ahead, and one that looks back and sees nothing; one Gaussian lies before the first camera
    # alone (nearest, so every set of decisions has it), the others behind it or off its frame
    back = scenes.make_camera(33, 9, c["fx"], c["fy"], 16.0, 4.0, R=np.diag([-1.0, 1.0, -1.0]))
    aside = scenes.make_camera(41, 50, c["fx"], c["fy"], c["cx"] - 35.0, c["cy"])
    views = [c, aside, back]
    g["means"][:, 0] = (-0.3, 0.0, 1.0)
    g["log_scales"][:, 0] = -4.0
    g["opacity"][0] = 0.5
    dev = raster.Context(0)
    for bad in (None, np.inf, -np.inf, np.nan):
        if bad is not None:
            g["uncert"][0] = bad
        print(f"scores tile={tile} mode={mode} u={bad}", flush=True)
        got = raster.score_views(dev, raster.to_device(g), views, s, mode=mode).cpu().numpy()
        ref = oracle.score(g, views, s, tile=tile, mode=m)
        if bad is not None:
            assert not np.isfinite(ref[0]) and np.isfinite(ref[1])
        for v, r in enumerate(ref):
            if np.isfinite(r):
                assert abs(got[v] - r) <= SCORE_TOL_PER_PIXEL * views[v]["width"] * views[v]["height"]
            else:
                assert np.array_equal(got[v], r, equal_nan=True)
