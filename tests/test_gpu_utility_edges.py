"""The matrix-core screen of the view utility, the moments and the trajectory choice
at their edges: remainders of a product's four views and 16 Gaussians, of a block's 32
views and a wave's 64 Gaussians, maps far from the origin, long ranges, images one pixel
wide, means beyond the screen's range, and ties among trajectories.  Counts are
integers decided as the oracle decides them: equal.  Sums are in 2^-40 fixed
point: each term is cut by less than 2^-40."""
import numpy as np
import pytest
import torch

import oracle
import scenes

pytestmark = pytest.mark.gpu

S = dict(scenes.DEFAULT_SETTINGS)


def _views(rng, nv, centre, scale):
    cams = []
    for v in range(nv):
        w, h = ((1, 9), (64, 1), (160, 120), (641, 479))[v % 4 if v % 7 == 0 else 2 + v % 2]
        f = max(w, h) * rng.uniform(0.4, 30.0 if v % 5 == 0 else 1.5)
        cams.append(scenes.make_camera(w, h, f, f, w * rng.uniform(0.2, 0.8), h * rng.uniform(0.2, 0.8),
                                       scenes.random_rotation(rng), centre + scale * rng.uniform(-1, 1, 3)))
    return cams


@pytest.mark.parametrize("n,nv,far,range_", [(1, 1, 0.0, 5.0), (63, 4, 0.0, 5.0), (64, 5, 30.0, 2.0), (257, 31, 0.0, 1e9),
                                             (4097, 32, 1000.0, 5.0), (5000, 33, 0.0, 0.3), (20000, 65, 3e4, 50.0)])
def test_counts(n, nv, far, range_):
    from paper_2409_18122_amd import raster
    print(f"utility n={n} nv={nv} far={far} range={range_}", flush=True)
    rng = np.random.default_rng(n + nv)
    g = scenes.subset(scenes.config1(n=max(n, 2), seed=3)[0], np.arange(n))
    centre = np.array([far, -far, 0.5 * far])
    g["means"] = (centre[:, None] + rng.uniform(-4, 4, (3, n))).astype(np.float32)
    cams = _views(rng, nv, centre, 3.0)
    if n > 200:  # on image borders and depth limits of the third view, and means that are not ordinary numbers
        c = cams[2]
        z = np.float32(min(range_, 4.0))
        d = np.array([[(-c["cx"]) / c["fx"] * z, 0.0, z], [(c["width"] - 1 - c["cx"]) / c["fx"] * z, 0.0, z], [0.0, 0.0, S["z_near"]],
                      [0.0, 0.0, min(range_, 1e6)]])
        g["means"][:, 10:14] = (np.asarray(c["R"], np.float64) @ d.T + np.asarray(c["T"], np.float64)[:, None]).astype(np.float32)
        g["means"][0, 0], g["means"][1, 1], g["means"][2, 2] = np.nan, np.inf, 1e20
        g["uncert"][5], g["uncert"][6], g["uncert"][7] = np.nan, np.inf, -1.0
    lo, hi = 0.3, 0.6
    dev = raster.to_device(g)
    got = raster.view_utility(raster.Context(0), dev, cams, torch.tensor([lo, hi], dtype=torch.float64, device="cuda"),
                              S, range_=range_)
    fin = np.isfinite(g["uncert"]) & (g["uncert"] > 0)
    nh, nl, _, xi = oracle.view_utility(g, cams, S, lo, hi, range_=range_)
    assert np.array_equal(got["n_high"].cpu().numpy(), nh) and np.array_equal(got["n_low"].cpu().numpy(), nl)
    assert np.array_equal(got["xi"].cpu().numpy(), xi)
    _, _, su, _ = oracle.view_utility(dict(g, uncert=np.where(fin, g["uncert"], 0).astype(np.float32)), cams, S, lo, hi,
                                      range_=range_)
    assert np.all(np.abs(got["sum_u"].cpu().numpy() - su) <= n * 2.0 ** -40 + 1e-12 * np.abs(su))


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 131_073])
def test_thresholds(n):
    from paper_2409_18122_amd import raster
    u = np.random.default_rng(n).random(n).astype(np.float32)
    th = raster.uncertainty_thresholds(raster.Context(0), torch.as_tensor(u).cuda(), 0.5).cpu().numpy()
    assert np.allclose(th, oracle.thresholds(u, 0.5), rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 600])
def test_trajectories(n):
    from paper_2409_18122_amd import raster
    rng = np.random.default_rng(n)
    ctx = raster.Context(0)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 5, n))]).astype(np.int32)
    xi = rng.integers(-3, 4, max(int(off[-1]), 1)).astype(np.float64)  # many ties
    util, best = raster.trajectory_select(ctx, torch.as_tensor(xi).cuda(), torch.as_tensor(off).cuda())
    ref, rb = oracle.traj_select(xi, off)
    assert np.array_equal(util.cpu().numpy(), ref) and int(best) == rb
    if off[1] > 0:  # nothing is greater than a NaN
        xi[0] = np.nan
        assert int(raster.trajectory_select(ctx, torch.as_tensor(xi).cuda(), torch.as_tensor(off).cuda())[1]) == 0
