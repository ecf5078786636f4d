"""Cameras whose matrix is no rotation (any finite one is taken): columns of length 0.02 to 1,000 and
Gaussians whose depth lies a few roundings around the near plane.  The binary32 screens may not settle
such pairs: the records are the binary64 oracle's."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


def scaled_scene(scale, nv, n=1500):
    rng = np.random.default_rng(int(scale * 100))
    near = np.float32(scenes.DEFAULT_SETTINGS["z_near"])
    cams, means = [], []
    for _ in range(nv):
        R = (scale * scenes.random_rotation(rng)).astype(np.float32)
        T = rng.uniform(-2, 2, 3).astype(np.float32)
        cams.append(scenes.make_camera(48, 32, 40.0, 40.0, 24.0, 16.0, R, T))
        # depth R[:, 2] . (mean - T) = near up to the binary32 rounding of the mean
        k = n // nv + 1
        d = np.concatenate([rng.uniform(-8, 8, (2, k)) / scale, np.full((1, k), near / scale ** 2)])
        means.append(R.astype(np.float64) @ d + T[:, None].astype(np.float64))
    g = {k: v.copy() for k, v in scenes.subset(scenes.config1(n=n, seed=5)[0], np.arange(n)).items()}
    g["means"] = np.concatenate(means, 1)[:, :n].astype(np.float32)
    g["log_scales"] = rng.uniform(2.5, 3.5, (3, n)).astype(np.float32)  # supports that cover the image
    return g, cams


def check_records(g, cams, iso):
    from paper_2409_18122_amd import raster
    if iso:
        g = scenes.isotropic_scene(g)
    s = dict(scenes.DEFAULT_SETTINGS, isotropic=iso)
    ctx = raster.Context(0)
    f = raster.Frame(ctx, raster.to_device(g), cams, s)
    e = f.export_records()
    got = set(zip(e["view"].cpu().tolist(), e["gid"].cpu().tolist()))
    f.close()
    ref = {(v, int(i)) for v, c in enumerate(cams) for i in np.flatnonzero(oracle.project(g, c, s)["valid"])}
    assert ref and got == ref, (len(got - ref), len(ref - got))
    ctx.close()


@pytest.mark.parametrize("scale", [0.02, 1.0, 10.0, 100.0, 1000.0])
@pytest.mark.parametrize("views,iso", [(40, False), (40, True), (20, False), (20, True)])
def test_scaled_cameras_at_the_near_plane(views, iso, scale):
    print(f"scaled cameras views={views} scale={scale} iso={iso}", flush=True)
    check_records(*scaled_scene(scale, views), iso)


@pytest.mark.parametrize("views,iso", [(40, False), (40, True), (20, False), (20, True)])
def test_sheared_cameras(views, iso):
    print(f"sheared cameras views={views} iso={iso}", flush=True)
    rng = np.random.default_rng(views)
    n = 3000
    g = {k: v.copy() for k, v in scenes.subset(scenes.config1(n=n, seed=5)[0], np.arange(n)).items()}
    g["means"] = rng.uniform(-4, 4, (3, n)).astype(np.float32)
    g["log_scales"] = rng.uniform(-6.0, 0.5, (3, n)).astype(np.float32)
    cams = []
    for v in range(views):
        R = scenes.random_rotation(rng) @ np.diag(rng.uniform(0.3, 3.0, 3)) @ scenes.random_rotation(rng)
        if v % 5 == 0:  # a plane or a line: no lower bound of a support
            R[:, v % 3] = R[:, (v + 1) % 3]
        cams.append(scenes.make_camera(64, 48, 50.0, 50.0, 32.0, 24.0, (R if v % 3 else scenes.random_rotation(rng)).astype(np.float32),
                                       rng.uniform(-3, 3, 3).astype(np.float32)))
    check_records(g, cams, iso)
