"""The collision check where lambda_g times a Gaussian's principal axis is beyond binary32 (a finite
log-scale above about 87.6): the Gaussian holds every point, and its clearance is below every binary32 number.  The flags are
the oracle's, with and without clearances and in both entry points."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [40.0, 90.0, 200.0])
@pytest.mark.parametrize("n,p", [(1, 1), (2, 70), (1000, 129), (5000, 300)])
def test_overflowing_axis(n, p, scale):
    from paper_2409_18122_amd import raster
    print(f"collision overflow n={n} p={p} scale={scale}", flush=True)
    rng = np.random.default_rng(n + p)
    means = rng.uniform(-9, 9, (3, n)).astype(np.float32)
    means[:, 0] = (1.0, 0.0, 0.0)
    ls = rng.normal(-2.5, 0.6, (3, n)).astype(np.float32)
    ls[1, 0] = scale
    pts = rng.uniform(-9, 9, (3, p)).astype(np.float32)
    pts[:, 0] = 0.0
    ref, _ = oracle.collision(means, ls, pts, 0.25, 3.0)
    assert ref.all()
    ctx = raster.Context(0)
    g = {"means": torch.as_tensor(means).cuda(), "log_scales": torch.as_tensor(ls).cuda()}
    x = torch.as_tensor(pts).cuda()
    for clearance in (True, False):
        for no_alloc in (True, False):
            hit, clr = raster.collision_check(ctx, g, x, 0.25, 3.0, clearance=clearance, no_alloc=no_alloc)
            assert np.array_equal(hit.cpu().numpy(), ref), (clearance, no_alloc)
            if clearance and scale > 88.0:
                assert torch.isneginf(clr).all()
            elif clearance:  # distances vanish beside the axis
                assert np.allclose(clr.cpu().numpy(), -3.0 * np.exp(scale), rtol=1e-6)
    ctx.close()
