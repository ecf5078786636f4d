"""Binning a frame again: the sorted pairs and the images are those of the first time, for maps
whose records are sorted in one block (up to 4,096) and in several passes."""
import pytest
import torch

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views", [(1, 1), (2000, 1), (9000, 1), (9000, 3), (120_000, 1)])
def test_bin_sort_twice(n, views):
    from paper_2409_18122_amd import raster
    print(f"bin again n={n} views={views}", flush=True)
    g, cams = scenes.config1(n=n, seed=3)
    f = raster.Frame(raster.Context(0), raster.to_device(g), list(cams) * views, dict(scenes.DEFAULT_SETTINGS))
    assert f.bin_sort() > 0
    first, images = f.export(), f.render()
    for _ in range(2):
        f.bin_sort()
        assert all(torch.equal(a, b) for a, b in zip(first, f.export()))
        again = f.render()
        assert all(torch.equal(images[k], again[k]) for k in images)
    f.close()
