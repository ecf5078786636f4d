"""The choice among trajectories at lengths around a batch of loads, and one long trajectory: the sums are
taken in order, bit for bit, and in less time than a load at a time would take."""
import numpy as np
import pytest
import torch

from test_gpu_collision_enclosed import _best_us

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[0], [1], [15, 16, 17, 0, 31, 32, 33], [100_000], [5000, 1, 0, 7000], [3] * 1000])
def test_sums_in_order(lengths):
    from paper_2409_18122_amd import raster
    print(f"trajectories {lengths[:4]}", flush=True)
    rng = np.random.default_rng(len(lengths))
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    xi = rng.normal(size=max(int(off[-1]), 1)) * 10.0 ** rng.integers(-8, 8, max(int(off[-1]), 1))
    ctx = raster.Context(0)
    x, o = torch.as_tensor(xi).cuda(), torch.as_tensor(off).cuda()
    util, best = raster.trajectory_select(ctx, x, o)
    ref = []
    for a, b in zip(off[:-1], off[1:]):
        s = 0.0
        for v in xi[a:b]:
            s += float(v)
        ref.append(s)
    assert util.cpu().tolist() == ref and int(best) == int(np.argmax(ref))
    ctx.close()


def test_one_long_trajectory():
    from paper_2409_18122_amd import raster
    ctx = raster.Context(0)
    x = torch.zeros(100_000, device="cuda", dtype=torch.float64)
    o = torch.tensor([0, 100_000], device="cuda", dtype=torch.int32)
    us = _best_us(lambda: raster.trajectory_select(ctx, x, o))
    print(f"one trajectory of 100,000 states: {us:.0f} us", flush=True)
    assert us < 3500.0  # a load at a time: 4,000 to 6,600
    ctx.close()
