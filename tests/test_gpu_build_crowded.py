"""Tables whose buckets hold far more points than a workgroup sorts in its LDS (a
cloud seen in a few pixels, coincident points): the order on both sides of the
limit between the two ways to sort them, against the oracle's, and how the time
grows with the bucket."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp
from paper_2404_14044_amd import scenes

from hp_timing import times_in_turn
from test_gpu_small_launches import LARGE, SIZES, _check_sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 2])
def test_order_of_crowded_buckets(views):
    _check_sizes([24_575, 24_576, 24_577, 131_075, 4096, 3, 0], 21, 9, views)


def test_time_of_one_bucket_does_not_grow_with_its_square():
    """One bucket of 32,768 and of 262,144 points.  A sorting network's work grows
    by 8 log2(262144)^2 / log2(32768)^2 = 11.5, work that grows with the square of
    the bucket by 64: the bound is their geometric mean, 27."""
    cam = scenes.pinhole(21, 9, 40.0, np.eye(3), np.zeros(3))
    p = scenes.default_params(0.002, 1.0, 5.0, K=4, S=8)
    times = []
    for n in (32_768, 262_144):
        rng = np.random.default_rng(n)
        z = rng.uniform(2.0, 3.0, n)
        xy = (np.array([[7.5, 4.5]]) + rng.uniform(-0.3, 0.3, (n, 2)) - [cam.cx, cam.cy]) / cam.fx * z[:, None]
        xyz = torch.from_numpy(np.concatenate([xy, z[:, None]], 1).astype(np.float32)).cuda()
        ws = torch.empty(hp.table_workspace(n, [cam], p), dtype=torch.uint8, device="cuda")
        times += times_in_turn([lambda: hp.build_table(xyz, [cam], p, ws=ws)], reps=3, inner=1)
    assert times[1] <= 27 * times[0], times


@pytest.mark.parametrize("sizes", [SIZES, LARGE, [8191, 8192, 8193, 13_000, 24_577, 1025, 1, 0]],
                         ids=["small", "large", "blocks"])
def test_one_level_build(sizes):
    """A view of more than 2^23 buckets is built in one level, which sorts the
    buckets' keys and makes the points of them afterwards."""
    cam = scenes.pinhole(3000, 3000, 40.0, np.eye(3), np.zeros(3))
    g, _ = hp.view_bounds(cam, scenes.default_params(0.002, 1.0, 5.0, K=4, S=8))
    assert (3000 + 2 * g) ** 2 > 2 ** 23
    _check_sizes(sizes, 3000, 3000, 1)
