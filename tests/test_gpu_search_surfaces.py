"""The multi-surface sampler's launches: rays dealt singly against rays dealt in
chunks (the same results, and a sparse cloud pays nothing for it), and
neighbour counts on both sides of the keys that a ray holds."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp
from paper_2404_14044_amd import scenes

from hp_timing import times_in_turn
from test_gpu_search_groups import _check, _ray_points, _scene
from test_gpu_search_launches import _same, _sheets, _valid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(1, 1), (129, 127), (171, 163), (401, 399), (1009, 803)])
@pytest.mark.parametrize("chunk", [1, 2, 3, 5, 64])
def test_chunks_of_every_size(W, H, chunk):
    """Launches of one wave per ray and of many rays per wave, set up sixteen at a
    time, against chunks that do not divide them."""
    sc = _sheets(20000, W, H, radius=0.004, K=5, S=6)
    p = sc.params.replace(sampler=1, ms_steps=60)
    tab = hp.build_table(torch.from_numpy(sc.xyz).cuda(), sc.cams, p)
    want = _valid(hp.search_sample(tab, p), 5)
    _same(_valid(hp.search_sample(tab, p.replace(search_chunk=chunk, search_blocks=8192 if chunk % 2 else 0)), 5), want)


@pytest.mark.parametrize("n", [383, 384, 385, 447, 448, 449, 512, 513])
@pytest.mark.parametrize("K", [3, 8, 16, 24])
def test_neighbour_counts_around_the_keys_held(n, K):
    rng = np.random.default_rng(n)
    cam = scenes.pinhole(4, 1, 40.0, np.eye(3), np.zeros(3))
    pts = [_ray_points(rng, cam, u, 0, m, 2.0, 2.6, 0.0009) for u, m in ((0, 9), (1, n), (2, 1), (3, n + 130))]
    sc = _scene(np.concatenate(pts)[rng.permutation(2 * n + 140)], 4, 1, radius=0.001, K=K, S=64)
    ex = _check(sc, sc.params.replace(sampler=1, ms_steps=3000))
    assert list(ex["n_nbr"]) == [9, 64, 1, 64]


def test_time_of_single_rays_in_a_sparse_cloud():
    """300 x 300 rays over a sheet of about two points a pixel: what a ray costs is
    its set-up, which a wave makes for sixteen rays at a time.  Single rays, the
    default, took 1.29 times as long as chunks of four where a wave set up fewer;
    they may take half of that longer at most."""
    cam = scenes.pinhole(300, 300, 60.0, np.eye(3), np.zeros(3))
    rng = np.random.default_rng(5)
    xy = rng.uniform(-1, 1, (200_000, 2)) * 150 / cam.fx
    z = rng.uniform(4.5, 4.52, (200_000, 1))
    xyz = torch.from_numpy(np.concatenate([xy * z, z], 1).astype(np.float32)).cuda()
    p = scenes.default_params(0.012, 1.5, 10.0, K=8, S=16).replace(sampler=1, ms_steps=200)
    tab = hp.build_table(xyz, [cam], p)
    out = hp.alloc_samples(tab.n_rays, p, xyz.device)
    times = times_in_turn([lambda q=q: hp.search_sample(tab, q, out=out) for q in (p, p.replace(search_chunk=4))])
    print(times)
    assert times[0] <= 1.13 * times[1], times
