"""Small launches: the render's four-ray chunks against its sixteen-ray ones
(the same operations per ray: equal bit for bit), and tables of every bucket
size around the sorts' limits, over up to 20 views, against the oracle's order."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp
from paper_2404_14044_amd import scenes

from hp_cases import check_depth_summaries, compare_table_rowmajor
from test_gpu_search_launches import _sheets

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [hp.HP_FP32, hp.HP_BF16])
@pytest.mark.parametrize("W,H,K,S", [(1, 1, 8, 16), (3, 1, 5, 6), (17, 3, 24, 64), (64, 64, 8, 8), (313, 314, 8, 16),
                                     (256, 384, 4, 48), (331, 297, 7, 16)])
def test_four_ray_chunks(W, H, K, S, prec):
    sc = _sheets(30000, W, H, radius=0.01, K=K, S=S, gamma=0.5)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(W)
    feat = torch.from_numpy(rng.normal(size=(sc.xyz.shape[0], 32)).astype(np.float32)).to(dev)
    mlp = hp.to_device_mlp(sc.mlp, dev)
    tab = hp.build_table(torch.from_numpy(sc.xyz).to(dev), sc.cams, sc.params)
    smp = hp.search_sample(tab, sc.params)
    a, b = (hp.render(smp, tab.n_rays, feat, mlp, sc.params.replace(render_rays=r), prec) for r in (0, 16))
    for k in ("rgb", "depth", "acc"):
        assert torch.equal(a[k].view(torch.int32), b[k].view(torch.int32)), k


SIZES = [0, 1, 2, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 200]


@pytest.mark.parametrize("views", [1, 2])
def test_buckets_of_several_blocks(views):
    _check_sizes([8191, 8192, 8193, 13000, 1025, 1, 0], 21, 9, views)


LARGE = [128, 129, 255, 256, 257, 300, 511, 512, 513, 600, 4095, 4096, 4097, 17, 40, 3, 0]


@pytest.mark.parametrize("W,H,views", [(21, 9, 1), (21, 9, 17), (800, 700, 2)])
def test_large_bucket_sizes(W, H, views):
    _check_sizes(LARGE, W, H, views)


@pytest.mark.parametrize("views", [1, 17, 20])
@pytest.mark.parametrize("W,H", [(21, 9), (800, 700)])
def test_bucket_sizes(W, H, views):
    if views > 1 and W > 100:
        views = 2
    _check_sizes(SIZES, W, H, views)


def _check_sizes(sizes, W, H, views):
    """Row 4 of the view has `sizes` points in its first pixels, shuffled so that
    each wave's four buckets differ, a third of them at equal depths."""
    rng = np.random.default_rng(views)
    cam = scenes.pinhole(W, H, 40.0, np.eye(3), np.zeros(3))
    pts = []
    for u, n in enumerate(rng.permutation(sizes)):
        z = rng.uniform(2.0, 3.0, n)
        z[: n // 3] = 2.5
        x = (u + 0.5 + rng.uniform(-0.3, 0.3, n) - cam.cx) / cam.fx * z
        y = (4.5 + rng.uniform(-0.3, 0.3, n) - cam.cy) / cam.fy * z
        pts.append(np.stack([x, y, z], 1))
    xyz = np.concatenate(pts)
    xyz = np.ascontiguousarray(xyz[rng.permutation(len(xyz))], np.float32)
    p = scenes.default_params(0.002, 1.0, 5.0, K=4, S=8)
    cams = [cam] + [scenes.pinhole(W + i % 3, H, 40.0, np.eye(3), np.zeros(3)) for i in range(1, views)]
    sc = scenes.Scene("sizes", xyz, np.zeros((len(xyz), 32), np.float32), cams, p, scenes.make_mlp(1))
    tab = hp.build_table(torch.from_numpy(xyz).cuda(), cams, p)
    for v in range(views):
        compare_table_rowmajor(sc, tab, v)
        check_depth_summaries(sc, tab, v)
