"""The search's launch shapes: launches of many rays, dealt out inside workgroups
as large as a CU, against one-wave workgroups; the one-call search and render
with lists of every length, both samplers and decoders, on both sides of its
chunk rule, against the separate calls; K nearest points in windows on both
sides of the limits between slot runs and buckets, against the oracle.  All
equal bit for bit (the same operations in the same order)."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp
from paper_2404_14044_amd import scenes

from test_gpu_fused import _both
from test_gpu_search_groups import _check_knp, _scene

pytestmark = pytest.mark.gpu


def _sheets(n, W, H, **kw):
    """Two sheets with holes that fill the middle half of the view, and clumps."""
    rng = np.random.default_rng(n)
    front = rng.uniform([-0.4, -0.4, 1.95], [0.4, 0.4, 2.05], (n, 3))
    front = front[np.sin(front[:, 0] * 40) > -0.3]
    back = rng.uniform([-0.3, -0.3, 3.0], [0.6, 0.2, 3.02], (n // 4, 3))
    clump = rng.normal(size=(n // 8, 3)) * 0.01 + [0.1, 0.05, 2.4]
    return _scene(np.concatenate([front, back, clump]), W, H, **kw)


def _same(a, b):
    assert a.keys() == b.keys()
    for k in a:
        if torch.is_tensor(a[k]):
            assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k


def _valid(s, K):
    """The entries a caller may read: rows past a ray's sample count are scratch."""
    out = {k: s[k] for k in ("n_sel", "n_nbr", "flags", "primary") if k in s}
    live = torch.arange(s["t"].reshape(s["n_sel"].numel(), -1).shape[1], device="cuda") < s["n_sel"].reshape(-1, 1)
    out["t"] = s["t"].reshape(live.shape)[live]
    for k in ("knn_idx", "knn_dist"):
        out[k] = s[k].reshape(*live.shape, K)[live]
    return out


@pytest.mark.parametrize("K", [3, 8, 16, 24])
@pytest.mark.parametrize("W,H", [(512, 512), (513, 512), (1009, 757)])
def test_dealt_launches(W, H, K):
    sc = _sheets(60000, W, H, radius=0.004, K=K, S=16)
    xyz = torch.from_numpy(sc.xyz).cuda()
    colors = torch.from_numpy(scenes.point_colors(sc.xyz.shape[0], 3)).cuda()
    outs = []
    for blocks in (0, 65536):
        p = sc.params.replace(search_blocks=blocks)
        tab = hp.build_table(xyz, sc.cams, p)
        outs.append((_valid(hp.search_sample(tab, p), K), hp.knp_blend(tab, p, K, colors)))
    assert int((outs[0][0]["n_sel"] > 0).sum()) > 10000
    _same(outs[0][0], outs[1][0])
    _same(outs[0][1], outs[1][1])


@pytest.mark.parametrize("prec", [hp.HP_FP32, hp.HP_BF16])
@pytest.mark.parametrize("K", [1, 4, 7, 8, 13, 16])
@pytest.mark.parametrize("ms", [0, 150])
@pytest.mark.parametrize("W,H", [(1, 1), (7, 9), (33, 61), (257, 263), (449, 451)])
def test_one_call_is_the_separate_calls(W, H, ms, K, prec):
    sc = _sheets(20000, W, H, radius=0.01, K=K, S=16)
    p = sc.params.replace(sampler=1, ms_steps=ms) if ms else sc.params
    sc.feat[:] = np.random.default_rng(K).normal(size=sc.feat.shape)
    _both(sc, p, prec)


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("n", [600, 640, 641, 700, 6300, 6400, 6401, 7000])
def test_nearest_points_of_crowded_windows(n, layout):
    """A 5 x 3 view whose rays' windows all hold the whole cloud of n points."""
    rng = np.random.default_rng(n)
    xyz = rng.uniform([-0.02, -0.02, 2.2], [0.02, 0.02, 2.9], (n, 3))
    _check_knp(_scene(xyz, 5, 3, radius=1.2, layout=layout), 12)
