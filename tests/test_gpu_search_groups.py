"""Rays searched in groups and walked four at a time, at the sizes where that can
go wrong: key counts on both sides of every buffer limit, equal keys at the
cut, groups cut short by image rows and by the slots left, and each of the
three ways to a window's points.  All discrete outputs bit for bit against the
oracle's brute force."""
import numpy as np
import pytest

import oracle
from paper_2404_14044_amd import scenes

from hp_cases import compare_exact, gpu_forward, host

pytestmark = pytest.mark.gpu


def _scene(xyz, W, H, radius=0.03, K=8, S=16, **kw):
    xyz = np.ascontiguousarray(xyz, np.float32)
    cam = scenes.pinhole(W, H, 40.0, np.eye(3), np.zeros(3))
    p = scenes.default_params(radius, 1.0, 5.0, K=K, S=S).replace(**kw)
    feat = np.zeros((xyz.shape[0], 32), np.float32)
    return scenes.Scene("groups", xyz, feat, [cam], p, scenes.make_mlp(1))


def _pix(sc):
    return np.arange(sc.cams[0].W * sc.cams[0].H, dtype=np.int32)


def _check(sc, params=None):
    out = gpu_forward(sc, params=params)
    return compare_exact(sc, out["samples"], _pix(sc), params=params)


def _check_knp(sc, K):
    import torch
    from paper_2404_14044_amd import hashpoint as hp
    colors = scenes.point_colors(sc.xyz.shape[0], 9)
    tab = hp.build_table(torch.from_numpy(sc.xyz).cuda(), sc.cams, sc.params)
    out = hp.knp_blend(tab, sc.params, K, torch.from_numpy(colors).cuda())
    cam = sc.cams[0]
    ref = oracle.knp(oracle.to_camera(sc.xyz, cam), cam, sc.params, K, colors, _pix(sc))
    assert np.array_equal(host(out["cnt"]), ref["cnt"])
    assert np.array_equal(host(out["idx"]).reshape(-1, K), ref["idx"])
    assert np.array_equal(host(out["dist"]).view(np.int32).reshape(-1, K), ref["dist"].view(np.int32))
    # weights of at most 64 terms in binary32: sums of n terms are off by less
    # than n units in the last place of values below 1
    assert np.abs(host(out["rgb"]).reshape(-1, 3) - ref["rgb"]).max() <= 64 * 2.0 ** -23


def _ray_points(rng, cam, u, v, n, t_lo, t_hi, off):
    """n points within `off` of the ray through pixel (u, v)."""
    d = np.array([(u + 0.5 - cam.cx) / cam.fx, (v + 0.5 - cam.cy) / cam.fy, 1.0])
    d /= np.linalg.norm(d)
    e = np.cross(d, rng.normal(size=(n, 3)))
    e *= (off * np.sqrt(rng.uniform(0, 1, (n, 1)))) / np.linalg.norm(e, axis=1, keepdims=True)
    return d * rng.uniform(t_lo, t_hi, (n, 1)) + e


# 64: list length; 128, 512: keys held by a walked ray and by the multi-surface
# sampler's; 192, 576: the same with a step's 64 more
COUNTS = [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 193, 511, 512, 513, 600]


@pytest.mark.parametrize("n", COUNTS)
def test_neighbour_counts_around_the_limits(n):
    """A row of six pixels whose third ray has exactly n neighbours (its own
    search radius is far below a pixel), the others 0, 1, 70 and 5."""
    rng = np.random.default_rng(n)
    cam = scenes.pinhole(6, 1, 40.0, np.eye(3), np.zeros(3))
    pts = [_ray_points(rng, cam, u, 0, m, 2.0, 2.6, 0.0009)
           for u, m in ((2, n), (0, 1), (3, 70), (5, 5))]
    sc = _scene(np.concatenate(pts)[rng.permutation(n + 76)], 6, 1, radius=0.001)
    ex = _check(sc)
    assert list(ex["n_nbr"]) == [1, 0, min(n, 64), 64, 0, 5]
    assert ex["flags"][2] == (1 if n > 64 else 0)
    _check(sc, sc.params.replace(m_cap=7, K=3))
    _check(sc, sc.params.replace(sampler=1, ms_steps=5000, K=5))
    _check_knp(sc, 8)
    _check_knp(sc, 64)


@pytest.mark.parametrize("copies", [65, 129, 300, 700])
def test_equal_keys_at_the_cut(copies):
    """Copies of one point: every key has the same upper half, so the kept 64
    are decided by the point index alone; nearer and farther copies beside."""
    rng = np.random.default_rng(copies)
    a = np.repeat([[0.01, 0.0, 2.5]], copies, 0)
    b = np.repeat([[0.0, 0.01, 2.7]], 40, 0)
    c = np.repeat([[0.0, 0.0, 2.4]], 20, 0)
    xyz = np.concatenate([a, b, c, rng.uniform([-0.5, -0.3, 2.3], [0.5, 0.3, 2.8], (500, 3))])
    sc = _scene(xyz[rng.permutation(len(xyz))], 9, 7, radius=0.05)
    ex = _check(sc)
    assert (ex["flags"] > 0).any()
    _check(sc, sc.params.replace(K=24, n_samples=64, gamma=0.1))
    _check(sc, sc.params.replace(sampler=1, ms_steps=400))
    _check_knp(sc, 30)


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("chunk", [1, 3, 4, 7, 64])
def test_groups_cut_by_rows_and_slots(layout, chunk):
    """37 x 5 pixels (no multiple of four), a sheet with holes in front of a
    second one: empty rays break the groups; every layout, both windows."""
    rng = np.random.default_rng(chunk)
    front = rng.uniform([-0.8, -0.15, 1.95], [0.8, 0.15, 2.05], (9000, 3))
    front = front[np.sin(front[:, 0] * 40) > -0.3]
    back = rng.uniform([-0.6, -0.1, 3.0], [0.2, 0.2, 3.02], (1500, 3))
    sc = _scene(np.concatenate([front, back]), 37, 5, radius=0.02, layout=layout, search_chunk=chunk,
                window_shape=chunk % 2)
    ex = _check(sc)
    assert (ex["n_nbr"] == 0).any() and (ex["n_nbr"] > 8).any()


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("n", [400, 4000, 40000])
def test_windows_of_few_and_of_many_points(layout, n):
    """The same 11 x 11 view with windows that hold few points (slot runs) and
    many (buckets, their tails flattened), and one grazing bucket of 2,000
    points; fixed radius and the per-pixel cone."""
    rng = np.random.default_rng(n)
    xyz = np.concatenate([rng.uniform([-0.8, -0.8, 2.0], [0.8, 0.8, 2.6], (n, 3)),
                          _ray_points(rng, scenes.pinhole(11, 11, 40.0, np.eye(3), np.zeros(3)), 4, 6, 2000, 1.2, 4.8,
                                      0.002)])
    sc = _scene(xyz, 11, 11, radius=0.04, layout=layout)
    _check(sc)
    _check(sc, sc.params.replace(radius_mode=1, rddot=scenes.eq3_rddot(1, 0.04, 1.0), K=16))
    _check_knp(sc, 12)
