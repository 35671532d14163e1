"""The rays a wave takes at a time: in launches of many rays, chunks smaller than the
default give its results in its time, though the caller names single rays; and
the default of a sparse cloud is as fast as any."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp
from paper_2404_14044_amd import scenes

from hp_timing import times_in_turn
from test_gpu_search_launches import _same, _valid

pytestmark = pytest.mark.gpu


def _sheet(W, H):
    """200k points on a sheet that fills the view."""
    cam = scenes.pinhole(W, H, 60.0, np.eye(3), np.zeros(3))
    rng = np.random.default_rng(5)
    xy = rng.uniform(-1, 1, (200_000, 2)) * np.array([W, H]) / 2 / cam.fx
    z = rng.uniform(4.5, 4.52, (200_000, 1))
    xyz = torch.from_numpy(np.concatenate([xy * z, z], 1).astype(np.float32)).cuda()
    colors = torch.from_numpy(scenes.point_colors(200_000, 3)).cuda()
    return cam, xyz, colors, scenes.default_params(0.02, 1.5, 10.0, K=8, S=16)


@pytest.mark.parametrize("op", ["search", "blend"])
@pytest.mark.parametrize("layout", [0, 2])
def test_sparse_clouds(layout, op):
    """200 x 200 rays, five points each: two rays at a time took 1.5 times as long as
    four."""
    cam, xyz, colors, p = _sheet(200, 200)
    p = p.replace(layout=layout)
    tab = hp.build_table(xyz, [cam], p)
    chunks = (0, 2, 4, 8)
    runs = []
    for chunk in chunks:
        q = p.replace(search_chunk=chunk)
        out = hp.alloc_samples(tab.n_rays, q, xyz.device)
        runs.append((lambda q=q, out=out: hp.search_sample(tab, q, out=out)) if op == "search" else
                    (lambda q=q: hp.knp_blend(tab, q, 8, colors)))
    times = dict(zip(chunks, times_in_turn(runs)))
    print(op, times)
    assert times[0] <= 1.25 * times[4], times


@pytest.mark.parametrize("op", ["search", "blend"])
@pytest.mark.parametrize("W,H", [(129, 128), (256, 255), (500, 501)])
@pytest.mark.parametrize("chunk", [1, 2, 3])
def test_small_chunks(W, H, chunk, op):
    cam, xyz, colors, p = _sheet(W, H)
    tab = hp.build_table(xyz, [cam], p)
    runs = [(lambda q=q: hp.search_sample(tab, q)) if op == "search" else (lambda q=q: hp.knp_blend(tab, q, 8, colors))
            for q in (p, p.replace(search_chunk=chunk))]
    _same(*[_valid(run(), 8) if op == "search" else run() for run in runs])
    times = times_in_turn(runs)
    print(op, W, H, chunk, times)
    # (single rays took 1.4 to 2.8 times the default's time)
    assert times[1] <= 1.25 * times[0], times
