"""The one-call search and render with a grid named by the caller: the results of the
default, in its time."""
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp

from hp_timing import times_in_turn
from test_gpu_search_launches import _sheets

pytestmark = pytest.mark.gpu


def _call(W, H, blocks, prec, ms=0):
    sc = _sheets(60000, W, H, radius=0.01, K=8, S=16)
    p = sc.params.replace(sampler=1, ms_steps=ms) if ms else sc.params
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    feat = torch.randn(sc.xyz.shape[0], 32, generator=gen, device="cuda")
    mlp = hp.to_device_mlp(sc.mlp, "cuda")
    tab = hp.build_table(torch.from_numpy(sc.xyz).cuda(), sc.cams, p)
    n_sel = torch.empty(tab.n_rays, dtype=torch.int32, device="cuda")
    out = {"rgb": torch.empty(3 * tab.n_rays, device="cuda"), "depth": torch.empty(tab.n_rays, device="cuda"),
           "acc": torch.empty(tab.n_rays, device="cuda"), "n_sel": n_sel}
    q = p.replace(search_blocks=blocks)
    return lambda: hp.search_render(tab, q, feat, mlp, prec, out=out)


@pytest.mark.parametrize("prec", [hp.HP_FP32, hp.HP_BF16])
@pytest.mark.parametrize("ms", [0, 100])
@pytest.mark.parametrize("blocks", [1, 7, 8, 100, 255, 256, 257, 4096, 65536, 2**31 - 1])
def test_grid_changes_no_result(blocks, ms, prec):
    want = {k: v.clone() for k, v in _call(83, 61, 0, prec, ms)().items() if torch.is_tensor(v)}
    got = _call(83, 61, blocks, prec, ms)()
    assert want
    for k, v in want.items():
        assert torch.equal(v.view(torch.int32), got[k].view(torch.int32)), k


@pytest.mark.parametrize("W", [192, 400])
def test_time_of_a_large_grid(W):
    """65,536 waves named, as for the search alone: one workgroup per CU still.  The
    2 to 5 times of a workgroup for every 16 named waves are far outside a half."""
    times = times_in_turn([_call(W, W, blocks, hp.HP_BF16) for blocks in (0, 65536)])
    print(times)
    assert times[1] <= 1.5 * times[0], times
