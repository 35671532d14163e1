"""Small launches: the render's four-ray chunks against its sixteen-ray ones
(the same operations per ray: equal bit for bit)."""
import numpy as np
import pytest
import torch

from paper_2404_14044_amd import hashpoint as hp

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
