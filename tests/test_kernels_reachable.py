"""The library holds no render kernel that no launch can choose."""
import re

from paper_2404_14044_amd import build


def test_render_kernels_of_four_ray_chunks():
    # chunks of four rays are the library's own choice, without a persistent
    # grid, and fit the shared-weights kernel at any sample cap
    blob = open(build.LIB_PATH, "rb").read()
    names = set(re.findall(rb"_ZN2hp\d+k_render_[A-Za-z0-9_]*ILi4E[A-Za-z0-9_]*|_ZN2hp15k_render_shared[A-Za-z0-9_]*", blob))
    assert any(b"k_render_sharedILi0ELi4E" in n for n in names) and any(b"k_render_sharedILi1ELi4E" in n for n in names)
    assert not [n for n in names if b"k_render_bf16" in n or b"k_render_fp32" in n]
