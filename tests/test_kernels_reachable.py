"""Nothing in the kernels' sources is out of reach: no kernel that no launch can
choose, no argument that no kernel reads, no function that nothing calls."""
import glob
import os
import re

import pytest

from paper_2404_14044_amd import build


def test_render_kernels_of_four_ray_chunks():
    # chunks of four rays are the library's own choice, without a persistent
    # grid, and fit the shared-weights kernel at any sample cap
    blob = open(build.LIB_PATH, "rb").read()
    names = set(re.findall(rb"_ZN2hp\d+k_render_[A-Za-z0-9_]*ILi4E[A-Za-z0-9_]*|_ZN2hp15k_render_shared[A-Za-z0-9_]*", blob))
    assert any(b"k_render_sharedILi0ELi4E" in n for n in names) and any(b"k_render_sharedILi1ELi4E" in n for n in names)
    assert not [n for n in names if b"k_render_bf16" in n or b"k_render_fp32" in n]


CSRC = sorted(glob.glob(os.path.join(build.CSRC, "*.h*")))


def _code(path):
    text = re.sub(r"/\*.*?\*/", "", open(path).read(), flags=re.S)
    return re.sub(r"//[^\n]*", "", text)


@pytest.mark.parametrize("struct,source", [("RenderArgs", "render.hip"), ("KnpArgs", "knp.hip"),
                                           ("FusedArgs", "fused.hip"), ("BwdArgs", "backward.hip")])
def test_kernels_read_every_argument(struct, source):
    decl = [m.group(1) for p in CSRC for m in re.finditer(r"struct %s \{(.*?)\n\};" % struct, _code(p), re.S)]
    assert len(decl) == 1
    fields = [re.sub(r"\[.*", "", f).strip(" *") for line in decl[0].split(";") if line.strip()
              for f in (line.split(None, 1)[1].replace("const ", "").replace("float *", "")).split(",")]
    used = _code(os.path.join(build.CSRC, source))
    fields = [f.split()[-1].strip("*") for f in fields]
    assert not [f for f in fields if not re.search(r"(\ba|\bA|phase_arg<\w+>\(\))\.%s\b" % f, used)], fields


def test_every_function_is_called():
    text = "\n".join(_code(p) for p in CSRC)
    names = set(re.findall(r"(?:inline|static|__global__|constexpr)[^;{}()=]*?\b([a-z_][a-z0-9_]*)\s*\([^;{}]*\)\s*\n?\{", text))
    assert len(names) > 80
    assert not sorted(n for n in names if len(re.findall(r"\b%s\b" % n, text)) < 2)
