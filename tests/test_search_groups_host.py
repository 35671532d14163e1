"""The rule that cuts a pass of rays into groups, evaluated by the compiler, which
refuses undefined steps (a shift by the width of the mask) in a constant."""
import subprocess

from paper_2404_14044_amd import build

SOURCE = r"""
#include "hp_search.hpp"
using namespace hp;

// the definition, ray by ray, for pseudo-random masks and their ends
constexpr bool agrees()
{
    uint64_t x = 88172645463325252ull;
    for (int n = 0; n < 400; ++n) {
        x ^= x << 13;
        x ^= x >> 7;
        x ^= x << 17;
        const uint64_t joined = (n == 0 ? ~0ull : n == 1 ? 0ull : n & 1 ? x : x | x >> 3) & 0x1111111111111110ull;
        for (int most = 1; most <= GROUP; ++most)
            for (int i = 0; i < RS_CAP; ++i) {
                int m = 1;
                for (int k = i + 1; k < RS_CAP && m < most && (joined & (1ull << (RS_LANES * k))); ++k) ++m;
                if (group_size(joined, i, most) != m) return false;
            }
    }
    return true;
}
static_assert(agrees(), "groups differ from their definition");
"""


def test_group_sizes(tmp_path):
    src = tmp_path / "groups.hip"
    src.write_text(SOURCE)
    res = subprocess.run([build.HIPCC, *build.FLAGS, "-fconstexpr-steps=100000000", f"-I{build.INCLUDE}",
                          f"-I{build.CSRC}", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
