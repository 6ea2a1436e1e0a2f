"""The number of a query's tap block, over every cell a query can have (within
2^24): as a constant expression, in which a signed overflow is an error, and
equal within a block of 4x4x4 voxels."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
#include "tap_block.h"
constexpr int LO = -(1 << 24) - 1, HI = (1 << 24) + 2;
constexpr int at[] = {LO, LO + 1, -5, -4, -1, 0, 3, 4, 511, 32767, 1 << 23, HI - 1, HI};
constexpr bool all()
{
    for (int x : at)
        for (int y : at)
            for (int z : at) {
                const uint32_t k = stf::tap_block(x, y, z);
                for (int d = 0; d < 4; ++d)
                    if (stf::tap_block((x & ~3) + d, (y & ~3) + 3 - d, (z & ~3) + (d ^ 1)) != k) return false;
                if (stf::tap_block(x ^ 4, y, z) == k || stf::tap_block(x, y ^ 4, z) == k || stf::tap_block(x, y, z ^ 4) == k)
                    return false;
            }
    return true;
}
static_assert(all(), "");
"""


def test_every_cell_has_a_number(tmp_path):
    (tmp_path / "p.cpp").write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I",
                        os.path.join(ROOT, "paper_2305_05810_amd", "csrc"), str(tmp_path / "p.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
