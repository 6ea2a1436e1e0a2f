"""The launches of a deterministic shading call, on the host: every query in
exactly one of them, none with 2^32 work-items or more (HIP refuses those), up
to the largest call (2^31 - 1 queries; a bicubic query takes four work-items)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "shade_grid.h"
int main(int argc, char** argv)
{
    const int64_t n = atoll(argv[1]);
    const int lanes = atoi(argv[2]), block = 256;
    for (int64_t first = 0; first < n; first += stf::SHADE_PART) {
        const int64_t m = stf::shade_part(n, first);
        printf("%lld %lld %llu\\n", (long long)first, (long long)m, (unsigned long long)stf::shade_blocks(m, lanes, block) * block);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("shade_grid")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2305_05810_amd", "csrc"),
                    str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return str(d / "p")


@pytest.mark.parametrize("lanes", [1, 2, 4])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 2 ** 22, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 1, 2 ** 30 - 63, 2 ** 30 + 1,
                               2 ** 31 - 127, 2 ** 31 - 1])
def test_launches_cover_the_call_and_can_be_launched(program, n, lanes):
    r = subprocess.run([program, str(n), str(lanes)], check=True, capture_output=True, text=True)
    at = 0
    for line in r.stdout.split("\n")[:-1]:
        first, m, items = map(int, line.split())
        assert first == at and m > 0
        assert m * lanes <= items < 2 ** 32
        assert items - m * lanes < 256   # no idle block
        at += m
    assert at == n
