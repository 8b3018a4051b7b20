"""The entry counts of a tile (csrc/tile_sum.hpp) at and above 2^32, where 32
bits would wrap: compiled for the host and compared with whole numbers."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_14814_amd", "csrc")

PROGRAM = """
#define MS_HD inline
#include "tile_sum.hpp"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv)
{
    uint64_t w[8] = {};
    for (int i = 1; i < argc; ++i) w[i - 1] = strtoull(argv[i], nullptr, 10);
    for (int wv = 0; wv < 8; ++wv) {
        uint32_t before;
        const uint64_t total = ms::tile_total<8>(w, wv, before);
        printf("%llu %u %d %u\\n", (unsigned long long)total, before, (int)ms::tile_placed(total), ms::tile_count(w[wv]));
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_sum")
    src, exe = str(d / "main.cpp"), str(d / "main")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-I", CSRC, src, "-o", exe], check=True)
    return exe


# a triangle of 64 x 64 x 64 x 32 occupied cells has 2^23 entries, a wave of them 2^29, a tile 2^32
@pytest.mark.parametrize("waves", [
    [0] * 8, [0, 0, 5, 0, 0, 0, 0, 7], [1 << 29] * 8, [1 << 29] * 7 + [(1 << 29) + 1], [1 << 29] * 7 + [(1 << 29) - 1],
    [1 << 32] + [0] * 7, [0] * 7 + [1 << 32], [(1 << 32) - 1] * 8, [64 * ((1 << 32) - 1)] * 8, [3, 1 << 40, 9, 0, 0, 0, 0, 1]])
def test_totals_do_not_wrap(program, waves):
    out = subprocess.run([program, *map(str, waves)], check=True, capture_output=True, text=True).stdout
    for wv, line in enumerate(out.split("\n")[:8]):
        total, before, placed, count = map(int, line.split())
        assert total == sum(waves)
        assert placed == (total < 1 << 32)
        if placed:
            assert before == sum(waves[:wv])
        assert count == min(waves[wv], (1 << 32) - 1)
