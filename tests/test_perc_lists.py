"""The percolation work lists' parts, on the host: how a batch's tiles spread
over them, and that no part is given more entries than it has room for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "perc_launch.hpp"
using namespace perc;
int main(int, char** argv) {
    const uint32_t L = atoi(argv[1]), count = atoi(argv[2]), n = (L + kTile - 1u) / kTile;
    uint64_t load[kSubs] = {}, most = 0;
    for (uint32_t m = 0; m < count; ++m)
        for (uint32_t ty = 0; ty < n; ++ty)
            for (uint32_t tx = 0; tx < n; ++tx) ++load[list_part(m, tx, ty)];
    for (uint64_t l : load) most = l > most ? l : most;
    printf("%llu %llu\\n", (unsigned long long)most, (unsigned long long)(count * part_entries(L)));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("perc_lists")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_cs_0312006_amd", "csrc"), str(d / "p.cpp"), "-o", str(d / "p")], check=True)
    return str(d / "p")


@pytest.mark.parametrize("L,count", [(1, 60), (64, 32), (64, 60), (64, 1000), (65, 60), (128, 60), (512, 48), (4096, 3),
                                     (5000, 1)])
def test_tiles_spread_over_the_parts(program, L, count):
    most, room = map(int, subprocess.run([program, str(L), str(count)], capture_output=True, text=True,
                                         check=True).stdout.split())
    tiles = count * ((L + 63) // 64) ** 2
    assert most <= room
    assert most <= 2 * -(-tiles // 64), "a few parts hold most of the tiles"
