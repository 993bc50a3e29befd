"""Host check of the work-group order of hoisted rotations' KeyMult (no GPU):
the header that the kernels use, compiled for the host, gives every (row,
rotation, tile) to one work-group, within the grid's limits for every number
of rotations that a call takes."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_13055_amd", "csrc")
DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "xcd_rows.h"
using namespace ckks;
// args: 0 rows tiles n_rot -> the grid; 1 rows tiles n_rot -> grid, lost and repeated items, work-groups of each XCD
int main(int argc, char** argv)
{
    const bool all = atoi(argv[1]) != 0;
    for (int a = 2; a + 2 < argc; a += 3) {
        const uint32_t rows = atoi(argv[a]), tiles = atoi(argv[a + 1]), n_rot = atoi(argv[a + 2]);
        const XcdGrid g = XcdRows::grid(rows, tiles, n_rot);
        printf("%u %u %u", g.x, g.y, g.z);
        if (all) {
            std::vector<int> seen((size_t)rows * tiles * n_rot, 0);
            long xcd[8] = {}, lost = 0, more = 0, out = 0, linear = 0;
            for (uint32_t z = 0; z < g.z; z++)
                for (uint32_t y = 0; y < g.y; y++)
                    for (uint32_t x = 0; x < g.x; x++, linear++) {
                        const XcdRows X(XcdGrid{x, y, z}, g.y, rows, tiles, n_rot);
                        if (X.row < 0) continue;
                        if (X.row >= (int)rows || X.rot < 0 || X.rot >= (int)n_rot || X.tile < 0 || X.tile >= (int)tiles) out++;
                        else seen[((size_t)X.row * n_rot + X.rot) * tiles + X.tile]++, xcd[linear & 7]++;
                    }
            for (int s : seen) lost += s == 0, more += s > 1;
            printf(" %ld %ld %ld", out, lost, more);
            for (long v : xcd) printf(" %ld", v);
        }
        printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("xcd_rows")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "driver.cpp"), "-o", exe], check=True)

    def run(every, sizes):
        args = [str(v) for s in sizes for v in s]
        out = subprocess.run([exe, str(int(every)), *args], check=True, capture_output=True, text=True).stdout
        return [[int(v) for v in line.split()] for line in out.splitlines()]

    return run


ROWS = list(range(2, 41)) + [63, 64]
TILES = [4, 8, 16, 32, 64]  # N / 1024
SIZES = [(r, t, n) for r in ROWS for t in TILES for n in (1, 2, 3, 7, 32)]


def test_grid_limits(order):
    """Work-groups along y and z, work-items of 256-thread work-groups along x."""
    sizes = [(r, t, n) for r in ROWS for t in TILES for n in (1, 8191, 8192, 32767, 32768, 65535)]
    for size, (x, y, z) in zip(sizes, order(False, sizes)):
        assert x * 256 < 1 << 32 and 1 <= y <= 65535 and 1 <= z <= 65535, size


def test_every_item_once(order):
    for size, r in zip(SIZES, order(True, SIZES)):
        assert r[3:6] == [0, 0, 0], size


def test_balance(order):
    """No XCD has more than its eighth of the items, up to a row's last tiles."""
    for size, r in zip(SIZES, order(True, SIZES)):
        rows, tiles, n_rot = size
        assert max(r[6:]) <= rows * tiles * n_rot / 8 + rows % 8, size
