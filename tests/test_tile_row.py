"""Tile number to row of tiles (lbm_tile.h) for every tile of a grid, on the host: the division by a
rounded reciprocal must be exact for each number of tiles, the longest rows above all, where the
last tile of a row is less than the reciprocal's error away from the next row."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1505_02976_amd", "csrc")

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "lbm_tile.h"
// arguments: nx ny tw th; prints the number of tiles and of those with a wrong row
int main(int, char **v)
{
    lbm::KParams P = {};
    P.nx = atoi(v[1]);
    P.ny = atoi(v[2]);
    const lbm::TileGrid g = lbm::tile_grid(P, atoi(v[3]), atoi(v[4]));
    const int n = g.nbx * g.nby;
    int wrong = 0;
    for (int b = 0; b < n; ++b) wrong += lbm::tile_row(g, b) != b / g.nbx;
    printf("%d %d\n", n, wrong);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_1505_02976_amd import build
    d = tmp_path_factory.mktemp("tile_row")
    src, exe = str(d / "row.hip"), str(d / "row")
    with open(src, "w") as fh:
        fh.write(SOURCE)
    subprocess.run([build.HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-I", CSRC, "-x", "hip", src, "-o", exe],
                   check=True, stderr=subprocess.DEVNULL)
    return exe


@pytest.mark.parametrize("nx,ny,tw,th", [
    (250, 250, 12, 8), (5, 9, 5, 4), (4096, 4096, 26, 10),
    (2163173, 1, 8, 8), (2163173, 1, 32, 8), (1829804, 2, 8, 8), (2400000, 5, 26, 10), (2200000, 4, 32, 8),
    (1579000, 4, 24, 14), (1000000, 40, 24, 14), (12000000, 1, 8, 8), (100000, 100, 8, 8), (70001, 900, 8, 8),
])
def test_row_of_every_tile(program, nx, ny, tw, th):
    out = subprocess.run([program] + [str(a) for a in (nx, ny, tw, th)], check=True, capture_output=True, text=True).stdout
    tiles, wrong = map(int, out.split())
    assert tiles >= 1 and wrong == 0, (tiles, wrong)
