"""What the plan of the launches on tiles decides (lbm_tile.hip), on the host: the fewest steps of a
launch, whether every step of a launch is stored, where a grid or a batch leaves tiles, and whether one small problem changes the tiles of a
whole batch.  The sizes lie well off the lines, on the side where the measured times are."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F64, F32, F16 = 0, 1, 2

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lbm_kernels.h"
// arguments: storage field periodic_x periodic_y, then nx ny count for every kind of problem; prints the
// most and the fewest steps of a launch, the largest tile of the first problem and whether launches
// that store every step pay
int main(int n, char **v)
{
    std::vector<lbm::KParams> P;
    for (int i = 5; i + 2 < n; i += 3) {
        lbm::KParams k = {};
        k.nx = atoi(v[i]);
        k.ny = atoi(v[i + 1]);
        k.field = atoi(v[2]);
        k.px = atoi(v[3]);
        k.py = atoi(v[4]);
        for (int m = 0; m < atoi(v[i + 2]); ++m) P.push_back(k);
    }
    std::vector<lbm::TileGrid> g(P.size());
    const lbm::TileSteps t = lbm::tile_plan(atoi(v[1]), P.data(), (int)P.size(), g.data());
    printf("%d %d %d %d %d\n", t.most, t.least, t.most ? g[0].tw + (g[0].rx > 0) : 0, t.most ? g[0].th + (g[0].ry > 0) : 0, (int)t.every);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    from paper_1505_02976_amd import build, lbm
    if not os.path.exists(lbm.LIB_PATH):
        build.build()
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "plan.hip"), str(d / "plan")
    with open(src, "w") as fh:
        fh.write(SOURCE)
    libdir = os.path.dirname(lbm.LIB_PATH)
    subprocess.run([build.HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(libdir, "csrc"), "-x", "hip", src,
                    "-x", "none", lbm.LIB_PATH, "-Wl,-rpath," + libdir, "-o", exe], check=True, stderr=subprocess.DEVNULL)

    def call(storage, grids, field=0, px=0, py=0):
        a = [storage, field, px, py] + [x for g in grids for x in g]
        out = subprocess.run([exe] + [str(x) for x in a], check=True, capture_output=True, text=True).stdout
        return tuple(map(int, out.split()))
    return call


@pytest.mark.parametrize("storage,nx,ny,field,least", [
    (F64, 128, 128, 0, 1), (F64, 350, 350, 0, 1), (F64, 500, 507, 0, 2), (F64, 1150, 1157, 0, 3), (F64, 2200, 2200, 0, 3),
    (F32, 250, 250, 0, 1), (F32, 460, 467, 0, 1), (F32, 640, 647, 0, 2), (F32, 950, 957, 0, 2), (F32, 1250, 1257, 0, 3),
    (F32, 1800, 1900, 0, 4), (F32, 1650, 1657, 1, 3), (F32, 2200, 2200, 1, 4),
    (F16, 640, 647, 0, 1), (F16, 850, 857, 0, 2), (F16, 1250, 1257, 0, 3),
    # walls few nodes apart; one wavefront of the passes across, one and a little
    (F64, 124, 1209, 0, 2), (F64, 2500, 60, 1, 2), (F32, 14705, 17, 1, 2), (F32, 64, 9375, 0, 2), (F32, 30303, 33, 0, 3), (F32, 60606, 33, 0, 4),
    (F64, 32, 100000, 0, 1), (F64, 64, 3906, 1, 1), (F64, 40, 60000, 0, 2), (F16, 80, 30000, 1, 2),
    # one block: any number, but for one step between walls
    (F64, 4, 64, 0, 1), (F32, 22, 22, 0, 2), (F16, 22, 22, 0, 1),
])
def test_fewest_steps_of_a_launch(plan, storage, nx, ny, field, least):
    most, got, _, _, _ = plan(storage, [(nx, ny, 1)], field)
    assert got == least and most >= got


@pytest.mark.parametrize("storage,grid,count,field,least", [
    (F64, (200, 203), 10, 0, 1), (F64, (200, 203), 20, 0, 2), (F64, (200, 203), 52, 0, 3),
    (F32, (200, 203), 6, 0, 1), (F32, (200, 203), 16, 0, 2), (F32, (200, 203), 65, 0, 3), (F32, (500, 503), 12, 1, 4),
    (F16, (200, 203), 10, 0, 1), (F16, (500, 503), 6, 0, 2), (F16, (500, 503), 15, 0, 3), (F16, (47, 400), 200, 0, 1),
])
def test_fewest_steps_of_a_batch(plan, storage, grid, count, field, least):
    most, got, _, _, _ = plan(storage, [grid + (count,)], field)
    assert got == least and most >= got


@pytest.mark.parametrize("storage", [F64, F32, F16])
@pytest.mark.parametrize("grid,count", [((200, 203), 64), ((1000, 1000), 3)])
def test_one_small_problem_does_not_change_the_tiles(plan, storage, grid, count):
    assert plan(storage, [grid + (count,), (40, 40, 1)]) == plan(storage, [grid + (count,)])


@pytest.mark.parametrize("storage,nx,ny,tile", [
    (F64, 20000, 40, (26, 10)), (F32, 20000, 40, (26, 10)), (F32, 123076, 26, (26, 9)), (F16, 20000, 40, (28, 10)),
])
def test_tiles_of_a_few_rows(plan, storage, nx, ny, tile):
    most, _, tw, th, _ = plan(storage, [(nx, ny, 1)])
    assert most >= 3 and (tw, th) == tile


@pytest.mark.parametrize("storage,nx,ny,count,field,tiles", [
    (F64, 26666, 60, 1, 0, False), (F64, 10000, 60, 1, 0, True), (F64, 16000, 200, 1, 1, False), (F64, 8000, 200, 1, 1, True),
    (F64, 15000, 400, 1, 0, False), (F64, 333333, 12, 1, 0, True), (F64, 96969, 33, 1, 0, False), (F64, 200000, 4, 1, 1, False),
    (F64, 62, 25806, 1, 1, False), (F64, 124, 12903, 1, 0, True), (F64, 1537, 1025, 1, 1, True), (F64, 3500, 3400, 1, 1, True),
    (F16, 26666, 60, 1, 0, False), (F16, 16000, 200, 1, 0, False), (F16, 13333, 60, 1, 1, True), (F16, 2500, 2507, 1, 1, False),
    (F32, 60000, 200, 1, 1, False), (F32, 30000, 200, 1, 1, True), (F32, 1800, 1900, 1, 0, True),
    (F64, 6000, 47, 12, 0, False), (F64, 500, 503, 12, 0, True), (F32, 1000, 1000, 5, 0, False), (F32, 1000, 1000, 5, 1, True),
])
def test_where_grids_leave_tiles(plan, storage, nx, ny, count, field, tiles):
    assert (plan(storage, [(nx, ny, count)], field)[0] > 0) == tiles


def test_rows_between_no_walls_have_no_limit(plan):
    assert plan(F64, [(26666, 60, 1)], 0, 0, 1)[0] > 0


@pytest.mark.parametrize("storage,n,every", [
    (F64, 640, True), (F64, 1024, False), (F32, 450, True), (F32, 640, False), (F16, 768, True), (F16, 1024, False),
])
def test_where_states_come_from_tiles(plan, storage, n, every):
    most, _, _, _, got = plan(storage, [(n, n, 1)], 1)
    assert most > 0 and bool(got) == every
