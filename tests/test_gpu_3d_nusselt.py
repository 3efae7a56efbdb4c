"""The wall Nusselt number of the 3-D path, a sum over blocks of 256 wall cells, against the
same mean taken from the temperature field: cell counts around one block, more blocks than
the threads that add their sums, all six walls and every storage type; a second call and a
call after more steps (the count of finished blocks starts from zero again).

Tolerance: the cell values are the same FP64 numbers on both sides, so that the two differ
by the order of summation of n cells and by the rounding of a few operations per cell, at
most (n + 16) 2^-53 on each side, times the mean of the absolute values."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, nz, periodic_x, periodic_y, periodic_z, walls
    (4, 16, 16, 0, 1, 1, (2, 3)),        # 256 cells
    (5, 3, 85, 0, 1, 1, (2, 3)),         # 255
    (257, 1, 4, 1, 1, 0, (0, 1)),        # 257
    (17, 9, 11, 0, 0, 0, (0, 1, 2, 3, 4, 5)),
    (277, 241, 4, 1, 1, 0, (0, 1)),      # 261 blocks
]


def _from_fields(T, per, wall, L, dT):
    ax = {0: 0, 1: 2, 2: 1}[wall // 2]                       # normal axis of [z][y][x]
    per = list(per)
    T = np.moveaxis(T, ax, 0)
    per = per[:ax] + per[ax + 1:]
    if wall % 2:
        T = T[::-1]
    d = (-3.0 * T[0] + 4.0 * T[1] - T[2]) / 2.0
    v = -L * (-d if wall % 2 else d) / dT
    w = [np.ones(n) for n in v.shape]
    den = 1.0
    for a in range(2):
        if not per[a]:
            w[a][[0, -1]] = 0.5
        den *= v.shape[a] if per[a] else v.shape[a] - 1
    v = v * w[0][:, None] * w[1][None, :]
    return float(v.sum() / den), float(np.abs(v).sum() / den), v.size


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny,nz,px,py,pz,walls", CASES)
def test_nusselt_is_the_mean_of_the_wall_cells(nx, ny, nz, px, py, pz, walls, storage):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm3d
    cfg = W.random_case3d(31, nx, ny, nz, periodic_z=pz, storage=storage, periodic_x=px, periodic_y=py)
    sim = lbm3d.Sim3(cfg)
    dT = cfg["T_hot"] - cfg["T_cold"]
    for steps in (0, 3, 0):
        print(f"case: {nx}x{ny}x{nz} {storage}, {steps} more steps", flush=True)
        sim.step(steps)
        T = sim.fields()["T"].double().cpu().numpy()
        for w in walls:
            ref, scale, n = _from_fields(T, (pz, py, px), w, cfg["L"], dT)
            assert abs(sim.nusselt(w) - ref) <= 2 * (n + 16) * 2.0 ** -53 * scale
