"""Steps against the 3-D oracle where the wall blocks lead the launch: FP16 grids whose planes or rows
are whole cache lines (layers heated from below, y walls, both), FP32 grids with y walls alone, with
planes smaller and larger than a block, walls that leave the last wall block unfilled, one interior
plane per slab and many; and FP16 x walls on both sides of the row length from which the interior
blocks take them.

Tolerance on the populations, from 12 steps of rounding, relative to the largest deviation from the
state of rest: in FP16 a stored value is rounded to 2^-11 of itself, and twice that is allowed per
step; the FP32 arithmetic adds up tens of terms, 16 roundings of 2^-23 per step."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 12
TOL = {"f32": STEPS * 2.0 ** -19, "f16": STEPS * 2.0 ** -10}


@pytest.mark.parametrize("storage,seed,nx,ny,nz,px,py,pz,ef", [
    ("f16", 61, 64, 1, 4, 1, 1, 0, False), ("f16", 62, 16, 12, 33, 1, 1, 0, True), ("f16", 63, 32, 10, 20, 1, 1, 0, False),
    ("f16", 64, 64, 40, 6, 1, 1, 0, True), ("f16", 65, 192, 11, 5, 1, 1, 0, False),
    ("f16", 66, 10, 9, 8, 0, 0, 0, True), ("f16", 67, 15, 14, 6, 0, 1, 0, False), ("f16", 68, 15, 6, 7, 0, 0, 0, True),
    ("f16", 69, 16, 14, 6, 0, 1, 0, False), ("f16", 70, 16, 6, 7, 0, 0, 0, True),
    ("f16", 71, 64, 4, 4, 1, 0, 0, False), ("f16", 72, 64, 9, 13, 1, 0, 0, True), ("f16", 73, 128, 7, 5, 1, 0, 1, False),
    ("f16", 74, 64, 5, 1, 1, 0, 1, True), ("f32", 75, 32, 4, 1, 1, 0, 1, False), ("f32", 76, 64, 9, 13, 1, 0, 1, True),
    ("f32", 77, 96, 21, 6, 1, 0, 1, False),
])
def test_step_matches_oracle(storage, seed, nx, ny, nz, px, py, pz, ef):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle.oracle3 as O3
    from paper_1505_02976_amd import lbm3d
    cfg = W.random_case3d(seed, nx, ny, nz, eps_field=ef, storage=storage, periodic_x=px, periodic_y=py, periodic_z=pz)
    print(f"case: {storage} {nx} x {ny} x {nz} field {ef}", flush=True)
    sim = lbm3d.Sim3(cfg)
    sim.step(STEPS)
    ref = O3.Oracle3(dict(cfg, storage="f64"))
    ref.step(STEPS)
    order = [tuple(int(v) for v in c) for c in O3.lattice()[0]]
    perm = [order.index(c) for c in lbm3d.lattice()]
    rest = [1.0] + [0.0] * 18
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12) * cfg["sigma"] * 0.5 * (cfg["T_hot"] + cfg["T_cold"])
    dev = [r[perm].reshape(19, -1) - np.array(o)[:, None] for r, o in zip(ref.populations(), (rest, w))]
    scale = max(float(np.abs(d).max()) for d in dev)
    for a, b in zip(sim.populations(), ref.populations()):
        assert float(np.abs(a.cpu().numpy() - b[perm]).max()) < TOL[storage] * scale
