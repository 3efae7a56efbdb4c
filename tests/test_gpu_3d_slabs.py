"""How one 3-D step is shared out over blocks, against the 3-D oracle over a few steps: rows of 7
interior nodes (x walls in the wall blocks) and of 8 (x walls in the interior blocks), rows longer
than a block, a last block and a last slab of planes that are not full, rows that are whole
cache lines and rows that are not, walls on one, two and three pairs, porosity per node.

Tolerances on the populations, from 12 steps of rounding: FP64 1e-10 as elsewhere; a stored value
is rounded to 2^-11 of itself in FP16, and twice that is allowed per step for the
neighbours' share; the FP32 arithmetic adds up tens of terms, 16 roundings of 2^-23 per step.  Both
are relative to the largest deviation from the state of rest."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

STEPS = 12
TOL = {"f64": 1e-10, "f32": STEPS * 2.0 ** -19, "f16": STEPS * 2.0 ** -10}

CASES = [
    # seed, nx, ny, nz, periodic_x, periodic_y, periodic_z, porosity field
    (41, 9, 11, 6, 0, 0, 0, False),      # 7 interior nodes per row
    (42, 10, 11, 6, 0, 0, 0, True),      # 8
    (43, 10, 5, 7, 0, 1, 1, False),      # 8, the x walls alone
    (44, 261, 4, 5, 0, 1, 0, False),     # rows of 259: a block may hold one end of a row, or none
    (45, 20, 19, 40, 0, 0, 0, True),     # three slabs, the last one short
    (46, 64, 9, 5, 1, 0, 0, False),      # whole lines in FP64, FP32 and FP16, y and z walls
    (47, 32, 4, 33, 1, 1, 1, False),     # whole lines in FP64 and FP32, no walls
    (48, 21, 7, 30, 1, 1, 0, False),     # z walls alone, ragged
]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("seed,nx,ny,nz,px,py,pz,ef", CASES)
def test_step_matches_oracle(seed, nx, ny, nz, px, py, pz, ef, storage):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle.oracle3 as O3
    from paper_1505_02976_amd import lbm3d
    cfg = W.random_case3d(seed, nx, ny, nz, periodic_z=pz, storage=storage, eps_field=ef, periodic_x=px, periodic_y=py)
    print(f"case: 3-D {storage} seed {seed} {nx}x{ny}x{nz}, walls {[w.get('kind') for w in cfg['walls']]}", flush=True)
    sim = lbm3d.Sim3(cfg)
    sim.step(STEPS)
    ref = O3.Oracle3(dict(cfg, storage="f64"))
    ref.step(STEPS)
    order = [tuple(int(v) for v in c) for c in O3.lattice()[0]]
    perm = [order.index(c) for c in lbm3d.lattice()]
    rest = [1.0] + [0.0] * 18
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12) * cfg["sigma"] * 0.5 * (cfg["T_hot"] + cfg["T_cold"])
    dev = [r[perm].reshape(19, -1) - np.array(o)[:, None] for r, o in zip(ref.populations(), (rest, w))]
    scale = max(float(np.abs(d).max()) for d in dev) if storage != "f64" else 1.0
    for a, b in zip(sim.populations(), ref.populations()):
        assert float(np.abs(a.cpu().numpy() - b[perm]).max()) < TOL[storage] * scale
