"""Larger grids on LDS-resident tiles, where the shapes of the tiles and, in FP64, the kernel
change, against single steps, bit for bit (the same node code with the same inputs): both sides
of 120,000, 350,000 and 700,000 nodes, a long narrow grid of that size, uneven tiles, walls and
periodic directions, with and without a porosity field, and batches on both sides of 700,000
nodes."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    (1, 346, 346, 0, 0, {"moving_walls": True}),                     # 119,716
    (2, 347, 347, 0, 0, {"eps_field": True, "moving_walls": True}),  # 120,409
    (3, 593, 591, 0, 1, {"with_Q": True}),                           # 350,463
    (4, 833, 841, 0, 0, {"eps_field": True, "moving_walls": True}),  # 700,553
    (5, 1301, 547, 1, 0, {"moving_walls": True}),                    # 711,647
    (6, 47, 15000, 0, 0, {"eps_field": True}),                       # narrow, 705,000
    (7, 1009, 1201, 1, 1, {"eps_field": True}),
]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm
    lbm.lib()
    return lbm


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("seed,nx,ny,px,py,extra", CASES, ids=[f"{c[1]}x{c[2]}" for c in CASES])
def test_large_tiles_are_bitwise_single_steps(gpu, storage, seed, nx, ny, px, py, extra):
    cfg = W.random_case(600 + seed, nx, ny, periodic_x=px, periodic_y=py, storage=storage, **extra)
    print(f"case: {storage} {nx} x {ny}", flush=True)
    a, b = gpu.Sim(cfg), gpu.Sim(cfg)
    b.fusion = 1
    for n in (1, 7):
        a.step(n)
        b.step(n)
        assert bool((a.get_state() == b.get_state()).all()), n


@pytest.mark.parametrize("count,eps_field", [(5, True), (9, False), (9, True)])   # 0.4 and 0.71 M nodes
def test_large_batches_are_bitwise_single_steps(gpu, count, eps_field):
    cfgs = [W.random_case(620 + k, 260 + 5 * k, 301 - 4 * k, storage="f64", eps_field=eps_field, moving_walls=True)
            for k in range(count)]
    print(f"case: f64 batch of {count}, {sum(c['nx'] * c['ny'] for c in cfgs)} nodes", flush=True)
    batch = gpu.Batch(cfgs)
    batch.step(7)
    for k, c in enumerate(cfgs):
        s = gpu.Sim(c)
        s.fusion = 1
        s.step(7)
        assert bool((batch[k].get_state() == s.get_state()).all()), k
