"""Several steps per launch on LDS-resident tiles (the default of lbm_step on grids that are
not large) against single steps, bit for bit: every node update is the one-step node code
with the same inputs, so any difference is an indexing or boundary error.  The grids lie at
the edges of the path's ranges: one block for the whole grid (at most 512 nodes, the periodic
directions wrapping inside it), one tile across a narrow direction (walled or periodic, down
to the fewest nodes a direction may have), tiles of uneven size, halos that reach past walls
and around a periodic direction, and the storage types' largest grids."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm
    lbm.lib()
    return lbm


CASES = [
    # one block
    (1, 16, 32, 0, 0, {"moving_walls": True, "with_Q": True}),
    (2, 23, 22, 1, 1, {"eps_field": True}),
    (3, 1, 300, 1, 0, {}),
    (4, 5, 64, 1, 0, {"moving_walls": True, "eps_field": True}),
    (5, 102, 5, 0, 1, {"with_Q": True}),
    (6, 4, 4, 0, 0, {"moving_walls": True}),
    # just above one block
    (7, 19, 27, 0, 0, {"eps_field": True, "moving_walls": True}),
    (8, 513, 1, 1, 1, {}),
    # one tile across a direction
    (9, 7, 900, 1, 0, {"eps_field": True}),
    (10, 4, 777, 0, 0, {"moving_walls": True}),
    (11, 1001, 6, 0, 1, {"with_Q": True}),
    # tiles in both directions, uneven
    (12, 61, 47, 0, 0, {"moving_walls": True, "eps_field": True, "with_Q": True}),
    (13, 130, 33, 1, 1, {"eps_field": True}),
    (14, 97, 211, 1, 0, {"moving_walls": True}),
    (15, 250, 250, 0, 0, {}),
    (16, 401, 307, 0, 1, {"eps_field": True}),
    (17, 905, 1101, 0, 0, {"moving_walls": True}),
]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("seed,nx,ny,px,py,extra", CASES, ids=[f"{c[1]}x{c[2]}-p{c[3]}{c[4]}" for c in CASES])
def test_tile_steps_are_bitwise_single_steps(gpu, storage, seed, nx, ny, px, py, extra):
    cfg = W.random_case(500 + seed, nx, ny, periodic_x=px, periodic_y=py, storage=storage, **extra)
    print(f"case: {storage} {nx} x {ny} p{px}{py}", flush=True)
    a = gpu.Sim(cfg)
    b = gpu.Sim(cfg)
    b.fusion = 1
    for n in (1, 2, 7, 30):
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        assert bool((sa == sb).all()), (n, float((sa - sb).abs().max()))
    assert a.time == b.time == 40


def test_three_isothermal_nodes_across(gpu):
    """The narrowest walled direction (three nodes, isothermal walls) beside a long one."""
    cfg = W.random_case(530, 3, 600, storage="f64", moving_walls=True)
    cfg["walls"] = [dict(w, kind="T") for w in cfg["walls"]]
    a, b = gpu.Sim(cfg), gpu.Sim(cfg)
    b.fusion = 1
    a.step(29)
    b.step(29)
    assert bool((a.get_state() == b.get_state()).all())


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_batched_tiles_are_bitwise_single_steps(gpu, storage):
    """A batch of uneven grids (with and without a porosity field, walled and periodic, one
    narrower than a tile), and one whose grids are all a single block."""
    mixed = [W.random_case(541, 61, 47, storage=storage, eps_field=True, moving_walls=True),
             W.random_case(542, 6, 200, periodic_x=1, storage=storage),
             W.random_case(543, 130, 33, periodic_x=1, periodic_y=1, storage=storage, with_Q=True),
             W.random_case(544, 20, 19, storage=storage, moving_walls=True)]
    blocks = [W.random_case(545, 16, 32, storage=storage), W.random_case(546, 9, 8, periodic_y=1, storage=storage)]
    for cfgs in (mixed, blocks):
        print(f"case: {storage} batch of {len(cfgs)}", flush=True)
        batch = gpu.Batch(cfgs)
        singles = [gpu.Sim(c) for c in cfgs]
        for s in singles:
            s.fusion = 1
        for n in (1, 5, 23):
            batch.step(n)
            for k, s in enumerate(singles):
                s.step(n)
                assert bool((batch[k].get_state() == s.get_state()).all()), (k, n)
