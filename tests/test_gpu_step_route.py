"""Calls of few steps and the steps left over from full launches on tiles, which go by passes and single
steps in between: bit for bit the single steps, in any order of calls, alone and in a batch."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CALLS = (1, 4, 2, 3, 5, 7, 6, 1, 9)


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm
    lbm.lib()
    return lbm


@pytest.mark.parametrize("storage,nx,ny,px,py,extra", [
    ("f64", 500, 507, 0, 0, {}), ("f64", 1150, 957, 1, 0, {"eps_field": True}), ("f64", 27777, 36, 0, 0, {"eps_field": True}),
    ("f32", 640, 647, 0, 1, {}), ("f32", 1250, 1257, 0, 0, {"moving_walls": True}), ("f32", 2100, 1601, 0, 0, {"with_Q": True}),
    ("f32", 30303, 33, 0, 0, {}), ("f32", 160, 8000, 0, 0, {"eps_field": True}),
    ("f16", 850, 857, 0, 0, {}), ("f16", 1250, 1257, 1, 1, {"eps_field": True}), ("f16", 100, 11000, 0, 0, {}),
])
def test_calls_are_bitwise_single_steps(gpu, storage, nx, ny, px, py, extra):
    cfg = W.random_case(95, nx, ny, periodic_x=px, periodic_y=py, storage=storage, **extra)
    print(f"case: {storage} {nx} x {ny} p{px}{py}", flush=True)
    a = gpu.Sim(cfg)
    b = gpu.Sim(cfg)
    b.fusion = 1
    for n in CALLS:
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        assert bool((sa == sb).all()), (n, float((sa - sb).abs().max()))
    assert a.time == b.time == sum(CALLS)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_batch_calls_are_bitwise_single_steps(gpu, storage):
    cfgs = [W.random_case(96 + k, 400 + 37 * k, 517 - 20 * k, storage=storage, eps_field=k == 2) for k in range(8)]
    print(f"case: batch of {len(cfgs)}, {storage}", flush=True)
    a, b = gpu.Batch(cfgs), gpu.Batch(cfgs)
    b.fusion = 1
    for n in CALLS:
        a.step(n)
        b.step(n)
        for k in range(len(cfgs)):
            sa, sb = a[k].get_state(), b[k].get_state()
            assert bool((sa == sb).all()), (n, k, float((sa - sb).abs().max()))
    assert a[0].time == b[0].time == sum(CALLS)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_gradient_with_left_over_states(gpu, storage):
    """The adjoint's forward states come from the same launches: with and without tiles the value and
    the gradient agree bit for bit."""
    import torch
    cfg = W.random_case(99, 640, 1150, storage=storage, eps_field=True)
    cfg["walls"] = [dict(w, kind="T") if k < 2 else w for k, w in enumerate(cfg["walls"])]
    out = []
    for fusion in (0, 1):
        sim = gpu.Sim(cfg)
        if fusion:
            sim.fusion = 1
        adj = gpu.Adjoint(sim, 11, wall=0)
        out.append((adj.value, adj.gradient()))
    assert out[0][0] == out[1][0] and bool((out[0][1] == out[1][1]).all()) and bool(torch.isfinite(out[0][1]).all())
