"""Grids of more than 65,000 tiles in a row of tiles: steps on tiles against single steps, bit for bit,
and the porosity gradient of a grid that repeats itself along x, which has to repeat as well (away
from the two end columns, whose weight in the average Nusselt number is one half)."""
import numpy as np
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


@pytest.mark.parametrize("storage,nx,ny,px,py,extra", [
    ("f64", 2163173, 1, 1, 1, {}),
    ("f32", 2163173, 1, 1, 1, {}),
    ("f16", 2163173, 1, 0, 1, {}),
    ("f64", 1829804, 2, 0, 1, {}),
    ("f32", 2400000, 5, 0, 0, {"eps_field": True}),
    ("f64", 2200000, 4, 1, 0, {"eps_field": True}),
])
def test_steps_are_bitwise_single_steps(gpu, storage, nx, ny, px, py, extra):
    cfg = W.random_case(91, nx, ny, periodic_x=px, periodic_y=py, storage=storage, **extra)
    print(f"case: {storage} {nx} x {ny} p{px}{py}", flush=True)
    a = gpu.Sim(cfg)
    b = gpu.Sim(cfg)
    b.fusion = 1
    for n in (1, 9):
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        assert bool((sa == sb).all()), (n, float((sa - sb).abs().max()))


def test_gradient_repeats(gpu):
    period, times, steps = 64, 25000, 6
    cfg = W.random_case(92, period, 4, periodic_x=1, eps_field=True)
    cfg["walls"] = [dict(w, kind="T") for w in cfg["walls"]]
    for k, v in cfg.items():
        if isinstance(v, np.ndarray):
            cfg[k] = np.tile(v.reshape(4, period), (1, times))
    cfg["nx"] = period * times
    print(f"case: gradient, f64 {period * times} x 4, {steps} steps", flush=True)
    adj = gpu.Adjoint(gpu.Sim(cfg), steps, wall=2)
    g = adj.gradient()
    one = g[:, period:2 * period]
    scale = float(one.abs().max())
    assert scale > 0.0
    full = one.repeat(1, times)
    k = 2 * steps          # the end columns' reach, on either side of the seam
    assert float((g - full)[:, k:-k].abs().max()) <= 1e-12 * scale
