"""The adjoint's tiles against the oracle: the gradient along a random direction equals the
oracle's complex-step derivative along it (one oracle run per grid).  The grids have several
tiles, of uneven sizes and with remainders; tiles beside walls and periodic edges; tiles whose
halo ends within two nodes of a wall (their side is moved to it); a direction one tile wide;
more steps than a launch takes, in several segments."""
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


@pytest.mark.parametrize("seed,nx,ny,px,py,wall,extra", [
    (61, 61, 47, 0, 0, 0, {"moving_walls": True, "with_Q": True}),
    (62, 45, 38, 0, 0, 3, {"moving_walls": True}),
    (63, 130, 33, 1, 0, 2, {"with_Q": True}),
    (64, 34, 70, 0, 1, 1, {}),
    (65, 5, 120, 0, 0, 0, {"moving_walls": True}),
], ids=lambda v: str(v) if isinstance(v, int) else "")
def test_directional_derivative(gpu, oracle_mod, seed, nx, ny, px, py, wall, extra):
    cfg = W.random_case(seed, nx, ny, periodic_x=px, periodic_y=py, **extra)
    for k in ("p_init", "ux_init", "uy_init"):
        cfg.pop(k)
    rng = np.random.default_rng(seed)
    eps = 0.65 + W.smooth_field(nx, ny, rng, 0.2)
    d = rng.uniform(-1, 1, size=(ny, nx))
    steps = 31
    o = oracle_mod.Oracle(dict(cfg, eps_field=eps + 1e-30j * d), complex_step=True)
    o.step(steps)
    v = o.nusselt(wall)
    print(f"case: {nx} x {ny} p{px}{py} wall {wall}", flush=True)
    adj = gpu.Adjoint(gpu.Sim(dict(cfg, eps_field=eps, storage="f64")), steps, wall)
    g = adj.gradient().cpu().numpy()
    got, ref = float(np.sum(g * d)), v.imag / 1e-30
    scale = float(np.sum(np.abs(g * d)))          # the terms' own size: cancellation counts
    assert abs(adj.value - v.real) < 1e-11
    assert abs(got - ref) < 1e-10 * scale, (got, ref, scale)
