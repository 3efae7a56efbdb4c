"""Batches that hold problems with a porosity field beside problems of uniform porosity, against each
problem alone, bit for bit.  The uniform ones are chosen so that c0 = (1 + eps nu / (2 K)) / 2
rounds differently when the product is rounded first (the host's coefficients, which a problem
alone takes) and when it is fused with the sum (device code)."""
from fractions import Fraction

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# side, Da, eps
UNIFORM = [(32, 1e-6, 0.4), (32, 1e-6, 0.6), (41, 1e-6, 0.7), (48, 1e-6, 0.8), (41, 1e-5, 0.4)]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm
    lbm.lib()
    return lbm


@pytest.mark.parametrize("n", [21, 64])        # the field problem's side: 441 nodes, or several tiles
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_mixed_batch_is_bitwise_the_problems_alone(gpu, storage, n):
    cfgs = [W.cavity(m, Da=Da, eps=eps, storage=storage) for m, Da, eps in UNIFORM]
    for c in cfgs:
        d = gpu.derived(c)
        h, r = 0.5 * c["eps"], d["nu"] / d["K"]
        assert 0.5 * (1.0 + h * r) != 0.5 * float(Fraction(h) * Fraction(r) + 1)
    cfgs.insert(2, W.random_case(25, n, n, storage=storage, eps_field=True))
    print(f"case: {storage}, {len(UNIFORM)} uniform problems and a field of {n} x {n}", flush=True)
    batch = gpu.Batch(cfgs)
    alone = [gpu.Sim(c) for c in cfgs]
    for steps in (1, 2, 13):
        batch.step(steps)
        for k, s in enumerate(alone):
            s.step(steps)
            a, b = batch[k].get_state(), s.get_state()
            assert bool((a == b).all()), (steps, k, float((a - b).abs().max()))
