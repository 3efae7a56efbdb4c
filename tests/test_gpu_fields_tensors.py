"""The fields of a small grid are tensors of their own: an in-place change of one, an in-place product
with a tensor that needs a gradient, and a saved file concern that field alone, on grids of every
size."""
import io

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


@pytest.mark.parametrize("nx,ny", [(24, 17), (512, 257)])        # below and above 131,072 nodes
def test_fields_are_tensors_of_their_own(gpu, nx, ny):
    import torch
    sim = gpu.Sim(W.random_case(84, nx, ny))
    sim.step(2)
    print(f"case: fields of {nx} x {ny}", flush=True)
    f = sim.fields()
    assert len({v.untyped_storage().data_ptr() for v in f.values()}) == 9
    for v in f.values():
        assert not v._is_view() and v.untyped_storage().nbytes() == v.numel() * v.element_size()
    w = torch.ones_like(f["T"], requires_grad=True)
    f["T"].mul_(w)
    w = torch.ones_like(f["ux"], requires_grad=True)
    loss = (w * f["ux"]).sum()          # saves ux
    f["p"].add_(1.0)
    loss.backward()
    assert bool((w.grad == f["ux"]).all())
    file = io.BytesIO()
    torch.save(f["uy"], file)
    assert file.getbuffer().nbytes < 2 * f["uy"].numel() * 8 + 16384
