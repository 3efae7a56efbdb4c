"""Steps captured into a graph and replayed, with eager work and synchronizations between the replays:
every replay goes on where the last one ended, bit for bit the same calls made eagerly."""
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


def _replays(torch, stream, sims, states, n):
    a, b = sims
    a.step(n)                       # the side stream of the passes is made outside the capture
    b.step(n)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(n)
    for r in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        b.step(n)
        torch.cuda.synchronize()
        x, y = states(a), states(b)
        assert all(bool((p == q).all()) for p, q in zip(x, y)), (n, r)
        torch.ones(1000, device="cuda").sum().item()


@pytest.mark.parametrize("n", [4, 20, 50, 100])
@pytest.mark.parametrize("storage,nx,ny", [
    ("f64", 20, 20), ("f64", 128, 128), ("f32", 128, 120), ("f16", 128, 120), ("f32", 500, 507), ("f64", 1150, 957),
])
def test_replays_go_on(gpu, storage, nx, ny, n):
    import torch
    print(f"case: {storage} {nx} x {ny}, {n} steps", flush=True)
    stream = torch.cuda.Stream()
    cfg = W.random_case(101, nx, ny, storage=storage)
    with torch.cuda.stream(stream):
        sims = [gpu.Sim(cfg, stream=stream) for _ in range(2)]
    _replays(torch, stream, sims, lambda s: [s.get_state()], n)


@pytest.mark.parametrize("n", [4, 20, 50])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_replays_of_a_batch_go_on(gpu, storage, n):
    import torch
    print(f"case: batch {storage}, {n} steps", flush=True)
    stream = torch.cuda.Stream()
    cfgs = [W.random_case(102 + k, 60 + 40 * k, 90, storage=storage) for k in range(3)]
    with torch.cuda.stream(stream):
        sims = [gpu.Batch(cfgs, stream=stream) for _ in range(2)]
    _replays(torch, stream, sims, lambda s: [p.get_state() for p in s.problems], n)
