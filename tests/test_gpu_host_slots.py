"""Results through the pinned slots: more contexts alive than there are slots (the later ones
copy), all reading out the same values, bit for bit, in two and three dimensions; slots given back are
used again.  And the fields of a small grid, which share one allocation: the values of a grid above
the bound, and separate memory."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SLOTS = 1024


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1505_02976_amd import lbm
    lbm.lib()
    return lbm


def test_more_contexts_than_slots(gpu):
    from paper_1505_02976_amd import lbm3d
    cfg = W.random_case(81, 6, 5)
    cfg["walls"] = [dict(w, kind="T") for w in cfg["walls"]]
    cfg3 = W.random_case3d(82, 4, 4, 4, periodic_x=0)

    def values(n):
        sims = [gpu.Sim(cfg) for _ in range(n)]
        s3 = [lbm3d.Sim3(cfg3) for _ in range(20)]
        for s in sims:
            assert s.residual() == (None, None)
            s.step(2)
        for s in s3:
            s.step(2)
        return [(s.residual(), s.nusselt(0), s.nusselt(3)) for s in sims], [s.nusselt(2) for s in s3]

    for n in (SLOTS + 30, 3):
        print(f"case: {n} contexts of 6 x 5 and 20 of 4 x 4 x 4", flush=True)
        a, b = values(n)
        assert len(set(a)) == 1 and len(set(b)) == 1
        if n > SLOTS:
            first = (a[0], b[0])
        assert (a[0], b[0]) == first


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("ny", [128, 129])          # 131,072 nodes and more
def test_fields_have_their_own_memory(gpu, ny, f32):
    cfg = W.random_case(83, 1024, ny, moving_walls=True)
    sim = gpu.Sim(cfg)
    sim.step(3)
    a = sim.fields(f32=f32)
    ends = sorted((v.data_ptr(), v.data_ptr() + v.numel() * v.element_size()) for v in a.values())
    assert len(a) == 9 and all(v.is_contiguous() and v.shape == (ny, 1024) for v in a.values())
    assert all(e[1] <= b[0] for e, b in zip(ends, ends[1:]))
    b = sim.fields(f32=f32, gradients=False)
    assert sorted(b) == ["T", "p", "ux", "uy"]
    for k in b:
        assert bool((a[k] == b[k]).all())
