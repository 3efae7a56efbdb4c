"""How many steps of a call go by launches on tiles and what takes the rest, on a stand-in for the HIP
runtime: equal launches of as many steps as pay, then two-step passes and single steps."""
import pytest

from hip_calls import run

SCRIPT = r"""
def kinds(calls):
    names = [c[7:] for c in calls if c.startswith("launch")]
    return sum("tile" in n for n in names), sum("step2" in n and "rows" not in n for n in names), sum(n in {singles!r} for n in names)
s = {make}
for n, want in {cases!r}:
    got = kinds(s.step(n))
    assert got == want, (n, got)
"""
STEPS = ("k_step_bulk", "k_step_edge")
BATCH = ("k_batch_edge", "k_batch_wall", "k_batch_bulk")


@pytest.mark.parametrize("make,cases", [
    # up to three steps a launch, two and three pay; a pass is two launches besides the walled rows, a step two
    ("Sim(dict(W.cavity(40, nx=640, ny=560), T_init=None))", [(1, (0, 0, 2)), (2, (1, 0, 0)), (4, (2, 0, 0)), (7, (3, 0, 0))]),
    # up to four, three and four pay
    ("Sim(dict(W.cavity(40, nx=1250, ny=1257, storage='f32'), T_init=None))",
     [(1, (0, 0, 2)), (2, (0, 2, 0)), (3, (1, 0, 0)), (4, (1, 0, 0)), (5, (1, 0, 2)), (6, (2, 0, 0)), (40, (10, 0, 0))]),
    # FP16: three, single steps besides
    ("Sim(dict(W.cavity(40, nx=1250, ny=1257, storage='f16'), T_init=None))", [(1, (0, 0, 2)), (2, (0, 0, 4)), (5, (1, 0, 4)), (7, (2, 0, 2))]),
    # any number pays
    ("Sim(dict(W.cavity(128), T_init=None))", [(1, (1, 0, 0)), (2, (1, 0, 0))]),
])
def test_steps_of_a_call(tmp_path, make, cases):
    run(SCRIPT.format(make=make, cases=cases, singles=STEPS), tmp_path)


def test_steps_of_a_batch(tmp_path):
    make = "Batch([dict(W.cavity(40, nx=500, ny=503, storage='f32'), T_init=None) for _ in range(6)])"
    log = run("b = " + make + "\nfor n in (1, 2, 3, 4, 5): print([c[7:] for c in b.step(n) if c.startswith('launch')])", tmp_path)
    lines = log.split("\n")
    assert "k_batch_tile" not in lines[0] and "k_batch_tile" not in lines[1] and "step2" in lines[1]
    assert lines[2] == lines[3] == "['k_batch_tile']"
    assert lines[4].startswith("['k_batch_tile', ") and lines[4].count("k_batch_tile") == 1
