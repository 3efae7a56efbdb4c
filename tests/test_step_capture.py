"""Calls of lbm_step and lbm_batch_step that are captured into a graph, on a stand-in for the HIP
runtime: two steps and more leave the state in the buffer they started from (an even number of launches
and passes, each of which changes the buffer), so that a replay goes on where the last one ended."""
import pytest

from hip_calls import run

SCRIPT = r"""
s = {make}
def changes(names):
    one = sum(n in ("launch k_step_bulk", "launch k_batch_edge") for n in names)     # one of each per step
    two = sum(n in ("launch k_step2_rows", "launch k_batch_step2_rows") for n in names)
    return sum("tile" in n for n in names) + one + two
plain = {{n: s.step(n) for n in range(1, 42)}}
calls.calls_capturing(1)
for n in range(2, 42):
    names = s.step(n)
    assert changes(names) % 2 == 0, (n, names)
    assert len(names) - len(plain[n]) in (0, 1), (n, names, plain[n])
assert s.step(1) == plain[1]
"""


@pytest.mark.parametrize("make", [
    "Sim(dict(W.cavity(20), T_init=None))",
    "Sim(dict(W.cavity(128), T_init=None))",
    "Sim(dict(W.cavity(128, storage='f16'), T_init=None))",
    "Sim(dict(W.cavity(40, nx=640, ny=560, storage='f32'), T_init=None))",
    "Batch([dict(W.cavity(64, storage='f32'), T_init=None) for _ in range(3)])",
    "Batch([dict(W.cavity(64, storage='f16'), T_init=None) for _ in range(3)])",
])
def test_captured_calls_end_where_they_began(tmp_path, make):
    run(SCRIPT.format(make=make), tmp_path)
