"""Which launches a batch steps with after its autotuner: the passes that the autotuner timed and
whose width it reports, as after lbm_batch_set_width and lbm_batch_set_fusion."""
import pytest

from hip_calls import run

SCRIPT = r"""
storage, call = {storage!r}, {call!r}
b = Batch([W.cavity(64, storage=storage) for _ in range(3)])
before = b.step(2)
assert before == ["launch k_batch_tile"], before
if call == "autotune":
    w = C.c_int32()
    lbm._check(lib.lbm_batch_autotune(b.h, 4, C.byref(w), None))
    timed = {{c for c in log() if c.startswith("launch")}}
    assert w.value in (64, 128, 256)
else:
    lbm._check(lib.lbm_batch_set_width(b.h, 128))
    timed = None
after = [c for c in b.step(2) if c.startswith("launch")]
assert after and "launch k_batch_tile" not in after, after
assert timed is None or set(after) == timed, (after, timed)
"""


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("call", ["autotune", "set_width"])
def test_passes_run_after_a_choice_of_width(tmp_path, storage, call):
    run(SCRIPT.format(storage=storage, call=call), tmp_path)
