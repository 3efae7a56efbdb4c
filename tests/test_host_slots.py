"""The pinned result slots on error paths and in odd orders, on a stand-in for the HIP runtime."""
from hip_calls import run

BATCH = r"""
take = lib._ZN3lbm14host_slot_takeEv       # lbm::host_slot_take()
take.restype = C.c_void_p
cfgs = [W.cavity(12), W.cavity(40), W.cavity(16)]
failed = 0
while True:
    calls.calls_fail_copy(failed)          # the copies of lbm_batch_init, one after the other
    try:
        b = Batch(cfgs)
    except lbm.LbmError:
        failed += 1
        continue
    break
calls.calls_fail_copy(-1)
lib.lbm_batch_destroy(b.h)
free = 0
while take():
    free += 1
print(failed, free)
assert failed > 3 and free == 1024, (failed, free)
"""

INIT = r"""
# a failed allocation is not the last one, and no allocation can disturb a stream capture
calls.calls_fail_alloc(0)
for i in range(3):
    log()
    s = Sim(W.cavity(12))
    allocs = [c for c in log() if c.startswith("host alloc")]
    assert allocs == (["host alloc 2"] if i < 2 else []), (i, allocs)
    assert calls.calls_mode() == 0
"""


def test_failed_batches_give_their_slots_back(tmp_path):
    run(BATCH, tmp_path)


def test_slots_are_allocated_outside_captures_and_tried_again(tmp_path):
    run(INIT, tmp_path)
