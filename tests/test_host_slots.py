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


def test_failed_batches_give_their_slots_back(tmp_path):
    run(BATCH, tmp_path)
