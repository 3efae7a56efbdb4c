// Pinned host memory for the few numbers a read-out returns: the reduction's last block writes
// them there, and the call has only to wait for the stream.  A copy of them from device memory
// takes 9.5 us of a call of 25 us.  A context takes one slot for its lifetime; the slots are one
// allocation of 64 KiB, made by the first context of the process (the next one where that
// failed) and held until the process ends.  A context that finds none left copies.
#pragma once

namespace lbm {

constexpr int HOST_SLOTS = 1024, HOST_SLOT_BYTES = 64;

double *host_slot_take();          // NULL: none left; any thread
void host_slot_give(double *slot);

}  // namespace lbm
