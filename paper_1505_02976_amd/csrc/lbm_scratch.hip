// Device-resident scratch for the entry point that allocates nothing (lbm_residual_noalloc):
// one file-scope array per device, held until the process ends.  Host code never uses the
// array's name as an address (in host code it is only a stand-in for the device symbol):
// each device's address is looked up once, with that device current, and kept.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/lbm.h"
#include "lbm_hostslot.h"
#include "lbm_kernels.h"

namespace lbm {

static __device__ __align__(256) unsigned char scratch[LBM_STATIC_SCRATCH_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_lock;
void *g_addr[MAX_DEVICES];
bool g_looked_up[MAX_DEVICES];
hipError_t g_status[MAX_DEVICES];

}  // namespace

hipError_t static_scratch_setup(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_lock);
    if (g_looked_up[device]) return g_status[device];
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != device) e = hipErrorInvalidDevice;   // the caller makes it current
    void *ptr = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_addr[device] = e == hipSuccess ? ptr : nullptr;
    g_status[device] = e;
    g_looked_up[device] = true;
    return e;
}

void *static_scratch(int device)
{
    if (device < 0 || device >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> guard(g_lock);
    return g_looked_up[device] ? g_addr[device] : nullptr;
}

namespace {

// Plain arrays: nothing to construct, to run out of or to destroy before the last context.
std::mutex g_slot_lock;
bool g_slots_made;
double *g_slot_free[HOST_SLOTS];
int g_slots_free;

}  // namespace

double *host_slot_take()
{
    std::lock_guard<std::mutex> guard(g_slot_lock);
    if (!g_slots_made) {
        // the allocation would invalidate a stream capture that is under way elsewhere in the process
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        void *p = nullptr;
        g_slots_made =
            hipHostMalloc(&p, (size_t)HOST_SLOTS * HOST_SLOT_BYTES, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess;
        if (g_slots_made)
            for (int i = HOST_SLOTS - 1; i >= 0; --i)
                g_slot_free[g_slots_free++] = reinterpret_cast<double *>(static_cast<char *>(p) + (size_t)i * HOST_SLOT_BYTES);
        else
            (void)hipGetLastError();
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    return g_slots_free > 0 ? g_slot_free[--g_slots_free] : nullptr;
}

void host_slot_give(double *s)
{
    if (!s) return;
    std::lock_guard<std::mutex> guard(g_slot_lock);
    g_slot_free[g_slots_free++] = s;
}

}  // namespace lbm
