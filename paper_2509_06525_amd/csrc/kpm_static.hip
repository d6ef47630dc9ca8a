// Static workspace of kpm_moments_noalloc: one array per GPU, part of a code object
// (no allocation call), shared by every call on that GPU.  It is this file's only
// device object: the runtime loads a file's code object when something in it is first
// used, so a process that never calls kpm_moments_noalloc holds none of it.
#include <mutex>

#include "common.hpp"
#include "kpm.hpp"

namespace tbk {

namespace {

constexpr int kScratchDevices = 64;
__device__ __align__(256) char scratch[kStaticBytes];
std::mutex g_scratch_mu;
void *g_scratch_ptr[kScratchDevices] = {};

}  // namespace

// The device address on the current device (never the array's name, a host-side stand-in).
tbk_status static_workspace(void **out) {
    int dev = -1;
    TBK_HIP(hipGetDevice(&dev));
    TBK_CHECK(dev >= 0 && dev < kScratchDevices, TBK_ERR_UNSUPPORTED, "device %d: no workspace slot", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        TBK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        TBK_CHECK(p != nullptr, TBK_ERR_DEVICE, "no device address for the static workspace");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TBK_OK;
}

}  // namespace tbk
