// Host-side process state of the library: the once-per-(kernel, device) raising of the dynamic-LDS limit and
// the explicit set-up call behind meteora_init.
#include <mutex>

#include "common.hpp"
#include "kernels.hpp"

namespace meteora {

namespace {
constexpr int kMaxDevices = 64;
// Places by the kernel's address, the next free one where that is taken.  Those that gemm_init_kernels and the others list are about
// 90: as a list, walked to its end on every launch, they took 64 ns, so 13 (host alone).
constexpr int kLdsBits = 9, kMaxKernels = 1 << kLdsBits;
struct LdsEntry { const void* kernel; uint64_t done; };   // bit d: the limit is set on device d
LdsEntry g_lds[kMaxKernels];
std::mutex g_lds_mutex;
}  // namespace

// Kernels with more than 64 KB of dynamic LDS need the limit raised by a host-side attribute, which HIP keeps
// per device.  The first launch of a kernel on a device does it (or init_kernels below, ahead of time); the
// table is guarded by a mutex so that threads launching on different streams do not race on it.
hipError_t ensure_lds_limit(const void* kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_lds_mutex);
    LdsEntry* ent = nullptr;
    uint32_t place = (uint32_t)(reinterpret_cast<uintptr_t>(kernel) >> 3) * 0x9e3779b1u >> (32 - kLdsBits);
    for (int i = 0; i < kMaxKernels && ent == nullptr; ++i, place = (place + 1) % kMaxKernels)
        if (g_lds[place].kernel == kernel || g_lds[place].kernel == nullptr) ent = &g_lds[place];
    if (ent == nullptr) return hipErrorOutOfMemory;
    ent->kernel = kernel;
    if (ent->done >> dev & 1) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) ent->done |= 1ull << dev;
    return e;
}

// Everything a first launch would set up lazily, for the current device.
hipError_t init_kernels() {
    hipError_t e = gemm_init_kernels();
    if (e != hipSuccess) return e;
    e = gemm_decode_init_kernels();
    if (e != hipSuccess) return e;
    e = gate_init_kernels();
    if (e != hipSuccess) return e;
    e = shrink_init_kernels();
    if (e != hipSuccess) return e;
    e = gate_bwd_init_kernels();
    if (e != hipSuccess) return e;
    return bucket_init_scratch();
}

}  // namespace meteora
