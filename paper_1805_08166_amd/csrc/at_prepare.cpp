// What a kernel needs before its first launch on a device.
#include "at_internal.h"

namespace at {

hipError_t prepare_kernel(const void* fn, int64_t static_lds, size_t dynamic_lds, std::atomic<uint64_t>& done) {
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const uint64_t bit = device < 64 ? (uint64_t)1 << device : 0;
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    if (static_lds >= 0) {
        hipFuncAttributes fa;
        if ((e = hipFuncGetAttributes(&fa, fn)) != hipSuccess) return e;
        if ((int64_t)fa.sharedSizeBytes != static_lds) return hipErrorInvalidKernelFile;
    }
    if (dynamic_lds > 0 &&
        (e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dynamic_lds)) != hipSuccess)
        return e;
    done.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

}  // namespace at
