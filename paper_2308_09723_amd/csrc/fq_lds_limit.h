// Dynamic LDS above the default limit, for every launcher.
#ifndef FQ_LDS_LIMIT_H_
#define FQ_LDS_LIMIT_H_

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

#include "../../include/fq.h"

namespace fqd {

// Kernels that need more than the default 64 KiB of dynamic LDS have their limit raised to the
// 160 KiB of a compute unit, once per (kernel instantiation, device): `done` holds one bit per device.
inline int raise_lds_limit(const void* kern, std::atomic<uint64_t>& done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return FQ_ERR_HIP;
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return FQ_OK;
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
        return FQ_ERR_HIP;
    done.fetch_or(bit, std::memory_order_release);
    return FQ_OK;
}

}  // namespace fqd

#endif  // FQ_LDS_LIMIT_H_
