// Results from device memory into a caller's pageable arrays.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace vplbm {

// A copy straight into pageable memory runs at 10.8 GB/s (4.4 without huge pages), bound by one thread
// that faults the pages in and copies, against 57 GB/s over the link into pinned memory.  Here up to
// eight threads each take chunks through two pinned slots of their own, one on the link while the
// other is copied out.  402 MB: 38.6 -> 10.5 ms (95 -> 18); 43 MB: 4.2 -> 1.5 ms; 1 MB: 0.49 -> 0.07 ms.
// The other direction gains nothing (the pages are there): 30 GB/s, against 40.
//
// An object serves one call at a time (as a handle does), several objects several at once.  The pinned
// memory, at most 32 MB a call, is shared: it is allocated where a copy finds none idle, and goes with the
// last object of the process.
class HostCopy {
public:
    HostCopy();
    ~HostCopy();
    HostCopy(const HostCopy &) = delete;
    HostCopy &operator=(const HostCopy &) = delete;

    // n bytes from dev + i * n to dst[i], for each dst[i] that is not null (parts of them), after the
    // work before it on the stream; done when it returns hipSuccess.
    hipError_t read(hipStream_t st, const void *dev, size_t n, void *const *dst, int parts);
};

// memcpy between host arrays, by several threads where that is worth their start.
void host_copy(void *dst, const void *src, size_t n);

}  // namespace vplbm
