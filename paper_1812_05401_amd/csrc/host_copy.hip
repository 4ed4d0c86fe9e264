#include "host_copy.hpp"

#include <string.h>

#include <algorithm>
#include <atomic>

#include "side_by_side.hpp"

namespace vplbm {

namespace {

int most_threads()
{
    const int n = (int)std::thread::hardware_concurrency();
    return n < 1 ? 1 : n;
}

}  // namespace

HostCopy::~HostCopy()
{
    for (hipEvent_t e : event_)
        if (e) (void)hipEventDestroy(e);
    if (pinned_) (void)hipHostFree(pinned_);
}

bool HostCopy::prepare(size_t bytes, int slots)
{
    for (int i = 0; i < slots; i++)
        if (!event_[i] && hipEventCreateWithFlags(&event_[i], hipEventDisableTiming) != hipSuccess) {
            event_[i] = nullptr;
            (void)hipGetLastError();
            return false;
        }
    if (bytes_ >= bytes) return true;
    if (pinned_) (void)hipHostFree(pinned_);
    pinned_ = nullptr;
    bytes_ = 0;
    if (hipHostMalloc((void **)&pinned_, bytes, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        pinned_ = nullptr;
        return false;
    }
    bytes_ = bytes;
    return true;
}

hipError_t HostCopy::read(hipStream_t st, const void *dev, size_t n, void *const *dst, int parts)
{
    const char *src = static_cast<const char *>(dev);
    const size_t total = n * parts;
    // us, fresh pages, 1 / 2 / 4 / 8 threads: 1 MB 70 / 79 / 74 / 108 (512 KB slots); 4 MB 223 / 233 / 238 / 245
    // and 642 / 457 / 396 / 336 without huge pages; 16 MB 1210 / 758 / 661 / 664 (1 MB slots), 1040 / 820 / 658 /
    // 611 (2 MB), 850 / 784 / 793 / 799 (512 KB).  A copy on the link takes about 18 us besides its bytes, so
    // slots are large where there are enough of them; but a pinned megabyte costs 50 us when it is first
    // used (18.9 MB of fields for the first time 2.8 ms with 32 MB of slots), so few where one copy is short.
    const size_t slot = total < ((size_t)8 << 20) ? (size_t)512 << 10 : total < ((size_t)64 << 20) ? (size_t)1 << 20 : (size_t)2 << 20;
    const size_t chunks = (total + slot - 1) / slot;
    const int want = total < ((size_t)2 << 20) ? 1 : total < ((size_t)64 << 20) ? 4 : kThreads;
    const int threads = (int)std::min<size_t>(std::min(want, most_threads()), chunks);
    // short copies are as quick straight; pinned and device destinations are quicker so; hipStreamPerThread
    // names another stream in each of the threads, which would not wait for the caller's work
    bool staged = total >= ((size_t)64 << 10) && st != hipStreamPerThread;
    for (int i = 0; i < parts && staged; i++) {
        if (!dst[i]) continue;
        hipPointerAttribute_t attr{};
        if (hipPointerGetAttributes(&attr, dst[i]) == hipSuccess) staged = attr.type == hipMemoryTypeUnregistered;
        else (void)hipGetLastError();
    }
    int device = 0;
    if (staged) staged = hipGetDevice(&device) == hipSuccess && prepare(2 * threads * std::min(slot, total), 2 * threads);
    if (!staged) {
        for (int i = 0; i < parts; i++)
            if (dst[i]) {
                const hipError_t e = hipMemcpyAsync(dst[i], src + i * n, n, hipMemcpyDeviceToHost, st);
                if (e != hipSuccess) return e;
            }
        return hipStreamSynchronize(st);
    }
    auto length = [&](size_t c) { return std::min(slot, total - c * slot); };
    // chunk c from its slot to the parts it lies in
    auto deliver = [&](size_t c, const char *from) {
        size_t at = c * slot, left = length(c);
        while (left > 0) {
            const size_t part = at / n, off = at - part * n, len = std::min(left, n - off);
            if (dst[part]) memcpy(static_cast<char *>(dst[part]) + off, from, len);
            from += len;
            at += len;
            left -= len;
        }
    };
    auto wanted = [&](size_t c) {
        for (size_t part = c * slot / n; part < (size_t)parts && part * n < c * slot + length(c); part++)
            if (dst[part]) return true;
        return false;
    };
    std::atomic<int> error{hipSuccess};
    side_by_side(threads, [&](int t) {
        hipError_t e = hipSetDevice(device);
        size_t held[2] = {chunks, chunks}, next = t;
        auto fetch = [&](int s) {
            while (next < chunks && !wanted(next)) next += threads;
            held[s] = next;
            if (next >= chunks || e != hipSuccess) return;
            e = hipMemcpyAsync(pinned_ + (2 * t + s) * std::min(slot, total), src + next * slot, length(next), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(event_[2 * t + s], st);
            next += threads;
        };
        fetch(0);
        fetch(1);
        for (int s = 0; held[s] < chunks && e == hipSuccess; s ^= 1) {
            e = hipEventSynchronize(event_[2 * t + s]);
            if (e != hipSuccess) break;
            deliver(held[s], pinned_ + (2 * t + s) * std::min(slot, total));
            fetch(s);
        }
        if (e != hipSuccess) error = e;
    });
    const hipError_t e = hipStreamSynchronize(st);   // no copy is under way when the slots are used again
    return error != hipSuccess ? (hipError_t)error.load() : e;
}

void host_copy(void *dst, const void *src, size_t n)
{
    // fresh pages: 4 GB/s by one thread
    const int threads = n < ((size_t)1 << 20) ? 1 : (int)std::min<size_t>(std::min(8, most_threads()), n >> 19);
    const size_t each = (n / threads + 4095) & ~(size_t)4095;
    side_by_side(threads, [&](int t) {
        const size_t at = std::min(n, t * each), end = t == threads - 1 ? n : std::min(n, at + each);
        if (end > at) memcpy(static_cast<char *>(dst) + at, static_cast<const char *>(src) + at, end - at);
    });
}

}  // namespace vplbm
