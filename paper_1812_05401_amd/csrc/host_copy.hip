#include "host_copy.hpp"

#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <utility>

#include "side_by_side.hpp"

namespace vplbm {

namespace {

int most_threads()
{
    const int n = (int)std::thread::hardware_concurrency();
    return n < 1 ? 1 : n;
}

constexpr int kThreads = 8;

// Pinned slots, and the events of the copies into them, of one device: two per thread.
struct HostSlots {
    int device;
    char *pinned = nullptr;
    size_t bytes = 0;
    hipEvent_t event[2 * kThreads] = {};

    explicit HostSlots(int d) : device(d) {}
    ~HostSlots()
    {
        for (hipEvent_t e : event)
            if (e) (void)hipEventDestroy(e);
        if (pinned) (void)hipHostFree(pinned);
    }

    // room for n bytes and `slots` events; on the set's device
    bool prepare(size_t n, int slots)
    {
        for (int i = 0; i < slots; i++)
            if (!event[i] && hipEventCreateWithFlags(&event[i], hipEventDisableTiming) != hipSuccess) {
                event[i] = nullptr;
                (void)hipGetLastError();
                return false;
            }
        if (bytes >= n) return true;
        if (pinned) (void)hipHostFree(pinned);
        pinned = nullptr;
        bytes = 0;
        if (hipHostMalloc((void **)&pinned, n, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            pinned = nullptr;
            return false;
        }
        bytes = n;
        return true;
    }
};

// The sets that no read is using, for all objects of the process: a read takes one, or makes one where none
// is left, and waits for nobody.  As many as reads have run at once, at most kIdle, and none once the last
// object has gone.  (Each object kept its own once, 32 MB for good: a hundred handles held 3 GB.)
constexpr int kIdle = 8;
std::mutex g_mu;
HostSlots *g_idle[kIdle];
int g_nidle = 0, g_objects = 0;

HostSlots *take(int device)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (int i = g_nidle - 1; i >= 0; i--)
            if (g_idle[i]->device == device) {
                HostSlots *s = g_idle[i];
                g_idle[i] = g_idle[--g_nidle];
                return s;
            }
    }
    return new (std::nothrow) HostSlots(device);
}

void give(HostSlots *s)
{
    if (!s) return;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_nidle < kIdle) {
            g_idle[g_nidle++] = s;
            return;
        }
        // the larger ones stay
        for (HostSlots *&o : g_idle)
            if (o->bytes < s->bytes) std::swap(o, s);
    }
    delete s;
}

// The calling thread's device is this one (-1: its own) while this lives.
struct OnDevice {
    int before = -1;
    explicit OnDevice(int device)
    {
        int now = device;
        if (device >= 0 && hipGetDevice(&now) == hipSuccess && now != device && hipSetDevice(device) == hipSuccess) before = now;
    }
    ~OnDevice()
    {
        if (before >= 0) (void)hipSetDevice(before);
    }
};

}  // namespace

HostCopy::HostCopy()
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_objects++;
}

HostCopy::~HostCopy()
{
    HostSlots *last[kIdle];
    int n = 0;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (--g_objects == 0)
            while (g_nidle > 0) last[n++] = g_idle[--g_nidle];
    }
    while (n > 0) delete last[--n];
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
    int device = -1;                     // an event belongs to the stream's device, whichever is current
    if (staged && hipStreamGetDevice(st, &device) != hipSuccess) {
        (void)hipGetLastError();
        staged = false;
        device = -1;
    }
    const OnDevice on(device);
    HostSlots *const slots = staged ? take(device) : nullptr;
    if (!slots || !slots->prepare(2 * threads * std::min(slot, total), 2 * threads)) {
        give(slots);
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
            e = hipMemcpyAsync(slots->pinned + (2 * t + s) * std::min(slot, total), src + next * slot, length(next), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(slots->event[2 * t + s], st);
            next += threads;
        };
        fetch(0);
        fetch(1);
        for (int s = 0; held[s] < chunks && e == hipSuccess; s ^= 1) {
            e = hipEventSynchronize(slots->event[2 * t + s]);
            if (e != hipSuccess) break;
            deliver(held[s], slots->pinned + (2 * t + s) * std::min(slot, total));
            fetch(s);
        }
        if (e != hipSuccess) error = e;
    });
    const hipError_t e = hipStreamSynchronize(st);   // no copy is under way when the slots are used again
    give(slots);
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
