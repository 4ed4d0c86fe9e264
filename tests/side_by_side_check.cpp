// Work spread over threads where starting one fails for want of memory: all of it is done, and nothing is
// thrown.  Prints "ok".
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>

#include "side_by_side.hpp"

static std::atomic<int> allocations_left{1 << 30};

void *operator new(std::size_t n)
{
    if (allocations_left-- <= 0) throw std::bad_alloc();
    if (void *p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main()
{
    for (int threads = 1; threads <= 8; threads++)
        for (int left = 0; left <= 8; left++) {
            std::atomic<int> done[8] = {};
            allocations_left = left;
            vplbm::side_by_side(threads, [&](int t) { done[t]++; });
            allocations_left = 1 << 30;
            for (int t = 0; t < 8; t++)
                if (done[t] != (t < threads)) {
                    std::printf("%d threads, %d allocations: part %d done %d times\n", threads, left, t, done[t].load());
                    return 1;
                }
        }
    std::puts("ok");
    return 0;
}
