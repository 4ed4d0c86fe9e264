// Host work spread over a few threads (no device code).
#pragma once

#include <functional>
#include <thread>

namespace vplbm {

// work(0) .. work(n - 1) side by side, n at most 8, all of them also where a thread cannot be started
// (no thread, no memory for one: whatever its start throws).  work throws nothing.
template <typename F> void side_by_side(int n, const F &work)
{
    std::thread threads[8];
    int started = 1;
    try {
        for (; started < n; started++) threads[started] = std::thread(std::cref(work), started);
    } catch (...) {
    }
    work(0);
    for (int t = started; t < n; t++) work(t);
    for (int t = 1; t < started; t++) threads[t].join();
}

}  // namespace vplbm
