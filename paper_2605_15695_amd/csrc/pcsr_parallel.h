// Ranges of a loop on a few host threads (internal to the library).
#pragma once
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <new>
#include <thread>
#include <vector>

namespace pcsr {

// fn(lo, hi) for equal parts of [0, n), at least `grain` long.  What no thread can be started for
// runs here; a part that runs out of memory makes the call throw bad_alloc once all have ended.
template <class F> void parallel_for(int64_t n, int64_t grain, F &&fn)
{
    if (n <= 0) return;
    const unsigned hw = std::thread::hardware_concurrency();
    int64_t nt = std::max<int64_t>(1, std::min<int64_t>(hw ? hw : 4, 16));
    nt = std::min<int64_t>(nt, (n + grain - 1) / grain);
    if (nt <= 1) {
        fn(int64_t(0), n);
        return;
    }
    std::atomic<bool> failed{false};
    auto part = [&failed, &fn](int64_t lo, int64_t hi) {
        try {
            fn(lo, hi);
        } catch (const std::bad_alloc &) {
            failed = true;
        }
    };
    std::vector<std::thread> th;
    try {
        th.reserve(nt);
    } catch (...) {
        fn(int64_t(0), n);
        return;
    }
    const int64_t per = (n + nt - 1) / nt;
    for (int64_t lo = 0; lo < n; lo += per) {
        const int64_t hi = std::min(n, lo + per);
        try {
            th.emplace_back(part, lo, hi);
        } catch (...) {
            part(lo, hi);
        }
    }
    for (auto &t : th) t.join();
    if (failed) throw std::bad_alloc();
}

} // namespace pcsr
