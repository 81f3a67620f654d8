// Host threads that share one piece of work, free of HIP so that a
// host-compiled test can run it.
#pragma once

#include <algorithm>
#include <functional>
#include <thread>
#include <vector>

namespace wc {

// work() on this thread and on up to `extra` others, until all have returned.  It
// takes its items from a shared counter and must not throw.  A thread that
// cannot be started, for want of threads or of memory, is done without: the
// others take its items, and those already running are joined in any case.
template <class F>
void run_shared(int extra, F&& work) {
    std::vector<std::thread> pool;
    try {
        pool.reserve(std::max(0, extra));
        for (int t = 0; t < extra; ++t) pool.emplace_back(std::ref(work));
    } catch (...) {
    }
    work();
    for (auto& t : pool) t.join();
}

}  // namespace wc
