// Ranges over the host's threads.  Plain host code, which any compiler takes.
#pragma once

#include <algorithm>
#include <cstdint>
#include <exception>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace shell {

// Runs fn(first, last) over [0, n) on at most 16 threads; n below `small` on this thread.  What a range throws (the
// first of several) is thrown here once every thread has ended: an exception that leaves a thread, or a thread that is
// dropped unjoined, would end the process.  A range for which there is no thread runs on this one.
template <typename F>
void host_parallel_for(int64_t n, F&& fn, int64_t small = 1) {
    const int64_t nt = std::max<int64_t>(1, std::min<int64_t>({16, int64_t(std::thread::hardware_concurrency()), n}));
    if (n < small || nt == 1) {
        if (n > 0) fn(int64_t(0), n);
        return;
    }
    std::exception_ptr thrown;
    std::mutex m;
    auto range = [&](int64_t a, int64_t b) {
        try {
            fn(a, b);
        } catch (...) {
            std::lock_guard<std::mutex> lk(m);
            if (!thrown) thrown = std::current_exception();
        }
    };
    const int64_t chunk = (n + nt - 1) / nt;
    std::vector<std::thread> th;
    th.reserve(size_t(nt));
    for (int64_t a = 0; a < n; a += chunk) {
        const int64_t b = std::min(n, a + chunk);
        try {
            th.emplace_back(range, a, b);
        } catch (const std::system_error&) {
            range(a, b);
        }
    }
    for (auto& t : th) t.join();
    if (thrown) std::rethrow_exception(thrown);
}

}  // namespace shell
