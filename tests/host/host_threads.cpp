// Every index once, and what a range throws reaches the caller.
#include <atomic>
#include <cstdio>
#include <new>

#include "host_threads.hpp"

using namespace shell;

int main() {
    for (int64_t n : {0, 1, 2, 15, 16, 17, 1000}) {
        std::vector<std::atomic<int>> seen(static_cast<size_t>(n));
        host_parallel_for(n, [&](int64_t a, int64_t b) {
            for (int64_t i = a; i < b; ++i) seen[size_t(i)]++;
        });
        for (auto& s : seen)
            if (s != 1) return 1;
    }
    for (int64_t bad : {0, 7, 999})
        for (int64_t small : {1, 2000}) {
            std::atomic<int> others{0};
            bool caught = false;
            try {
                host_parallel_for(
                    1000,
                    [&](int64_t a, int64_t b) {
                        if (bad >= a && bad < b) throw std::bad_alloc();
                        ++others;
                    },
                    small);
            } catch (const std::bad_alloc&) {
                caught = true;
            }
            if (!caught) return 1;
        }
    std::puts("ok");
}
