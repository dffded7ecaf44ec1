// Arrivals of one launch and of launches that share their counters and overlap: an arrival may be held up before each
// of its operations while others run.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "arrivals.hpp"

using namespace shell;

static void check(bool ok, const char* what, long n) {
    if (ok) return;
    std::printf("%s, %ld work-groups\n", what, n);
    std::exit(1);
}

struct Run {
    std::vector<uint32_t> counters;
    std::vector<long> pending;  // work-groups yet to arrive, of all launches
    std::mt19937 rng;
    long n;
    int lasts = 0;
    bool overlapped;

    void next() {
        const long blk = pending.back();
        pending.pop_back();
        lasts += arrive_last(counters.data(), blk, n, [&](uint32_t* c, uint32_t top) {
            while (overlapped && !pending.empty() && rng() % 4 == 0) next();
            const uint32_t was = *c;
            *c = was >= top ? 0 : was + 1;
            return was;
        });
    }
};

int main() {
    for (long n : {1, 2, 15, 16, 17, 31, 32, 33, 255, 256, 512})
        for (unsigned seed = 0; seed < 200; ++seed)
            for (int launches : {1, 2, 4}) {
                Run r{std::vector<uint32_t>(arrival_counters(n), 0u), {}, std::mt19937(seed), n, 0, launches > 1};
                for (int l = 0; l < launches; ++l)
                    for (long b = 0; b < n; ++b) r.pending.push_back(b);
                std::shuffle(r.pending.begin(), r.pending.end(), r.rng);
                while (!r.pending.empty()) {
                    check(launches > 1 || r.lasts == 0, "a work-group after the last", n);
                    r.next();
                }
                check(r.lasts == launches, "as many last work-groups as launches", n);
                for (uint32_t c : r.counters) check(c == 0, "counters back at zero", n);
            }
    std::puts("ok");
}
