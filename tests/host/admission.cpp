// Admission of teams: requests that have waited for their patience in the order in which they came, from one thread that
// polls and from several that wait.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <thread>
#include <vector>

#include "team_host.hpp"

using namespace shell;

static void check(bool ok, const char* what) {
    if (ok) return;
    std::printf("%s\n", what);
    std::exit(1);
}

static void polled() {
    TeamSlots s(256, std::chrono::microseconds(0));
    auto a = std::make_unique<TeamLease>(), b = std::make_unique<TeamLease>(), all = std::make_unique<TeamLease>(),
         gone = std::make_unique<TeamLease>(), c = std::make_unique<TeamLease>();
    check(a->try_take(s, 100) && b->try_take(s, 100), "two leases that fit");
    check(!all->try_take(s, 256), "a request for all waits");
    a.reset();
    check(!gone->try_take(s, 8) && !c->try_take(s, 100), "nothing passes the request for all");
    b.reset();
    check(!c->try_take(s, 100), "nothing passes it when it could be served, either");
    check(all->try_take(s, 256) && all->try_take(s, 256), "the request for all is served, and stays so");
    all.reset();
    check(!c->try_take(s, 100), "its turn comes after the one before");
    gone.reset();  // a request that is given up leaves the line
    check(c->try_take(s, 100), "then its own");
    c.reset();
    bool refused = false;
    try {
        TeamLease over(s, 257);
    } catch (const std::length_error&) {
        refused = true;
    }
    check(refused, "more than there are");
    TeamLease again(s, 256);
}

// A request that has waited less may be passed, one that has waited longer not.
static void patience() {
    TeamSlots s(256, std::chrono::milliseconds(200));
    auto a = std::make_unique<TeamLease>(), all = std::make_unique<TeamLease>(), b = std::make_unique<TeamLease>(),
         c = std::make_unique<TeamLease>();
    check(a->try_take(s, 64) && !all->try_take(s, 256), "a request for all waits");
    check(b->try_take(s, 64), "a small one passes it");
    std::this_thread::sleep_for(std::chrono::milliseconds(250));
    check(!c->try_take(s, 64), "none passes it any more");
    a.reset();
    check(!c->try_take(s, 64) && !all->try_take(s, 256), "while one is in flight");
    b.reset();
    check(!c->try_take(s, 64) && all->try_take(s, 256), "it is served next");
    all.reset();
    check(c->try_take(s, 64), "then the one behind it");
}

// Whatever teams are in flight together, no XCD has more of their members than units.
static void xcds() {
    std::mt19937 rng(1);
    for (int cus : {32, 64, 256})
        for (int trial = 0; trial < 2000; ++trial) {
            TeamSlots s(cus);
            std::vector<std::unique_ptr<TeamLease>> held;
            std::vector<int> load(size_t(cus / kCusPerXcd), 0);
            for (int k = 0; k < 12; ++k) {
                const int n = 1 + int(rng() % (k % 2 ? 20u : unsigned(cus)));
                held.push_back(std::make_unique<TeamLease>());
                if (!held.back()->try_take(s, n)) {
                    held.pop_back();  // not admitted
                    continue;
                }
                const int first = int(rng() % load.size());
                for (int m = 0; m < n; ++m) load[size_t(first + m) % load.size()]++;
            }
            check(!held.empty(), "a team that fits");
            for (int l : load) check(l <= kCusPerXcd, "more members on an XCD than units");
        }
}

static void threads() {
    TeamSlots s(256, std::chrono::milliseconds(1));
    std::atomic<int> in_use{0};
    std::atomic<bool> stop{false};
    auto worker = [&](int n, bool poll) {
        while (!stop) {
            auto lease = poll ? std::make_unique<TeamLease>() : std::make_unique<TeamLease>(s, n);
            while (poll && !lease->try_take(s, n)) std::this_thread::yield();
            check((in_use += s.units(n)) <= 256, "more units than there are");
            std::this_thread::sleep_for(std::chrono::microseconds(50));
            in_use -= s.units(n);
        }
    };
    std::vector<std::thread> small;
    for (int k = 0; k < 4; ++k) small.emplace_back(worker, 64 + 16 * k, k % 2 == 1);
    for (int k = 0; k < 100; ++k) {
        TeamLease all(s, 256);
        check((in_use += 256) == 256, "all units");
        in_use -= 256;
    }
    stop = true;
    for (auto& t : small) t.join();
}

int main() {
    polled();
    patience();
    xcds();
    threads();
    std::puts("ok");
}
