// How teams (team.hpp) are dealt out on a device.  Plain host code, which any compiler takes.
#pragma once

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <deque>
#include <mutex>
#include <stdexcept>

namespace shell {

// Rows per member by the mesh's rows and the device's compute units: one member up to `alone` rows, then at least
// `least` rows each, and never more members than units, since all of them have to be resident together.
inline int64_t team_rows_spread(int64_t nv, int cus, int64_t alone, int64_t least) {
    auto whole = [](int64_t n) { return (n + 63) / 64 * 64; };
    return nv <= alone ? whole(nv) : std::max(least, whole((nv + cus - 1) / cus));
}

// Rows per member of a bending simulation on its own.  One member up to 1024 rows (no meetings: 6.8 us per iteration
// against 7.5 with two members of 512); then few rows each, since an iteration's product is a chain of
// latencies that grows with a member's rows: 256 while one wave can read all members' sums (4225 rows: 7.6 us
// against 8.5 with 512 and 10.5 with 1024), 512 up to as many members as compute units (32761 rows: 9.5 us
// against 10.4 with 256), beyond that whatever keeps one member per unit.
inline int64_t team_rows(int64_t nv, int cus) {
    const int64_t wave = std::min<int64_t>(64, cus);
    if (nv > 1024 && nv <= wave * 256) return 256;
    return team_rows_spread(nv, cus, 1024, 512);
}

// Rows per member with the membrane: one member up to 512, then as many members as compute units, of at least 256 rows
// (an iteration reads four times the matrix of the bending solve, so the rows are dealt out sooner: 65536 rows 15.6
// us with 256, 16.2 with 512; 128 rows gain 8% at 1089 and lose 10% at 16384).
inline int64_t team_rows_membrane(int64_t nv, int cus) { return team_rows_spread(nv, cus, 512, 256); }

constexpr int kCusPerXcd = 32;  // compute units that an XCD of the MI355X has in use

// Compute units free for resident teams on one device, one member per unit.  A launch takes its members'
// units before it is enqueued and gives them back once the host has seen it end.  The device deals a launch's
// work-groups round-robin over its XCDs, so a team of n members may bring any XCD ceil(n / XCDs) of them, and it takes
// that many units of each: with n alone counted, teams of 66, 66, 66 and 58 members (256) would bring the first XCD 35
// for its 32 units, and each of them might hold back one member that the others' wait for.
// Who finds room takes it until the oldest request has waited for its patience, 100 ms; from then on none passes that
// one, so that a mesh which needs all units gets them once the launches in flight have ended.  In strict order a batch
// with the membrane of 32 meshes, a fifth of which need all units, drained the device for each of their launches: 375 ms
// a step, against 349 without order and with this one.
class TeamSlots {
  public:
    TeamSlots() = default;
    explicit TeamSlots(int capacity, std::chrono::microseconds patience = std::chrono::milliseconds(100))
        : patience_(patience), capacity_(capacity), free_(capacity) {}
    int capacity() const { return capacity_; }
    // whether other launches are in flight or in line
    bool shared() const {
        std::lock_guard<std::mutex> lk(m_);
        return free_ != capacity_ || !line_.empty();
    }
    // units a team of n members takes
    int units(int n) const {
        const int xcds = std::max(1, capacity_ / kCusPerXcd);
        return std::min(capacity_, (n + xcds - 1) / xcds * xcds);
    }

  private:
    friend struct TeamLease;
    struct Request {
        int n;
        std::chrono::steady_clock::time_point since;
    };
    bool ready(const Request* r) const {
        const Request* oldest = line_.front();
        return free_ >= r->n && (r == oldest || std::chrono::steady_clock::now() - oldest->since < patience_);
    }
    void leave(const Request* r) { line_.erase(std::find(line_.begin(), line_.end(), r)); }
    void grant(const Request* r) {
        leave(r);
        free_ -= r->n;
    }

    mutable std::mutex m_;
    std::condition_variable cv_;
    std::deque<const Request*> line_;  // requests that wait, the oldest in front
    std::chrono::microseconds patience_{};
    int capacity_ = 0, free_ = 0;
};

// Iterations of one launch at most.  A launch keeps its units until it ends, which other work waits for (a chain of
// kernels lets it in at every kernel), so it takes some 50 ms, or 10 ms where other teams want units too; a longer solve
// goes on in another launch, on the same bits (1M rows, 8000 iterations: 337.6 -> 338.2 ms FP64 and 247.8 -> 249.5 mixed
// against one launch).  An iteration takes about
// 8 us and 1 us per 120 rows of a member (42 us at 4096 rows FP64), with the membrane 9 us and 1 us per 36 (122 us).
inline int team_launch_iterations(int64_t rows, bool membrane, bool shared) {
    const double us = membrane ? 9.0 + double(rows) / 36 : 8.0 + double(rows) / 120;
    return int((shared ? 10e3 : 50e3) / us);
}

// What a handle knows of how its teams fare.  Members that cannot all become resident (another process's team
// dispatched at the same time, a stream with fewer compute units) wait for kTeamWaitTicks and hand the solve to the chain
// of kernels; the next 16 solves then take the chain at once, twice as many after each further failure, up to 1024.
struct TeamRecord {
    // once per solve: whether it is to take the chain
    bool rests() { return rest_ > 0 && rest_-- > 0; }
    void gave_up() { rest_ = last_ = std::min(1024, std::max(16, 2 * last_)); }
    void met() { last_ = 0; }

  private:
    int rest_ = 0, last_ = 0;
};

// The units of one launch, or a place in the line for them; both end with it.
struct TeamLease {
    TeamLease() = default;
    // waits until the units are there
    TeamLease(TeamSlots& s, int n) {
        std::unique_lock<std::mutex> lk(s.m_);
        enter(s, n);
        s.cv_.wait(lk, [&] { return s.ready(&request_); });
        s.grant(&request_);
        held_ = true;
        lk.unlock();
        s.cv_.notify_all();  // what is left may do for the next
    }
    // true once the units are there; until then the request keeps its place in the line.  The caller asks again.
    bool try_take(TeamSlots& s, int n) {
        std::lock_guard<std::mutex> lk(s.m_);
        if (!slots_) enter(s, n);
        if (!held_ && s.ready(&request_)) {
            s.grant(&request_);
            held_ = true;
            s.cv_.notify_all();
        }
        return held_;
    }
    TeamLease(const TeamLease&) = delete;
    TeamLease& operator=(const TeamLease&) = delete;
    ~TeamLease() {
        if (!slots_) return;
        {
            std::lock_guard<std::mutex> lk(slots_->m_);
            if (held_)
                slots_->free_ += request_.n;
            else
                slots_->leave(&request_);
        }
        slots_->cv_.notify_all();
    }

  private:
    void enter(TeamSlots& s, int n) {
        if (n > s.capacity_) throw std::length_error("a team with more members than the device has compute units");
        s.line_.push_back(&request_);
        slots_ = &s;
        request_.n = s.units(n);
        request_.since = std::chrono::steady_clock::now();
    }
    TeamSlots* slots_ = nullptr;
    TeamSlots::Request request_{};
    bool held_ = false;
};

}  // namespace shell
