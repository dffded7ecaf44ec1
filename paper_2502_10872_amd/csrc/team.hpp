// Teams: solves whose work-groups stay resident and meet once per reduction instead of ending a kernel.
//
// A conjugate-gradient iteration needs two global sums.  As two kernels per iteration, every sum costs a
// kernel boundary and every vector makes a round trip through memory between them.  A team is the set of
// work-groups (members) of one launch that solve one mesh together: each keeps its own rows' vectors in
// registers and the directions it multiplies in LDS for the whole solve, and the members exchange only
// their partial sums and the few rows their neighbours read.
//
// Exchange.  Every member publishes its partial sums in slots of its own and every member reads all slots
// and adds them in member order, so all of them obtain the same bits, in every run.  A slot that has not
// been written holds kUnset, a NaN pattern no sum is published as; a reader waits for every slot to change,
// so the sums are their own flags and no counter or fence is needed.  Slots are double-buffered by
// iteration parity: a member unsets its slots of one parity after it has read every member's next sum
// (which every member publishes only after it has read those slots), and has waited for that store (vmcnt)
// before it publishes the sum after that.  Rows that other members read are exchanged the same way, every
// value its own flag.  All of these accesses are agent-scope relaxed atomics, which bypass the caches that
// are private to a compute unit or an XCD.
//
// Waiting.  A reader polls the sum a member stores last and then reads the others.  Measured on the 65 x 65
// plate (9 to 17 members): 2 us from a member's first store to every member's total.
//
// Every wait is bounded: past the launch's limit a member gives up, raises the team's flag and leaves, as
// every other member then does; the host finds the flag and runs the solve, and the next few (TeamRecord), as a
// chain of kernels.  That can only happen when other work keeps some members from becoming resident.  Within a
// process the host admits a launch only while compute units are left for all of its members (TeamSlots).
#pragma once

#include <hip/hip_runtime.h>

#include "devmath.hpp"
#include "internal.hpp"

namespace shell {

constexpr unsigned long long kUnset = 0x7ff8dead0000beefull;
constexpr unsigned long long kPlainNan = 0x7ff8000000000000ull;
constexpr int kTeamQ = 6;                    // sums per exchange at most
// The longest wait: 100 ms of the 100 MHz wall clock, 800 iterations of the largest meshes (a member once resident waits
// for part of one).
constexpr uint64_t kTeamWaitTicks = 10000000;

// slots of one mesh: [set][parity][sum][member], then the flag
__host__ __device__ constexpr size_t team_slot_count(int members) { return size_t(2 * 2 * kTeamQ) * size_t(members); }

__device__ __forceinline__ double* team_set(double* slots, int members, int set, long par) {
    return slots + (size_t(set) * 2 + size_t(par & 1)) * kTeamQ * size_t(members);
}

__device__ __forceinline__ void team_publish(double* slot, double v) {
    const unsigned long long u = __builtin_isnan(v) ? kPlainNan : (unsigned long long)__double_as_longlong(v);
    agent_store(reinterpret_cast<unsigned long long*>(slot), u);
}

// The sum of v over the wave, in lane 63 (the other lanes hold partial sums): rows of 16 by shifts, then the
// rows' ends broadcast to the rows after them.  Register moves between lanes instead of LDS permutes: six of
// these sums took 0.45 us as butterflies of __shfl_xor.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(0, int(unsigned(u)), CTRL, ROWS, 0xf, false));
    const unsigned hi = unsigned(__builtin_amdgcn_update_dpp(0, int(unsigned(u >> 32)), CTRL, ROWS, 0xf, false));
    return v + __longlong_as_double((long long)((unsigned long long)lo | ((unsigned long long)hi << 32)));
}
__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add<0x118, 0xf>(v);  // row_shr:8
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// a wave-uniform double from lane `lane`
__device__ __forceinline__ double read_lane(double v, int lane) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(unsigned(u)), lane));
    const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(unsigned(u >> 32)), lane));
    return __longlong_as_double((long long)((unsigned long long)lo | ((unsigned long long)hi << 32)));
}

// What a work-group keeps to meet its team.
struct TeamMeet {
    double* slots;
    int* flag;        // set when a member has given up
    int* lost;        // LDS: this member has (zero at the start)
    int members, member;
    uint64_t limit;   // ticks a wait may take
};

// One round of a bounded wait: true when the waiting thread is to give up.
struct TeamWait {
    uint64_t began = 0;
    unsigned spin = 0;
    __device__ __forceinline__ bool over(const TeamMeet& tm) {
        if ((++spin & 63u) != 0 && tm.limit != 0) return false;
        const uint64_t now = wall_clock64();
        if (!began) began = now;
        return now - began >= tm.limit || agent_load(tm.flag) != 0;
    }
};

__device__ __forceinline__ void team_give_up(const TeamMeet& tm) {
    *tm.lost = 1;
    agent_store(tm.flag, 1);
}

// A work-group's sums of NQ quantities over its threads into sh[q * waves + wave] (no barrier).
template <int NQ>
__device__ __forceinline__ void wave_partials(double (&v)[NQ], double* sh) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = wave_sum_last(v[q]);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 63)
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[q * nw + w] = v[q];
}

// lane q of the wave adds sum q's `count` wave partials in order
template <int NQ>
__device__ __forceinline__ double add_partials(const double* sh, int count) {
    const int nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    double t = 0.0;
    if (lane < NQ)
        for (int k = 0; k < count; ++k) t += sh[lane * nw + k];
    return t;
}

// Publishes this member's NQ sums from the wave partials in sh (complete: a barrier lies between).
template <int NQ>
__device__ __forceinline__ void team_send(const TeamMeet& tm, int set, long par, const double* sh) {
    if (tm.members == 1 || threadIdx.x >= 64) return;
    const double t = add_partials<NQ>(sh, blockDim.x >> 6);
    if (threadIdx.x < NQ)
        team_publish(team_set(tm.slots, tm.members, set, par) + size_t(threadIdx.x) * tm.members + tm.member, t);
}

// The team's totals of NQ sums once every member has sent them: lane q of every wave returns the total of sum q
// (lanes from NQ up: nothing of use).  sh: what this member sent; out_sh: NQ * waves doubles of LDS that
// nothing else uses until the next barrier after this call.  Every thread calls it; then *tm.lost says whether
// to leave.
template <int NQ>
__device__ __forceinline__ double team_receive(const TeamMeet& tm, int set, long par, const double* sh, double* out_sh) {
    const int nw = blockDim.x >> 6, lane = threadIdx.x & 63;
    if (tm.members == 1) return add_partials<NQ>(sh, nw);
    const double* base = team_set(tm.slots, tm.members, set, par);
    const int w = threadIdx.x >> 6, used = min(nw, (tm.members + 63) >> 6);
    if (w < used) {
        double v[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = 0.0;
        for (int m = threadIdx.x; m < tm.members; m += blockDim.x) {
            const unsigned long long* at = reinterpret_cast<const unsigned long long*>(base) + m;
            TeamWait wait;
            // the sum stored last is watched, the others are then there or about to be
            unsigned long long u[NQ];
            bool unset = true;
            while (unset) {
                u[NQ - 1] = agent_load(at + size_t(NQ - 1) * tm.members);
                unset = u[NQ - 1] == kUnset;
                if (!unset) {
#pragma unroll
                    for (int q = 0; q < NQ - 1; ++q) u[q] = agent_load(at + size_t(q) * tm.members);
#pragma unroll
                    for (int q = 0; q < NQ - 1; ++q) unset |= u[q] == kUnset;
                }
                if (unset && wait.over(tm)) break;
            }
            if (unset) {
                team_give_up(tm);
                break;
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[q] += __longlong_as_double((long long)u[q]);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = wave_sum_last(v[q]);
        if (lane == 63)
#pragma unroll
            for (int q = 0; q < NQ; ++q) out_sh[q * nw + w] = v[q];
    }
    __syncthreads();
    return add_partials<NQ>(out_sh, used);
}

// unsets this member's slots of a set whose sums every member has read (NQ threads store)
template <int NQ>
__device__ __forceinline__ void team_unset(const TeamMeet& tm, int set, long par) {
    if (tm.members > 1 && threadIdx.x < NQ)
        agent_store(reinterpret_cast<unsigned long long*>(team_set(tm.slots, tm.members, set, par)) +
                        size_t(threadIdx.x) * tm.members + tm.member,
                    kUnset);
}

// a mesh's slots and flag as a solve expects them; every thread of one work-group takes part
__device__ __forceinline__ void team_clear(double* slots, int* flag, int members) {
    for (size_t k = threadIdx.x; k < team_slot_count(members); k += blockDim.x)
        agent_store(reinterpret_cast<unsigned long long*>(slots) + k, kUnset);
    if (threadIdx.x == 0) agent_store(flag, 0);
}

constexpr int kTeamThreads = 512;  // of a member: two waves per SIMD, 256 registers each

template <typename MR>
struct Pair;
template <>
struct Pair<double> {
    typedef double type __attribute__((ext_vector_type(2)));
};
template <>
struct Pair<float> {
    typedef float type __attribute__((ext_vector_type(2)));
};

// An exchanged row's value as bits; `unset` is a NaN pattern that no value is published as.
template <typename VR>
struct Row;
template <>
struct Row<double> {
    typedef unsigned long long bits_t;
    static constexpr bits_t unset = kUnset;
    __device__ __forceinline__ static bits_t bits(double v) {
        return __builtin_isnan(v) ? kPlainNan : bits_t(__double_as_longlong(v));
    }
    __device__ __forceinline__ static double value(bits_t u) { return __longlong_as_double((long long)u); }
};
template <>
struct Row<float> {
    typedef unsigned bits_t;
    static constexpr bits_t unset = 0x7fdeadbeu;
    __device__ __forceinline__ static bits_t bits(float v) { return __builtin_isnan(v) ? 0x7fc00000u : __float_as_uint(v); }
    __device__ __forceinline__ static float value(bits_t u) { return __uint_as_float(u); }
};

// The same value, unknown to the compiler: what is computed from it inside a loop is computed there, in place
// of once before the loop with a register per row held through it.
template <typename V>
__device__ __forceinline__ V here(V v) {
    asm volatile("" : "+v"(v));
    return v;
}

// compute units for teams on the current device (host)
TeamSlots& team_slots();

}  // namespace shell
