// The coupled Jacobi PCG of the step with the membrane as one kernel per solve (see team.hpp for how its
// work-groups meet).  Included once, by membrane.hip, after its scalars.
//
// As in the bending solve a member keeps r, y and q of its rows in registers and the directions of its rows and
// halo columns in LDS (all float64, in both precisions).  Per iteration it streams its rows' off-diagonal K_s
// entries (the bending Hessian's pairs) and the nine component arrays of the tangent's blocks, and exchanges
// the z of the rows that others read and three sums.
//
// What bounds it: the matrix stream at a million rows (742 MB FP64 in 113 us, 6.6 TB/s; 400 MB mixed in 63 us, 6.3
// TB/s), latency below some 30,000 (two meetings, the halo's round trip and the reads of a row's blocks).  Per
// iteration, before (three kernels) and now, FP64 and mixed: 11.5 / 10.4 -> 7.7 / 5.9 us at 484 vertices, 10.9 /
// 12.5 -> 9.2 / 8.1 at 4096, 19.7 / 18.6 -> 15.6 / 12.3 at 65536, 182 / 126 -> 122 / 73 at 1M.
#pragma once

#include "team.hpp"

namespace shell {

namespace {

struct TeamMembraneArgs {
    const int64_t* tptr;   // K_s pairs: slots, widths, values, local columns
    const int32_t* twid;
    const void* tval;
    const uint32_t* tcol;
    const int64_t* mptr;   // blocks: slots, widths, component values, local columns
    const int32_t* mwidth;
    const void* mval;
    const uint16_t* mcol;
    long mstride;
    const int32_t* hptr;
    const int32_t* hcols;
    const uint8_t* send;
    const double* mass;
    const double* kdiag;
    const uint8_t* pinned;
    const double* dinv;
    const double* g;
    double *r, *y, *p;
    double* rows[2];       // the exchanged rows' z by iteration parity
    double* slots;
    double* scal;          // state set 0
    long nv;
    double dt2, rtol2;
    int R, members, target, replay, resume, limit, every;
    uint64_t wait;
};

__host__ __device__ constexpr size_t team_membrane_lds(int rows, int halo) {
    return size_t(rows + halo) * 3 * sizeof(double) + size_t(rows) * sizeof(double);
}

// Pairs of K_s and blocks requested together (see kTeamBatch): as many as the registers beside the rows'
// vectors hold.  Registers by rows per thread, FP64 / mixed: 1 106 / 136, 2 132 / 160, 4 171 / 196, 6 195 / 218, 8 238 /
// 256, where the mixed instance spills two (12 bytes of scratch per lane); those of one and two rows hold 20 bytes of
// scratch, for scalar values, and no vector register.
template <typename VT>
constexpr int kMsTeamPairs = sizeof(VT) == 8 ? 3 : 9;
template <typename VT, int RPL>
constexpr int kMsTeamBlocks = sizeof(VT) == 8 ? (RPL <= 4 ? 2 : 1) : (RPL <= 4 ? 4 : 2);

// Matrices that outgrow the 256 MB last-level cache are read with non-temporal loads, which keep the halo's exchange and
// the little that is read again in the caches: 1M rows 144 -> 122 us per iteration FP64 and 87 -> 73 mixed, 524K
// rows FP64 74 -> 64.  Smaller ones are read again from the caches with plain loads (16384 rows: 10.4 us FP64 against
// 12.1 non-temporal).  The line is drawn by rows per thread, a constant of the instance: a smoothed or FVM mesh's
// matrices pass 256 MiB at some 380,000 rows FP64 and 700,000 mixed, and the instances change at 262144 and
// 524288, just below; an edge mesh's, of fewer entries per row, at some 420,000 and 790,000.
template <typename VT, int RPL>
constexpr bool kMsTeamStream = sizeof(VT) == 8 ? RPL > 2 : RPL > 4;
template <bool STREAM, typename V>
__device__ __forceinline__ V stream_or_cached(const gbl<const V>* p) {
    if constexpr (STREAM)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <typename VT, int RPL>
__global__ __launch_bounds__(kTeamThreads) void ms_team_pcg(TeamMembraneArgs A) {
    typedef typename Pair<VT>::type VT2;
    constexpr int T = kTeamThreads, NW = T / 64, B = kMsTeamPairs<VT>, BB = kMsTeamBlocks<VT, RPL>;
    constexpr bool ST = kMsTeamStream<VT, RPL>;
    constexpr bool DIFF = sizeof(VT) == 4;
    extern __shared__ double ps[];
    __shared__ double shA[NW], outA[NW], shB[2 * NW], outB[2 * NW];
    __shared__ int lost;
    __shared__ uint64_t ticks[2], since;
    __shared__ int samples;
    struct Rec {
        double rz, rr, tol2;
        int iters, active, budget;
    };
    __shared__ Rec rec[2];
    const int member = blockIdx.x, wave = threadIdx.x >> 6, R = A.R;
    const long nv = A.nv, base = long(member) * R;
    const TeamMeet tm{A.slots, reinterpret_cast<int*>(A.scal + S_GONE), &lost, A.members, member, A.wait};
    const int h0 = G(A.hptr)[member], nh = G(A.hptr)[member + 1] - h0;
    const gbl<const int32_t>* hc = G(A.hcols) + h0;
    double* dj = ps + 3 * (R + nh);  // the rows' Jacobi entries
    if (threadIdx.x == 0) {
        lost = 0;
        ticks[0] = ticks[1] = 0;
        samples = 0;
        Rec o{};
        if (A.resume) {
            o.rz = A.scal[S_RZ];
            o.rr = A.scal[S_RR];
            o.tol2 = A.scal[S_TOL2];
            o.iters = int(A.scal[S_IT]);
            o.active = 1;
        }
        rec[0] = o;
    }
    double r[RPL][3], y[RPL][3];
    unsigned send = 0, held = 0;
    const long slice0 = base >> 6;
    const int64_t tp0 = G(A.tptr)[slice0], mp0 = G(A.mptr)[slice0];
    int off[RPL], w[RPL], moff[RPL], mw[RPL];  // K_s pairs and blocks of the thread's slices; wave-uniform
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
        const int lr = s * T + int(threadIdx.x), lw = s * T + wave * 64;
        const long i = base + lr;
        const bool live = lw < R && base + lw < nv;
        const long slice = live ? (base + lw) >> 6 : slice0;
        w[s] = live ? __builtin_amdgcn_readfirstlane(G(A.twid)[slice]) : 0;
        mw[s] = live ? __builtin_amdgcn_readfirstlane(G(A.mwidth)[slice]) : 0;
        off[s] = __builtin_amdgcn_readfirstlane(int(G(A.tptr)[slice] - tp0));
        moff[s] = __builtin_amdgcn_readfirstlane(int(G(A.mptr)[slice] - mp0));
#pragma unroll
        for (int c = 0; c < 3; ++c) r[s][c] = y[s][c] = 0.0;
        if (lr < R) {  // also the rows past nv of the last slice: their direction stays zero
#pragma unroll
            for (int c = 0; c < 3; ++c) ps[3 * lr + c] = 0.0;
            dj[lr] = 0.0;
        }
        if (live && i < nv) {
            dj[lr] = G(A.dinv)[i];
            held |= unsigned(G(A.pinned)[i] & 7u) << (3 * s);
            if (G(A.send)[i]) send |= 1u << s;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[s][c] = A.resume ? G(A.r)[3 * i + c] : -G(A.g)[3 * i + c];
                if (A.resume) {
                    y[s][c] = G(A.y)[3 * i + c];
                    ps[3 * lr + c] = G(A.p)[3 * i + c];
                }
            }
        }
    }
    if (A.resume)
        for (int h = threadIdx.x; h < nh; h += T)
#pragma unroll
            for (int c = 0; c < 3; ++c) ps[3 * (R + h) + c] = G(A.p)[3L * hc[h] + c];

    auto rows_of = [&](int par) { return reinterpret_cast<unsigned long long*>(A.rows[par & 1]); };
    auto unset_rows = [&](int par) {
        unsigned long long* zx = rows_of(par);
        const unsigned at = 3u * (unsigned(base) + unsigned(here(int(threadIdx.x))));
#pragma unroll
        for (int s = 0; s < RPL; ++s)
            if (send >> s & 1u)
#pragma unroll
                for (int c = 0; c < 3; ++c) agent_store(zx + (at + unsigned(3 * s * T + c)), kUnset);
    };
    // z = D^-1 r: published where others read it; the sums r.z, r.r
    auto publish_rows = [&](int par, double (&acc)[2]) {
        unsigned long long* zx = rows_of(par);
        const int tid = here(int(threadIdx.x));
        const unsigned at = 3u * (unsigned(base) + unsigned(tid));
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const double di = s * T + tid < R ? dj[s * T + tid] : 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double z = di * r[s][c];
                acc[0] += r[s][c] * z;
                acc[1] += r[s][c] * r[s][c];
                if (send >> s & 1u) agent_store(zx + (at + unsigned(3 * s * T + c)), Row<double>::bits(z));
            }
            if (RPL > 2) __builtin_amdgcn_sched_barrier(0);  // one row's temporaries at a time
        }
    };
    {
        // the first rows replace whatever an earlier solve left, so they are in place before the first sums
        double acc[2] = {0, 0};
        unset_rows(1);
        publish_rows(0, acc);
        wait_stores();
        wave_partials<2>(acc, shB);
    }
    __syncthreads();
    team_send<2>(tm, 1, 0, shB);
    int n = 0;
    bool done = false;
    for (;; ++n) {
        double beta;
        {
            const double tb = team_receive<2>(tm, 1, n, shB, outB);
            if (lost) return;
            team_unset<1>(tm, 0, n + 1);  // the previous product's sum: every member has read it
            // the recurrence moves on (every thread alike; thread 0 stores it)
            const double rzn = read_lane(tb, 0), rrn = read_lane(tb, 1);
            Rec o = rec[n & 1];
            beta = 0.0;
            if (n == 0 && !A.resume) {
                o.tol2 = A.rtol2 * rrn;
                o.active = 0 < A.target && (A.replay || rrn > o.tol2);
            } else {
                beta = o.rz != 0.0 ? rzn / o.rz : 0.0;
                o.iters += 1;
                const bool more = A.replay || rrn > o.tol2;
                if (!A.replay && o.iters >= A.target && more) o.budget = 1;
                if (!isfinite(rrn)) o.budget = 2;
                o.active = o.iters < A.target && more && isfinite(rrn);
            }
            o.rz = rzn;
            o.rr = rrn;
            if (threadIdx.x == 0) rec[(n + 1) & 1] = o;
            done = __ballot(o.active != 0) == 0;
        }
        if (done) break;
        const bool sample = A.every > 0 && n % A.every == 0 && member == 0 && threadIdx.x == 0;
        if (sample) since = wall_clock64();
        // p = z + beta p: the first halo column's z is requested, the own rows advance, then the halo does
        const int tid = here(int(threadIdx.x));
        {
            const unsigned long long* zx = rows_of(n);
            unsigned long long zb[3] = {0, 0, 0};
            unsigned col = 0;
            if (tid < nh) {
                col = 3u * unsigned(hc[tid]);
#pragma unroll
                for (int c = 0; c < 3; ++c) zb[c] = agent_load(zx + col + c);
            }
#pragma unroll
            for (int s = 0; s < RPL; ++s) {
                const int lr = s * T + here(tid);
                if (lr < R) {
                    const double di = dj[lr];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double z = di * r[s][c];
                        ps[3 * lr + c] = beta != 0.0 ? fma(beta, ps[3 * lr + c], z) : z;
                    }
                }
                if (RPL > 2) __builtin_amdgcn_sched_barrier(0);
            }
            for (int h = tid; h < nh; h += T) {
                if (h != tid) {
                    col = 3u * unsigned(hc[h]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) zb[c] = agent_load(zx + col + c);
                }
                TeamWait wait;
                while (zb[0] == kUnset || zb[1] == kUnset || zb[2] == kUnset) {
                    if (wait.over(tm)) {
                        team_give_up(tm);
                        break;
                    }
#pragma unroll
                    for (int c = 0; c < 3; ++c) zb[c] = agent_load(zx + col + c);
                }
                double* pj = ps + 3 * (R + h);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double z = Row<double>::value(zb[c]);
                    pj[c] = beta != 0.0 ? fma(beta, pj[c], z) : z;
                }
            }
        }
        __syncthreads();
        if (lost) return;
        // q = (M + dt^2 (K_s (x) I3 + K_m)) p, held coordinates zero; p.q
        double q[RPL][3];
        double pq[1] = {0.0};
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const int lr = s * T + here(tid);
            const unsigned ln = unsigned(here(tid)) & 63u;
            double pi[3] = {0, 0, 0}, a[3] = {0, 0, 0}, m = 0.0;
            const bool own = w[s] > 0 && base + lr < nv;
            if (own) {
                m = G(A.mass)[base + lr];
                if constexpr (!DIFF) m += A.dt2 * G(A.kdiag)[base + lr];
            }
            if (DIFF && w[s] > 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) pi[c] = ps[3 * lr + c];
            {
                const gbl<const VT2>* gv = G(static_cast<const VT2*>(A.tval)) + tp0 + off[s];
                const gbl<const uint32_t>* gc = G(A.tcol) + tp0 + off[s];
                auto use = [&](VT2 v, uint32_t cc) {
                    const double* p0 = ps + 3 * (cc & 0xffffu);
                    const double* p1 = ps + 3 * (cc >> 16);
#pragma unroll
                    for (int c = 0; c < 3; ++c) a[c] = fma(double(v.x), DIFF ? p0[c] - pi[c] : p0[c], a[c]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) a[c] = fma(double(v.y), DIFF ? p1[c] - pi[c] : p1[c], a[c]);
                };
                int k = 0;
                for (; k + B <= w[s]; k += B) {
                    VT2 v[B];
                    uint32_t cc[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        v[u] = stream_or_cached<ST>(gv + 64u * unsigned(k + u) + ln);
                        cc[u] = gc[64u * unsigned(k + u) + ln];
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        use(v[u], cc[u]);
                        __builtin_amdgcn_sched_barrier(0);  // one pair's directions in registers at a time
                    }
                }
                for (; k < w[s]; k += 3) {
                    VT2 v[3];
                    uint32_t cc[3];
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        const unsigned at = 64u * unsigned(min(k + u, w[s] - 1)) + ln;
                        v[u] = gv[at];
                        cc[u] = gc[at];
                    }
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (k + u < w[s]) use(v[u], cc[u]);
                }
            }
            {
                const gbl<const VT>* gb = G(static_cast<const VT*>(A.mval)) + mp0 + moff[s];
                const gbl<const uint16_t>* gc = G(A.mcol) + mp0 + moff[s];
                for (int k = 0; k < mw[s]; k += BB) {
                    VT v[BB][9];
                    int cc[BB];
#pragma unroll
                    for (int u = 0; u < BB; ++u)
                        if (k + u < mw[s]) {  // wave-uniform
                            const unsigned at = 64u * unsigned(k + u) + ln;
#pragma unroll
                            for (int e = 0; e < 9; ++e) v[u][e] = stream_or_cached<ST>((gb + e * A.mstride) + at);
                            cc[u] = gc[at];
                        }
#pragma unroll
                    for (int u = 0; u < BB; ++u)
                        if (k + u < mw[s]) {
                            const double* pc = ps + 3 * cc[u];
                            const double d0 = DIFF ? pc[0] - pi[0] : pc[0], d1 = DIFF ? pc[1] - pi[1] : pc[1],
                                         d2 = DIFF ? pc[2] - pi[2] : pc[2];
#pragma unroll
                            for (int c = 0; c < 3; ++c)
                                a[c] += double(v[u][3 * c]) * d0 + double(v[u][3 * c + 1]) * d1 +
                                        double(v[u][3 * c + 2]) * d2;
                            __builtin_amdgcn_sched_barrier(0);
                        }
                }
            }
            if (!DIFF && w[s] > 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) pi[c] = ps[3 * lr + c];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                q[s][c] = own && !(held >> (3 * s + c) & 1u) ? fma(A.dt2, a[c], m * pi[c]) : 0.0;
                pq[0] = here(fma(pi[c], q[s][c], pq[0]));  // now, not with every row's p and q held
            }
        }
        wait_stores();  // the slots and rows unset since the last product have reached memory long since
        wave_partials<1>(pq, shA);
        __syncthreads();
        team_send<1>(tm, 0, n, shA);
        const double ta = read_lane(team_receive<1>(tm, 0, n, shA, outA), 0);
        if (lost) return;
        team_unset<2>(tm, 1, n);  // this iteration's first sums and rows: every member has read them
        unset_rows(n);
        if (sample) {
            const uint64_t now = wall_clock64();
            ticks[0] += now - since;
            since = now;
        }
        const double al = ta != 0.0 ? rec[(n + 1) & 1].rz / ta : 0.0;
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const int lr = s * T + here(tid);
            if (w[s] > 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    y[s][c] = fma(al, ps[3 * lr + c], y[s][c]);
                    r[s][c] = fma(-al, q[s][c], r[s][c]);
                }
            if (RPL > 2) __builtin_amdgcn_sched_barrier(0);
        }
        {
            double acc[2] = {0, 0};
            publish_rows(n + 1, acc);
            wave_partials<2>(acc, shB);
        }
        __syncthreads();
        team_send<2>(tm, 1, n + 1, shB);
        if (sample) {
            ticks[1] += wall_clock64() - since;
            ++samples;
        }
        if (n + 1 == A.limit) break;  // the next launch takes it from here
    }
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
        const int lr = s * T + here(int(threadIdx.x));
        const long i = base + lr;
        if (w[s] > 0 && i < nv)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                G(A.y)[3 * i + c] = y[s][c];
                if (!done) {
                    G(A.r)[3 * i + c] = r[s][c];
                    G(A.p)[3 * i + c] = ps[3 * lr + c];
                }
            }
    }
    if (member == 0 && threadIdx.x == 0) {
        const Rec& o = rec[(n + 1) & 1];
        double* st = A.scal;
        st[S_RZ] = o.rz;
        st[S_RR] = o.rr;
        st[S_TOL2] = o.tol2;
        st[S_IT] = double(o.iters);
        st[S_BUDGET] = double(o.budget);
        st[S_ACTIVE] = done ? 0.0 : 1.0;
        st[S_SAMPLE0] = double(ticks[0]);
        st[S_SAMPLE1] = double(ticks[1]);
        st[S_SAMPLES] = double(samples);
    }
}

__global__ __launch_bounds__(kTeamThreads) void ms_team_clear(double* slots, double* scal, int members) {
    team_clear(slots, reinterpret_cast<int*>(scal + S_GONE), members);
}

}  // namespace

}  // namespace shell
