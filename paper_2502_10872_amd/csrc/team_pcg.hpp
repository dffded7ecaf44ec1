// The three-column Jacobi PCG of the bending step as one kernel per solve (see team.hpp for how its
// work-groups meet).  Included once, by solver.hip, after pcg_kernels.hpp.
//
// z = D^-1 r takes the reciprocal of the diagonal from inv_fast (an estimate and two Newton steps, the last bit or two
// off), where the chain reads a stored, correctly rounded 1 / d: the preconditioner alone differs, and the two
// solves by rounding.
//
// A member owns d.trows consecutive rows: row base + s T + thread is the thread's s-th.  r, y, q and the row's
// diagonal stay in registers from the first iteration to the last; the directions p of the own rows and
// of the halo columns (the columns of other members' rows) in LDS, where every member advances its own
// copy, p = z + beta p, from the same z bits.  Per iteration a member therefore streams only its rows'
// off-diagonal entries, and exchanges the z of the rows that other members read and nine sums.
//
// What bounds it.  Up to some 100,000 rows latency: two meetings (about 2 us each with 9 to 17 members, 3.5 us with 128), the
// halo's round trip through memory and a row's chain of LDS reads; 7.6 us per iteration at 4225 rows (17 members),
// 11.5 at 65536.  At a million rows the matrix stream: 239 MB of float64 pairs in 32 us (7.4 TB/s, part of it from the
// last-level cache), 126 MB of float32 pairs in 22.5 us, of 42 and 31 us per iteration; the chain's two kernels
// moved 483 and 301 MB in 107 and 71.  Measured at 1M rows and not kept: 1024 threads with 128 registers (y in
// memory or scratch: 50 and 35 us), the next batch of entries requested while one is multiplied (48 and 42 us: the
// registers it takes shorten the batches), float64 batches of 5 and 9 pairs (44.6 and 48 us against 42.3 with 3),
// mixed batches of 3 and 5 (35.4 and 35.7 us against 31.0 with 9).
#pragma once

#include "pcg_kernels.hpp"
#include "team.hpp"

namespace shell {

namespace {

// How a team solve starts: from r = -g; from the residual in d.r with y added to (a refinement pass); or
// where the previous launch of the same solve stopped.
enum : int { kTeamFresh = 0, kTeamRefine = 1, kTeamResume = 2 };

// A member runs 512 threads (two waves per SIMD, 256 registers each).  It holds the first kTeamResident pairs of each
// row's entries in registers for the whole solve: with up to 1024 rows, in mixed precision up to 1536, nine pairs
// (the eighteen neighbours of a regular triangle-model row), so that an iteration reads no matrix at all, with
// up to 1536 in float64 a third of them; the others it streams in batches of kTeamBatch pairs.  The three rows per
// thread at 393129 vertices: 24.4 -> 23.1 us per iteration FP64 and 18.5 -> 16.2 mixed against streaming all.  With
// four rows and more, holding some pairs shortens the batches and not their number: 26.9 -> 27.9 us FP64 (two
// pairs), 20.6 -> 20.0 mixed (six) at 524176, 27.0 -> 26.1 mixed (three) at 784996, and 1M spills.
constexpr int kTeamPairs = 9;
template <typename MR, int RPL>
constexpr int kTeamResident = RPL <= 2 ? kTeamPairs : RPL == 3 ? (sizeof(MR) == 8 ? 3 : kTeamPairs) : 0;
template <typename MR>
constexpr int kTeamBatch = sizeof(MR) == 8 ? 3 : 9;

// LDS of a member: the directions of its rows and its halo, and of its rows the diagonal (float64: m + dt^2 K_ii;
// mixed: the mass and the Jacobi entry).
template <typename VR>
constexpr size_t team_lds(int rows, int halo) {
    return size_t(rows + halo) * 3 * sizeof(VR) + size_t(rows) * 8;
}

template <typename VR, typename MR, int RPL>
__global__ __launch_bounds__(kTeamThreads) void k_team_pcg(const SolveDesc* __restrict__ descs,
                                                const WorkItem* __restrict__ items, int mode, int limit, int every,
                                                uint64_t wait_ticks) {
    typedef typename Pair<MR>::type MR2;
    constexpr bool mixed = sizeof(VR) == 4;
    constexpr int T = kTeamThreads, NW = T / 64, B = kTeamBatch<MR>, RES = kTeamResident<MR, RPL>,
                  REM = RES == kTeamPairs ? 2 : 3;
    static_assert(RES % 3 == 0, "the held pairs are used in threes");
    extern __shared__ unsigned char smem_raw[];
    VR* ps = reinterpret_cast<VR*>(smem_raw);
    __shared__ double shA[3 * NW], outA[3 * NW], shB[6 * NW], outB[6 * NW];
    const WorkItem wi = items[blockIdx.x];
    const SolveDesc& d = descs[wi.mesh];
    const int R = d.trows, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long nv = d.nv, base = long(wi.unit) * R;
    const double dt2 = d.dt2;
    PcgState* st = d.st;
    __shared__ int lost;
    if (threadIdx.x == 0) lost = 0;
    const TeamMeet tm{d.slots, &st[0].gone, &lost, d.tmembers, wi.unit, wait_ticks};
    const int h0 = G(d.hptr)[wi.unit], nh = G(d.hptr)[wi.unit + 1] - h0;
    const gbl<const int32_t>* hc = G(d.hcols) + h0;
    VR* ydst = static_cast<VR*>(d.y);

    typedef typename Row<VR>::bits_t Bits;
    // The recurrence's state lives in LDS, double-buffered: lane c of every wave takes column c's step, the
    // first wave stores it.
    struct Rec {
        double rz[3], rr[3], tol2[3];
        int iters[3], active[3], budget[3], nonfinite[3];
    };
    __shared__ Rec rec[2];

    double r[RPL][3];
    VR y[RPL][3];
    double* dg = reinterpret_cast<double*>(ps + 3 * (R + nh));  // FP64: the diagonal, zero on fixed rows
    float* jac = reinterpret_cast<float*>(ps + 3 * (R + nh));   // mixed: the Jacobi entry, zero on fixed rows,
    float* mas = jac + R;                                       // and the mass
    unsigned send = 0;
    const long slice0 = base >> 6;
    const int64_t tp0 = G(d.tptr)[slice0];
    int off[RPL], w[RPL];  // first slot of the thread's slice (from tp0) and its pairs per row; wave-uniform
    MR2 mv[RPL][RES > 0 ? RES : 1];
    uint32_t mc[RPL][RES > 0 ? RES : 1];
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
        const int lr = s * T + int(threadIdx.x), lw = s * T + wave * 64;
        const long i = base + lr;
        // slices are whole waves: one that starts inside the member's rows and the mesh is read
        const bool live = lw < R && base + lw < nv;
        const long slice = live ? (base + lw) >> 6 : slice0;
        w[s] = live ? __builtin_amdgcn_readfirstlane(G(d.twid)[slice]) : 0;
        off[s] = __builtin_amdgcn_readfirstlane(int(G(d.tptr)[slice] - tp0));
        if constexpr (RES > 0) {
            const gbl<const MR2>* gv = G(static_cast<const MR2*>(d.tval)) + tp0 + off[s];
            const gbl<const uint32_t>* gc = G(d.tcol) + tp0 + off[s];
#pragma unroll
            for (int u = 0; u < RES; ++u) {
                const bool in = u < w[s];
                const int at = 64 * (in ? u : 0) + lane;
                const MR2 v = gv[at];
                mv[s][u].x = in ? v.x : MR(0);
                mv[s][u].y = in ? v.y : MR(0);
                mc[s][u] = in ? gc[at] : 0u;
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r[s][c] = 0.0;
            y[s][c] = VR(0);
        }
        if (lr < R) {  // also the rows past nv of the last slice: fixed, their direction stays zero
#pragma unroll
            for (int c = 0; c < 3; ++c) ps[3 * lr + c] = VR(0);
            if constexpr (mixed)
                jac[lr] = mas[lr] = 0.f;
            else
                dg[lr] = 0.0;
        }
        if (live && i < nv) {
            const VR di = G(static_cast<const VR*>(d.dinv))[i];
            if constexpr (mixed) {
                jac[lr] = di;
                mas[lr] = float(G(d.mass)[i]);
            } else {
                if (di != VR(0)) dg[lr] = G(d.mass)[i] + dt2 * G(d.kdiag)[i];
            }
            if (G(d.tsend)[i]) send |= 1u << s;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[s][c] = mode == kTeamFresh ? -G(static_cast<const double*>(d.g))[3 * i + c] : G(d.r)[3 * i + c];
                if (mode != kTeamFresh)
                    y[s][c] = G(ydst)[3 * i + c];
                else if constexpr (mixed)
                    G(d.y64)[3 * i + c] = 0.0;
                if (mode == kTeamResume) ps[3 * lr + c] = G(static_cast<const VR*>(d.p0))[3 * i + c];
            }
        }
    }
    // the Jacobi entry of a row of this thread (zero on fixed rows and past the member's)
    auto jacobi = [&](int lr) -> VR {
        if (lr >= R) return VR(0);
        if constexpr (mixed) {
            return jac[lr];
        } else {
            const double v = dg[lr];
            return v != 0.0 ? inv_fast(v) : 0.0;
        }
    };
    if (mode == kTeamResume)
        for (int h = threadIdx.x; h < nh; h += T)
#pragma unroll
            for (int c = 0; c < 3; ++c) ps[3 * (R + h) + c] = G(static_cast<const VR*>(d.p0))[3L * hc[h] + c];
    if (threadIdx.x == 0) {
        Rec o{};
        if (mode == kTeamResume) {
            const PcgState& q = st[1];
            for (int c = 0; c < 3; ++c) {
                o.rz[c] = q.rz[c];
                o.rr[c] = q.rr[c];
                o.tol2[c] = q.tol2[c];
                o.iters[c] = q.iters[c];
                o.active[c] = q.active[c];
                o.budget[c] = q.budget;
                o.nonfinite[c] = q.nonfinite;
            }
        }
        rec[0] = o;
    }
    // sampled durations (thread 0 of the first member), kept in LDS
    __shared__ uint64_t ticks[2], since;
    __shared__ int samples;
    if (threadIdx.x == 0) {
        ticks[0] = ticks[1] = 0;
        samples = 0;
    }

    // The rows that other members read, by iteration parity.
    auto rows_of = [&](int par) { return static_cast<Bits*>(par & 1 ? d.p1 : d.q); };
    auto unset_rows = [&](int par) {
        Bits* zx = rows_of(par);
        const unsigned at = 3u * (unsigned(base) + unsigned(here(int(threadIdx.x))));
#pragma unroll
        for (int s = 0; s < RPL; ++s)
            if (send >> s & 1u)
#pragma unroll
                for (int c = 0; c < 3; ++c) agent_store(zx + (here(at) + unsigned(3 * s * T + c)), Row<VR>::unset);
    };
    // z = D^-1 r: published where others read it; the sums r.z, r.r
    auto publish_rows = [&](int par, double (&acc)[6]) {
        Bits* zx = rows_of(par);
        const int tid = here(int(threadIdx.x));
        const unsigned at = 3u * (unsigned(base) + unsigned(tid));
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const VR di = jacobi(s * T + here(tid));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const VR z = di * VR(r[s][c]);
                acc[c] += r[s][c] * double(z);
                acc[3 + c] += r[s][c] * r[s][c];
                if (send >> s & 1u) agent_store(zx + (here(at) + unsigned(3 * s * T + c)), Row<VR>::bits(z));
            }
            if (RPL > 2) __builtin_amdgcn_sched_barrier(0);  // one row's temporaries at a time
        }
    };
    {
        // the first rows replace whatever an earlier solve left, so they are in place before the first sums
        double acc[6] = {0, 0, 0, 0, 0, 0};
        unset_rows(1);
        publish_rows(0, acc);
        wait_stores();
        wave_partials<6>(acc, shB);
    }
    __syncthreads();
    team_send<6>(tm, 1, 0, shB);
    int n = 0;
    // iterations before this launch (the last of them is counted at the first meeting)
    const int before =
        mode == kTeamResume ? 1 + max(st[1].iters[0], max(st[1].iters[1], st[1].iters[2])) : 0;
    bool done = false;
    for (;; ++n) {
        // r.z and r.r of the residual as it stands: the recurrence moves on
        VR b[3];
        {
            const double tb = team_receive<6>(tm, 1, n, shB, outB), tr = __shfl(tb, lane + 3, 64);
            if (lost) return;
            team_unset<3>(tm, 0, n + 1);  // the previous product's sums: every member has read them
            double beta = 0.0;
            int active = 0;
            if (lane < 3) {
                const Rec& o = rec[n & 1];
                Rec& x = rec[(n + 1) & 1];
                const int c = lane, target = d.target[c];
                double rz = o.rz[c], rr = o.rr[c], tol2 = o.tol2[c];
                int iters = o.iters[c], budget = o.budget[c], nonfinite = o.nonfinite[c];
                active = o.active[c];
                if (n == 0 && mode != kTeamResume) {
                    tol2 = d.tol2_abs[c] > 0.0 ? d.tol2_abs[c] : d.rtol2 * tr;
                    active = 0 < target && (d.replay || tr > tol2);
                    rz = tb;
                    rr = tr;
                } else if (active) {
                    beta = rz != 0.0 ? tb / rz : 0.0;
                    iters += 1;
                    const bool more = d.replay || tr > tol2;
                    if (!d.replay && iters >= target && more) budget = 1;
                    active = iters < target && more;
                    if (!isfinite(tr)) {
                        nonfinite = 1;
                        active = 0;
                    }
                    rz = tb;
                    rr = tr;
                }
                if (wave == 0) {
                    x.rz[c] = rz;
                    x.rr[c] = rr;
                    x.tol2[c] = tol2;
                    x.iters[c] = iters;
                    x.active[c] = active;
                    x.budget[c] = budget;
                    x.nonfinite[c] = nonfinite;
                }
            }
            done = __ballot(active != 0) == 0;
            for (int c = 0; c < 3; ++c) b[c] = VR(read_lane(beta, c));
        }
        if (done) break;
        const bool sample = every > 0 && n % every == 0 && wi.unit == 0 && threadIdx.x == 0;
        if (sample) since = wall_clock64();
        // p = z + beta p: the first halo column's z is requested, the own rows advance, then the halo does
        const int tid = here(int(threadIdx.x));
        {
            const Bits* zx = rows_of(n);
            Bits zb[3] = {0, 0, 0};
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
                    const VR di = jacobi(lr);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const VR z = di * VR(r[s][c]);
                        ps[3 * lr + c] = b[c] != VR(0) ? fma(b[c], ps[3 * lr + c], z) : z;
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
                while (zb[0] == Row<VR>::unset || zb[1] == Row<VR>::unset || zb[2] == Row<VR>::unset) {
                    if (wait.over(tm)) {
                        team_give_up(tm);
                        break;
                    }
#pragma unroll
                    for (int c = 0; c < 3; ++c) zb[c] = agent_load(zx + col + c);
                }
                VR* pj = ps + 3 * (R + h);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const VR z = Row<VR>::value(zb[c]);
                    pj[c] = b[c] != VR(0) ? fma(b[c], pj[c], z) : z;
                }
            }
        }
        __syncthreads();
        if (lost) return;
        // q = (M + dt^2 K_s) p, fixed rows zero; p.q
        VR q[RPL][3];
        double pq[3] = {0, 0, 0};
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const int lr = s * T + here(tid);
            const unsigned ln = unsigned(here(tid)) & 63u;
            VR pi[3] = {0, 0, 0};
            MR a[3] = {0, 0, 0};
            if (w[s] > 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) pi[c] = ps[3 * lr + c];
            auto use = [&](MR2 v, uint32_t cc) {  // one pair
                const VR* p0 = ps + 3 * (cc & 0xffffu);
                const VR* p1 = ps + 3 * (cc >> 16);
#pragma unroll
                for (int c = 0; c < 3; ++c) a[c] = fma(v.x, kDiffForm<MR> ? MR(p0[c]) - MR(pi[c]) : MR(p0[c]), a[c]);
#pragma unroll
                for (int c = 0; c < 3; ++c) a[c] = fma(v.y, kDiffForm<MR> ? MR(p1[c]) - MR(pi[c]) : MR(p1[c]), a[c]);
            };
            int k = RES;
            if constexpr (RES > 0) {
#pragma unroll
                for (int u = 0; u < RES; u += 3)
                    if (u < w[s]) {  // wave-uniform; the pairs past the row's end hold zeros
                        use(mv[s][u], mc[s][u]);
                        use(mv[s][u + 1], mc[s][u + 1]);
                        use(mv[s][u + 2], mc[s][u + 2]);
                    }
            } else {
                k = 0;
            }
            const gbl<const MR2>* gv = G(static_cast<const MR2*>(d.tval)) + tp0 + off[s];
            const gbl<const uint32_t>* gc = G(d.tcol) + tp0 + off[s];
            if constexpr (RES < kTeamPairs)
                for (; k + B <= w[s]; k += B) {
                    MR2 v[B];
                    uint32_t cc[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        v[u] = gv[64u * unsigned(k + u) + ln];
                        cc[u] = gc[64u * unsigned(k + u) + ln];
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        use(v[u], cc[u]);
                        __builtin_amdgcn_sched_barrier(0);  // one pair's directions in registers at a time
                    }
                }
            for (; k < w[s]; k += REM) {  // the rest of the row (wave-uniform)
                MR2 v[REM];
                uint32_t cc[REM];
#pragma unroll
                for (int u = 0; u < REM; ++u) {
                    const unsigned at = 64u * unsigned(min(k + u, w[s] - 1)) + ln;
                    v[u] = gv[at];
                    cc[u] = gc[at];
                }
#pragma unroll
                for (int u = 0; u < REM; ++u)
                    if (k + u < w[s]) use(v[u], cc[u]);
            }
            MR dii = 0;
            bool fixed = true;
            if (w[s] > 0) {
                if constexpr (mixed) {
                    dii = mas[lr];
                    fixed = jac[lr] == 0.f;
                } else {
                    dii = dg[lr];
                    fixed = dii == MR(0);
                }
            }
            VR qv[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) qv[c] = fixed ? VR(0) : VR(fma(dii, MR(pi[c]), MR(dt2) * a[c]));
            if (d.partial_held && w[s] > 0 && base + lr < nv) {
                const unsigned held = G(d.pinned)[base + lr];
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (held >> c & 1u) qv[c] = VR(0);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                pq[c] = here(fma(double(pi[c]), double(qv[c]), pq[c]));  // now, not with every row's p and q held
                q[s][c] = qv[c];
            }
        }
        wait_stores();  // the slots and rows unset since the last product have reached memory long since
        wave_partials<3>(pq, shA);
        __syncthreads();
        double al[3];
        {
            team_send<3>(tm, 0, n, shA);
            const double ta = team_receive<3>(tm, 0, n, shA, outA);
            if (lost) return;
            team_unset<6>(tm, 1, n);  // this iteration's first sums and rows: every member has read them
            unset_rows(n);
            if (sample) {
                const uint64_t now = wall_clock64();
                ticks[0] += now - since;
                since = now;
            }
            double alpha = 0.0;
            if (lane < 3) {
                const Rec& o = rec[(n + 1) & 1];
                if (o.active[lane] && ta != 0.0) alpha = o.rz[lane] / ta;
            }
            for (int c = 0; c < 3; ++c) al[c] = read_lane(alpha, c);
        }
#pragma unroll
        for (int s = 0; s < RPL; ++s) {
            const int lr = s * T + here(tid);
            if (w[s] > 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    y[s][c] = VR(fma(al[c], double(ps[3 * lr + c]), double(y[s][c])));
                    r[s][c] = fma(-al[c], double(q[s][c]), r[s][c]);
                }
            if (RPL > 2) __builtin_amdgcn_sched_barrier(0);
        }
        {
            double acc[6] = {0, 0, 0, 0, 0, 0};
            publish_rows(n + 1, acc);
            wave_partials<6>(acc, shB);
        }
        __syncthreads();
        team_send<6>(tm, 1, n + 1, shB);
        // mixed precision: the float32 increment into its float64 sum (see kFoldIters), while the sums travel
        if (mixed && (before + n) % kFoldIters == kFoldIters - 1) {
#pragma unroll
            for (int s = 0; s < RPL; ++s) {
                const long i = base + s * T + here(tid);
                if (w[s] > 0 && i < nv)
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        G(d.y64)[3 * i + c] += double(y[s][c]);
                        y[s][c] = VR(0);
                    }
            }
        }
        if (sample) {
            ticks[1] += wall_clock64() - since;
            ++samples;
        }
        if (n + 1 == limit) break;  // the next launch takes it from here
    }
#pragma unroll
    for (int s = 0; s < RPL; ++s) {
        const int lr = s * T + here(int(threadIdx.x));
        const long i = base + lr;
        if (w[s] > 0 && i < nv)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                G(ydst)[3 * i + c] = y[s][c];
                if (!done) {
                    G(d.r)[3 * i + c] = r[s][c];
                    G(static_cast<VR*>(d.p0))[3 * i + c] = ps[3 * lr + c];
                }
            }
    }
    if (wi.unit == 0 && threadIdx.x == 0) {
        const Rec& q = rec[(n + 1) & 1];  // thread 0 is a lane of the wave that stored it
        PcgState& o = st[1];
        for (int c = 0; c < 3; ++c) {
            o.rz[c] = q.rz[c];
            o.rr[c] = q.rr[c];
            o.tol2[c] = q.tol2[c];
            o.iters[c] = q.iters[c];
            o.target[c] = d.target[c];
            o.active[c] = q.active[c];
        }
        o.done = done;
        o.budget = q.budget[0] | q.budget[1] | q.budget[2];
        o.nonfinite = q.nonfinite[0] | q.nonfinite[1] | q.nonfinite[2];
        o.sample[0] = double(ticks[0]);
        o.sample[1] = double(ticks[1]);
        o.samples = samples;
    }
}

// the slots and flags of a launch's meshes
__global__ __launch_bounds__(kRedBlk) void k_team_clear(const SolveDesc* __restrict__ descs,
                                                        const int32_t* __restrict__ meshes) {
    const SolveDesc& d = descs[meshes[blockIdx.x]];
    team_clear(d.slots, &d.st[0].gone, d.tmembers);
}

}  // namespace

}  // namespace shell
