// Constant bending Hessian K = K_s (x) I3 (eqs 21, 41, 53; the shell models reuse it), assembled once,
// and its product inside the implicit step.
//
// K_s = sum over stencils of P^T G P with G = B^T D B (k x k): every stencil block of the paper's
// Hessian is G (x) I3, so only the scalar K_s is stored.  Storage is SELL-64: slice s holds rows
// 64s..64s+63 and entry q of row i sits at sptr[s] + 64 q + (i mod 64), so the 64 lanes of a wave read
// 64 consecutive values and column ids per step (fully coalesced), one row per lane, no reduction.
#include <algorithm>

#include "devmath.hpp"
#include "host_threads.hpp"
#include "internal.hpp"
#include "spmv.hpp"

namespace shell {

namespace {

// slot of column c in row i (columns sorted within the row's rowlen entries)
__device__ __forceinline__ long find_slot(const int32_t* __restrict__ scol, const int64_t* __restrict__ sptr,
                                          const int32_t* __restrict__ rowlen, long i, int c) {
    long s0 = sptr[i >> 6] + (i & 63);
    int lo = 0, hi = rowlen[i] - 1;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (scol[s0 + 64L * mid] < c)
            lo = mid + 1;
        else
            hi = mid;
    }
    return s0 + 64L * lo;
}

// Row i of K_s: over the stencils that contain vertex i (as local vertex j), in ascending order, row j of
// the stencil's block B^T D B.  One thread per row writes only its own slots, so the sums take the same
// order in every run.
template <int K, int R>
__global__ void assemble_rows(const int64_t* __restrict__ inc_ptr, const int64_t* __restrict__ inc,
                              const int32_t* __restrict__ idx, const double* __restrict__ B, long ns,
                              const int32_t* __restrict__ missing, double kb, double nu,
                              const int32_t* __restrict__ scol, const int64_t* __restrict__ sptr,
                              const int32_t* __restrict__ rowlen, long nv, double* __restrict__ val) {
    const long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i >= nv) return;
    for (int64_t e = inc_ptr[i]; e < inc_ptr[i + 1]; ++e) {
        const long s = long(inc[e] >> 3);
        const int j = int(inc[e] & 7);
        int v[K];
        double Bm[R][K];
        for (int l = 0; l < K; ++l) v[l] = idx[l * ns + s];
        for (int r = 0; r < R; ++r)
            for (int l = 0; l < K; ++l) Bm[r][l] = B[(r * K + l) * ns + s];
        const int miss = missing ? missing[s] : 0;
        // D B (the stiffness is already folded into B for edges; triangles carry D_b)
        double DB[R][K];
        if constexpr (R == 1) {
            for (int l = 0; l < K; ++l) DB[0][l] = Bm[0][l];
        } else {
            const double t = 0.5 * (1.0 - nu);
            for (int l = 0; l < K; ++l) {
                DB[0][l] = kb * (Bm[0][l] + nu * Bm[1][l]);
                DB[1][l] = kb * (nu * Bm[0][l] + Bm[1][l]);
                DB[2][l] = kb * t * Bm[2][l];
            }
        }
        for (int l = 0; l < K; ++l) {
            if (l >= 3 && (miss & (1 << (l - 3)))) continue;
            double g = 0.0;
            for (int r = 0; r < R; ++r) g += Bm[r][j] * DB[r][l];
            val[find_slot(scol, sptr, rowlen, i, v[l])] += g;
        }
    }
}

__global__ void fill_zero(double* __restrict__ p, long n) {
    long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

__global__ void extract_diag(const double* __restrict__ val, const int64_t* __restrict__ dslot, long nv,
                             double* __restrict__ kdiag) {
    long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i < nv) kdiag[i] = dslot[i] >= 0 ? val[dslot[i]] : 0.0;
}

__global__ void to_float(const double* __restrict__ a, float* __restrict__ b, long n) {
    long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i < n) b[i] = float(a[i]);
}

// The off-diagonal entries of row i in the pairs of a team solve: the value pairs (float64 or float32).
template <typename MR>
__global__ void team_values(const int32_t* __restrict__ scol, const double* __restrict__ val,
                            const int64_t* __restrict__ sptr, const int32_t* __restrict__ rowlen, long nv,
                            const int64_t* __restrict__ tptr, const int32_t* __restrict__ twid,
                            MR* __restrict__ tval) {
    const long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i >= 64 * ((nv + 63) / 64)) return;
    const long s = i >> 6, s0 = sptr[s] + (i & 63), t0 = tptr[s] + (i & 63);
    const int n = i < nv ? rowlen[i] : 0;
    int o = 0;
    for (int k = 0; k < n; ++k) {
        if (scol[s0 + 64L * k] == i) continue;
        tval[2 * (t0 + 64L * (o >> 1)) + (o & 1)] = MR(val[s0 + 64L * k]);
        ++o;
    }
    for (; o < 2 * twid[s]; ++o) tval[2 * (t0 + 64L * (o >> 1)) + (o & 1)] = MR(0);
}

// Their columns as ids of a member of R rows: an own row's offset, or R + the halo column's index.
__global__ void team_columns(const int32_t* __restrict__ scol, const int64_t* __restrict__ sptr,
                             const int32_t* __restrict__ rowlen, long nv, const int64_t* __restrict__ tptr,
                             const int32_t* __restrict__ twid, int R, const int32_t* __restrict__ hptr,
                             const int32_t* __restrict__ hcols, uint32_t* __restrict__ tcol) {
    const long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    if (i >= 64 * ((nv + 63) / 64)) return;
    const long s = i >> 6, s0 = sptr[s] + (i & 63), t0 = tptr[s] + (i & 63);
    const long m = i / R, base = m * R;
    const int n = i < nv ? rowlen[i] : 0;
    const uint32_t self = uint32_t(i - base);
    int o = 0;
    uint32_t pair = 0;
    auto put = [&](uint32_t id) {
        pair = (o & 1) ? pair | (id << 16) : id;
        if (o & 1) tcol[t0 + 64L * (o >> 1)] = pair;
        ++o;
    };
    for (int k = 0; k < n; ++k) {
        const int c = scol[s0 + 64L * k];
        if (c == i) continue;
        if (c >= base && c < base + R) {
            put(uint32_t(c - base));
        } else {
            int lo = hptr[m], hi = hptr[m + 1] - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (hcols[mid] < c)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            put(uint32_t(R + lo - hptr[m]));
        }
    }
    while (o < 2 * twid[s]) put(self);
}

// q = diag(mass) p + dt2 K_s p over 3 columns.  With `perm` q is in the caller's order, and with THROUGH p and mass
// are too: the matrix stream bounds the kernel (262144 rows of 19 entries: 50 of 65 MB, 10.4 us at the rate of a
// copy), and gather and scatter kernels around it took as long again (24.9 us; now 13.4).
template <bool THROUGH>
__global__ void apply_sell(const int32_t* __restrict__ scol, const double* __restrict__ val,
                           const int64_t* __restrict__ sptr, const int32_t* __restrict__ width,
                           const int32_t* __restrict__ gptr, const int32_t* __restrict__ gcols,
                           const uint16_t* __restrict__ lcol, long nv, const int32_t* __restrict__ perm,
                           const double* __restrict__ mass, double dt2, const double* __restrict__ p,
                           double* __restrict__ q) {
    long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
    extern __shared__ unsigned char smem_raw[];
    double* ps = reinterpret_cast<double*>(smem_raw);
    const long to = perm && i < nv ? perm[i] : i;  // where row i goes
    const long from = THROUGH ? to : i;
    double m = 0.0, px = 0.0, py = 0.0, pz = 0.0;
    if (i < nv) {
        if (mass) m = mass[from];
        px = p[3 * from];
        py = p[3 * from + 1];
        pz = p[3 * from + 2];
    }
    if (THROUGH || gptr) {
        const int a = gptr[blockIdx.x], n = gptr[blockIdx.x + 1] - a;
        for (int k = threadIdx.x; k < n; k += blockDim.x) {
            const long c = THROUGH ? perm[gcols[a + k]] : gcols[a + k];
            ps[3 * k] = p[3 * c];
            ps[3 * k + 1] = p[3 * c + 1];
            ps[3 * k + 2] = p[3 * c + 2];
        }
        __syncthreads();
    }
    if (i >= nv) return;
    double ax, ay, az;
    if (THROUGH || gptr)
        sell_row_product_staged<double, double>(lcol, val, sptr, width, i, ps, ax, ay, az);
    else
        sell_row_product<double, double>(scol, val, sptr, width, i, p, ax, ay, az);
    q[3 * to] = fma(m, px, dt2 * ax);
    q[3 * to + 1] = fma(m, py, dt2 * ay);
    q[3 * to + 2] = fma(m, pz, dt2 * az);
}

}  // namespace

void launch_assemble(shell_hessian_s& h, hipStream_t s) {
    shell_stencils_s& st = *h.st;
    const long nslots = h.pat.nslots;
    fill_zero<<<(nslots + 255) / 256, 256, 0, s>>>(h.val.p, nslots);
    SHELL_HIP(hipGetLastError());
    const long ns = st.ns;
    DevArray<int32_t> md;
    if (!model_is_edge(st.model) && ns) {
        std::vector<int32_t> mask(size_t(ns), 0);
        for (long q = 0; q < ns; ++q)
            for (int L = 0; L < 3; ++L)
                if (st.h_idx[size_t(6 * q + 3 + L)] < 0) mask[size_t(q)] |= 1 << L;
        md.alloc(size_t(ns));
        md.upload(mask.data(), size_t(ns), s);
    }
    if (ns) {
        const Incidence inc = build_incidence(st.h_idx, st.k, ns, st.nv);
        DevArray<int64_t> iptr(inc.ptr.size()), icode(std::max<size_t>(inc.code.size(), 1));
        iptr.upload(inc.ptr.data(), inc.ptr.size(), s);
        icode.upload(inc.code.data(), inc.code.size(), s);
        const long grid = (st.nv + 255) / 256;
        if (model_is_edge(st.model))
            assemble_rows<4, 1><<<grid, 256, 0, s>>>(iptr.p, icode.p, st.idx.p, st.B.p, ns, nullptr, st.kb,
                                                     st.poisson, h.scol.p, h.sptr.p, h.rowlen.p, st.nv, h.val.p);
        else
            assemble_rows<6, 3><<<grid, 256, 0, s>>>(iptr.p, icode.p, st.idx.p, st.B.p, ns, md.p, st.kb,
                                                     st.poisson, h.scol.p, h.sptr.p, h.rowlen.p, st.nv, h.val.p);
        SHELL_HIP(hipGetLastError());
        SHELL_HIP(hipStreamSynchronize(s));  // the incidence lists are released on return
    }
    DevArray<int64_t> dslot(static_cast<size_t>(st.nv));
    dslot.upload(h.pat.dslot.data(), size_t(st.nv), s);
    if (st.nv) {
        extract_diag<<<(st.nv + 255) / 256, 256, 0, s>>>(h.val.p, dslot.p, st.nv, h.kdiag.p);
        SHELL_HIP(hipGetLastError());
    }
    if (h.valf.p) {
        to_float<<<(nslots + 255) / 256, 256, 0, s>>>(h.val.p, h.valf.p, nslots);
        SHELL_HIP(hipGetLastError());
    }
    SHELL_HIP(hipStreamSynchronize(s));  // temporaries are released on return
}

int compute_units() {
    int dev = 0, cus = 0;
    SHELL_HIP(hipGetDevice(&dev));
    SHELL_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    return cus;
}

std::unique_ptr<TeamPart> build_part(shell_hessian_s& h, int64_t R, size_t real, hipStream_t s,
                                     const std::vector<int64_t>* row2, const std::vector<int32_t>* col2,
                                     std::vector<std::vector<int32_t>>* lists) {
    const SellPattern& P = h.pat;
    const int64_t nv = P.nv, members = (nv + R - 1) / R;
    if (R > kTeamMaxRows || !h.tpairs) return nullptr;
    std::vector<std::vector<int32_t>> halo(static_cast<size_t>(members));
    host_parallel_for(members, [&](int64_t a, int64_t b) {
        for (int64_t m = a; m < b; ++m) {
            auto& v = halo[size_t(m)];
            const int64_t lo = m * R, hi = std::min(nv, lo + R);
            for (int64_t e = P.rowptr[size_t(lo)]; e < P.rowptr[size_t(hi)]; ++e)
                if (P.col[size_t(e)] < lo || P.col[size_t(e)] >= hi) v.push_back(P.col[size_t(e)]);
            if (row2)
                for (int64_t e = (*row2)[size_t(lo)]; e < (*row2)[size_t(hi)]; ++e)
                    if ((*col2)[size_t(e)] < lo || (*col2)[size_t(e)] >= hi) v.push_back((*col2)[size_t(e)]);
            std::sort(v.begin(), v.end());
            v.erase(std::unique(v.begin(), v.end()), v.end());
        }
    });
    auto part = std::make_unique<TeamPart>();
    part->rows = int32_t(R);
    part->members = int32_t(members);
    std::vector<int32_t> hptr(size_t(members + 1), 0), hcols;
    std::vector<uint8_t> send(size_t(nv), 0);
    for (int64_t m = 0; m < members; ++m) {
        const auto& v = halo[size_t(m)];
        part->max_halo = std::max(part->max_halo, int32_t(v.size()));
        hcols.insert(hcols.end(), v.begin(), v.end());
        hptr[size_t(m + 1)] = int32_t(hcols.size());
        for (int32_t c : v) send[size_t(c)] = 1;
    }
    // directions and diagonal in LDS; local columns in 16 bits
    if (size_t(R + part->max_halo) * 3 * real + size_t(R) * 8 > kTeamLds || R + part->max_halo > 65536) return nullptr;
    part->hptr.alloc(hptr.size());
    part->hptr.upload(hptr.data(), hptr.size(), s);
    part->hcols.alloc(std::max<size_t>(hcols.size(), 1));
    part->hcols.upload(hcols.data(), hcols.size(), s);
    part->send.alloc(send.size());
    part->send.upload(send.data(), send.size(), s);
    part->col.alloc(size_t(h.tpairs));
    const unsigned grid = unsigned((64 * P.nslices + 255) / 256);
    team_columns<<<grid, 256, 0, s>>>(h.scol.p, h.sptr.p, h.rowlen.p, nv, h.tptr.p, h.twid.p, int(R), part->hptr.p,
                                      part->hcols.p, part->col.p);
    SHELL_HIP(hipGetLastError());
    SHELL_HIP(hipStreamSynchronize(s));  // the host lists are released on return
    if (lists) *lists = std::move(halo);
    return part;
}

// The off-diagonal entries in pairs, in the stencils' precision.
static void build_team_values(shell_hessian_s& h, hipStream_t s) {
    const SellPattern& P = h.pat;
    const int64_t nv = P.nv;
    // slices of pairs
    std::vector<int64_t> tptr(size_t(P.nslices + 1), 0);
    std::vector<int32_t> twid(size_t(P.nslices), 1);
    for (int64_t sl = 0; sl < P.nslices; ++sl) {
        int w = 1;
        for (int64_t i = 64 * sl; i < std::min(nv, 64 * sl + 64); ++i)
            w = std::max(w, (P.rowlen[size_t(i)] - (P.dslot[size_t(i)] >= 0 ? 1 : 0) + 1) / 2);
        twid[size_t(sl)] = w;
        tptr[size_t(sl + 1)] = tptr[size_t(sl)] + 64 * int64_t(w);
    }
    h.tpairs = tptr[size_t(P.nslices)];
    h.tptr.alloc(tptr.size());
    h.tptr.upload(tptr.data(), tptr.size(), s);
    h.twid.alloc(twid.size());
    h.twid.upload(twid.data(), twid.size(), s);
    const unsigned grid = unsigned((64 * P.nslices + 255) / 256);
    if (h.valf.p) {
        h.tvalf.alloc(size_t(2 * h.tpairs));
        team_values<float><<<grid, 256, 0, s>>>(h.scol.p, h.val.p, h.sptr.p, h.rowlen.p, nv, h.tptr.p, h.twid.p,
                                                h.tvalf.p);
    } else {
        h.tval.alloc(size_t(2 * h.tpairs));
        team_values<double><<<grid, 256, 0, s>>>(h.scol.p, h.val.p, h.sptr.p, h.rowlen.p, nv, h.tptr.p, h.twid.p,
                                                 h.tval.p);
    }
    SHELL_HIP(hipGetLastError());
    SHELL_HIP(hipStreamSynchronize(s));  // the host lists are released on return
}

void build_team(shell_hessian_s& h, hipStream_t s) {
    if (!h.pat.nv) return;
    const int64_t rows = team_rows(h.pat.nv, compute_units());
    if (rows > kTeamMaxRows) return;
    build_team_values(h, s);
    if (h.st->cfg_flags & SHELL_FLAG_MEMBRANE) return;  // its solver's part covers the tangent's columns too
    auto part = build_part(h, rows, h.valf.p ? sizeof(float) : sizeof(double), s);
    if (part) {
        h.parts.push_back(std::move(part));
        return;
    }
    h.tpairs = 0;
    h.tptr.release();
    h.twid.release();
    h.tval.release();
    h.tvalf.release();
}

const TeamPart* team_part(shell_hessian_s& h, int64_t rows, hipStream_t s) {
    std::lock_guard<std::mutex> lk(h.parts_mutex);
    if (h.parts.empty()) return nullptr;
    const TeamPart* own = h.parts[0].get();
    if (rows <= own->rows || own->members == 1) return own;
    for (const auto& p : h.parts)
        if (p->rows == rows) return p.get();
    auto part = build_part(h, rows, h.valf.p ? sizeof(float) : sizeof(double), s);
    if (!part) return own;
    h.parts.push_back(std::move(part));
    return h.parts.back().get();
}

void launch_apply(const shell_hessian_s& h, const double* mass, double dt2, const double* p, double* q,
                  hipStream_t s, const int32_t* perm, bool through) {
    const long nv = h.pat.nv;
    if (!nv) return;
    const size_t lds = h.gptr.p ? size_t(h.pat.max_gcols) * 3 * sizeof(double) : 0;
    const unsigned grid = unsigned((nv + kRowGroup - 1) / kRowGroup);
    auto* kernel = through ? apply_sell<true> : apply_sell<false>;
    kernel<<<grid, kRowGroup, lds, s>>>(h.scol.p, h.val.p, h.sptr.p, h.width.p, h.gptr.p, h.gcols.p, h.lcol.p, nv, perm,
                                        mass, dt2, p, q);
    SHELL_HIP(hipGetLastError());
}

}  // namespace shell
