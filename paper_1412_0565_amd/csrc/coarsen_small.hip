// Setup of the small levels in one workgroup: for a chain of levels of at
// most kChainMaxN vertices, the row pass (Gershgorin shift, heaviest
// neighbours), HEC (Algorithm 2, in the round-synchronous form of the grid
// kernels in setup.hip) and the Galerkin coarse graph (Section 2, the
// Proposition on restriction) run level after level inside one launch,
// separated only by workgroup barriers.  The grid kernels need about 40
// launches and 7 host synchronisations per level; on small levels those
// gaps, not the work, set the setup time.
//
// The Galerkin product sorts the fine entries of each coarse row in LDS, so
// the contributions to each coarse entry (a, b) are added in fine CSR order,
// the order the grid path's stable sort produces.  Results are bit-exact
// with the grid path and the oracle (integer and real weights alike).
#include "cmg_internal.h"

namespace cmg {

namespace {

constexpr uint8_t kSeedC = 1;
constexpr uint8_t kPartnerC = 2;
constexpr unsigned long long kNoKeyC = 0xFFFFFFFFFFFFFFFFull;

// Inclusive scan over a wavefront.
__device__ __forceinline__ int wave_scan_incl(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan of in(0..m-1), out(i, sum before i), by the whole workgroup
// (each thread a contiguous chunk); returns the total.  A chunk is read
// again as it is written, so out(i, .) may overwrite what in(i) reads.
// `sh` holds 17 ints.
template <class In, class Out>
__device__ __forceinline__ int chain_scan(int m, int* sh, In in, Out out) {
    const int T = blockDim.x, tid = threadIdx.x;
    const int per = (m + T - 1) / T;
    const int lo = min(m, tid * per), hi = min(m, lo + per);
    int s = 0;
    for (int i = lo; i < hi; ++i) s += in(i);
    const int inc = wave_scan_incl(s);
    const int wv = tid >> 6, nw = T >> 6;
    if ((tid & 63) == 63) sh[wv] = inc;
    __syncthreads();
    int off = 0, all = 0;
    for (int q = 0; q < nw; ++q) {
        if (q < wv) off += sh[q];
        all += sh[q];
    }
    int run = off + inc - s;
    for (int i = lo; i < hi; ++i) {
        const int x = in(i);
        out(i, run);
        run += x;
    }
    __syncthreads();
    return all;
}

// max over the workgroup of 4 doubles (exact, order independent)
__device__ void block_max4(double (&m)[4], double* sm) {
    for (int o = 32; o > 0; o >>= 1)
        for (int q = 0; q < 4; ++q) m[q] = fmax(m[q], __shfl_xor(m[q], o, kWave));
    const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 4; ++q) sm[q * 16 + wv] = m[q];
    __syncthreads();
    for (int q = 0; q < 4; ++q) {
        double r = 0.0;
        for (int w = 0; w < nw; ++w) r = fmax(r, sm[q * 16 + w]);
        m[q] = r;
    }
    __syncthreads();
}

// Longest fine row of a level this kernel coarsens (measured on MI355X:
// 3D-grid levels with 27-47 entries per row took 0.27-1.9 ms here against
// a few hundred microseconds on the grid kernels).
constexpr int kChainLongRow = 24;

// Everything per vertex or aggregate lives in LDS (16-bit ids, as a level
// has at most kChainMaxN = 8192 vertices); only the CSR arrays and the arenas
// of the levels produced are in memory.  The 8-byte slots of the greedy
// rounds are dead once the matching stands, as are the arrays of a phase once
// the next one stands; `tile` takes their space for the coarse rows.
constexpr int kChainTile = 13 * kChainThreads;  // contributions held at once
constexpr int kChainRuns = kChainTile / 64;
struct ChainLds {
    union {
        unsigned long long slot[kChainMaxN];
        struct {
            uint16_t agg[kChainMaxN];
            union {
                struct {
                    uint16_t rank[kChainMaxN];  // aggregate opened by a vertex
                    int32_t astart[kChainMaxN / 2];  // first member of each aggregate
                    int32_t acnt[kChainMaxN / 2];
                    union {
                        uint16_t h[kChainMaxN];
                        uint16_t members[kChainMaxN];
                    } v;
                    union {
                        struct {
                            uint8_t live[kChainMaxN], state[kChainMaxN];
                        } f;
                        int32_t rcount[kChainMaxN / 2];
                    } l;
                } m;
                struct {
                    uint32_t key[kChainTile];   // coarse column << 19 | fine entry
                    uint16_t row[kChainTile];
                    uint16_t head[kChainTile];  // slots that open a coarse entry
                } tile;
            } t;
        } a;
    } u;
    union {
        uint16_t pair[kChainMaxN];
        int32_t afill[kChainMaxN / 2];
        uint16_t off[kChainMaxN];  // a vertex's first slot within its coarse row
    } p;
    union {
        uint16_t root[kChainMaxN];
        int32_t soff[kChainMaxN / 2 + 1];  // first slot of a coarse row
    } r;
};
static_assert(offsetof(ChainLds, u.a.t.m.v) >= sizeof(unsigned long long) * kChainMaxN, "alive beside the slots");
static_assert(sizeof(ChainLds) <= 156 * 1024, "one workgroup's LDS");
static_assert(kChainMaxN / 2 < 0x1fff && kChainMaxNnz <= 1 << 18 && kChainMaxRow + 3 <= kChainTile, "slot keys");
constexpr uint32_t kChainDrop = 0x1fffu << 19;  // keys from here on: inside the aggregate, or a row's padding

// a thread's walk over entries [a, b): `many` loads in flight, in order
template <int U, class F>
__device__ __forceinline__ void chain_walk(const int32_t* col, const double* w, int a, int b, F f) {
    for (int e = a; e < b; e += U) {
        int c[U];
        double x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int t = min(e + q, b - 1);
            c[q] = gld(col, t);
            x[q] = gld(w, t);
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (e + q < b) f(c[q], x[q]);
    }
}

__global__ void __launch_bounds__(kChainThreads) k_coarsen_chain(ChainJob J) {
    extern __shared__ __align__(16) double lds_raw[];
    ChainLds& S = *(ChainLds*)lds_raw;
    auto& M = S.u.a.t.m;
    auto& R = S.u.a.t.tile;
    __shared__ int sh[17];
    __shared__ double sm[4 * 16];
    __shared__ int runs[kChainRuns];
    __shared__ int s_bad;
    __shared__ int s_iso;
    const int tid = threadIdx.x, T = blockDim.x;
    if (tid == 0) s_iso = 0;
    __syncthreads();
    int n = J.n0;
    int64_t nnz = J.nnz0;
    const int32_t* rp = J.rp0;
    const int32_t* col = J.col0;
    const double* w = J.w0;
    int64_t i32_used = 0, cw_used = 0;
    int64_t cur_rp_off = -1, cur_cw_off = -1;
    int K = 0, collapsed = 0, stop_reason = 0;
    for (int k = 0;; ++k) {
        const int level = J.level0 + k;
        // ---- row pass: h, g = 2 max d, largest weight, FP32 rounding, longest row
        double m4[4] = {0.0, 0.0, 0.0, 0.0};
        for (int v = tid; v < n; v += T) {
            const int a = gld(rp, v), b = gld(rp, v + 1);
            m4[3] = fmax(m4[3], (double)(b - a));
            double bw = -1.0, d = 0.0;
            int bc = 0x7fffffff;
            chain_walk<4>(col, w, a, b, [&](int c, double x) {
                d += x;
                m4[2] = fmax(m4[2], fabs(x - (double)(float)x));
                if (x > bw || (x == bw && c < bc)) {
                    bw = x;
                    bc = c;
                }
            });
            // a vertex with no neighbour (a component that became one
            // aggregate) names itself and stops the chain below
            if (b == a) {
                bc = v;
                s_iso = 1;
            }
            M.v.h[v] = (uint16_t)bc;
            m4[0] = fmax(m4[0], 2.0 * d);
            m4[1] = fmax(m4[1], bw);
        }
        block_max4(m4, sm);
        ChainHdr hd{};
        hd.n = n;
        hd.nnz = nnz;
        hd.g = m4[0];
        hd.wmax = m4[1];
        hd.w32err = m4[2];
        hd.maxlen = m4[3];
        hd.rp_off = cur_rp_off;
        hd.cw_off = cur_cw_off;
        hd.agg_off = -1;
        hd.rounds = 0;
        K = k + 1;
        if (n <= J.coarsest_n || k + 1 >= J.max_levels) {
            stop_reason = (n <= J.coarsest_n) ? 1 : 5;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        if (s_iso) {
            // HEC needs every vertex to have a neighbour (CMG_E_ISOLATED)
            stop_reason = 6;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        if (hd.maxlen > kChainLongRow) {
            // rows this long make coarse rows that outgrow the register
            // slots, and one thread per row then works in global scratch,
            // slower than the grid kernels' sort: leave the level to them
            stop_reason = 4;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        // ---- HEC: candidates, greedy rounds
        for (int v = tid; v < n; v += T) {
            S.p.pair[v] = (uint16_t)v;
            M.l.f.live[v] = (hec_key(J.seed, level, v) < hec_key(J.seed, level, M.v.h[v])) ? 1 : 0;
            M.l.f.state[v] = 0;
            S.u.slot[v] = kNoKeyC;
        }
        __syncthreads();
        int rounds = 0;
        while (true) {
            for (int v = tid; v < n; v += T) {
                if (!M.l.f.live[v]) continue;
                const unsigned long long kv = hec_key(J.seed, level, v);
                atomicMin(&S.u.slot[v], kv);
                atomicMin(&S.u.slot[M.v.h[v]], kv);
            }
            __syncthreads();
            for (int v = tid; v < n; v += T) {
                if (!M.l.f.live[v]) continue;
                const unsigned long long kv = hec_key(J.seed, level, v);
                const int m = M.v.h[v];
                if (S.u.slot[v] == kv && S.u.slot[m] == kv) {
                    M.l.f.state[v] = kSeedC;
                    M.l.f.state[m] = kPartnerC;
                    S.p.pair[v] = (uint16_t)v;
                    S.p.pair[m] = (uint16_t)v;
                    M.l.f.live[v] = 0;
                }
            }
            __syncthreads();
            int alive = 0;
            for (int v = tid; v < n; v += T) {
                if (!M.l.f.live[v]) continue;
                const int m = M.v.h[v];
                if (M.l.f.state[v] != 0 || M.l.f.state[m] != 0) {
                    M.l.f.live[v] = 0;
                } else {
                    S.u.slot[v] = kNoKeyC;
                    S.u.slot[m] = kNoKeyC;
                    alive = 1;
                }
            }
            ++rounds;
            if (!__syncthreads_or(alive)) break;
        }
        hd.rounds = rounds;
        // ---- attach: follow h to a matched vertex
        for (int v = tid; v < n; v += T) {
            int r = v;
            for (int guard = 0; guard < n && M.l.f.state[r] == 0; ++guard) r = M.v.h[r];
            S.r.root[v] = S.p.pair[r];
        }
        __syncthreads();
        // number the opening vertices (the slots are dead from here on)
        const int nc = chain_scan(
            n, sh, [&](int v) { return M.l.f.state[v] == kSeedC ? 1 : 0; },
            [&](int v, int q) { M.rank[v] = (uint16_t)q; });
        if (nc < 2) {
            collapsed = 1;
            stop_reason = 2;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        // room for agg[n], rp[nc+1] in the int arena and the coarse entries
        // (at most nnz: every coarse entry comes from a fine one; at most
        // nc (nc - 1): no diagonal)
        const int64_t nnz_bound = min(nnz, (int64_t)nc * (int64_t)(nc - 1));
        if (i32_used + n + nc + 1 > J.ai32_cap || cw_used + nnz_bound > J.acw_cap) {
            stop_reason = 3;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        int32_t* agg = J.ai32 + i32_used;
        hd.agg_off = i32_used;
        for (int a = tid; a < nc; a += T) {
            M.acnt[a] = 0;
            S.p.afill[a] = 0;
        }
        if (tid == 0) s_bad = 0;
        __syncthreads();
        // ---- members of each aggregate, in increasing vertex index
        for (int v = tid; v < n; v += T) {
            const int a = M.rank[S.r.root[v]];
            S.u.a.agg[v] = (uint16_t)a;
            gst(agg, v, (int32_t)a);
            atomicAdd(&M.acnt[a], 1);
        }
        __syncthreads();
        chain_scan(
            nc, sh, [&](int a) { return M.acnt[a]; }, [&](int a, int q) { M.astart[a] = q; });
        for (int v = tid; v < n; v += T) {
            const int a = S.u.a.agg[v];
            M.v.members[M.astart[a] + atomicAdd(&S.p.afill[a], 1)] = (uint16_t)v;
        }
        __syncthreads();
        for (int a = tid; a < nc; a += T) {
            uint16_t* ms = M.v.members + M.astart[a];
            const int cnt = M.acnt[a];
            for (int i = 1; i < cnt; ++i) {
                const uint16_t x = ms[i];
                int j = i - 1;
                while (j >= 0 && ms[j] > x) {
                    ms[j + 1] = ms[j];
                    --j;
                }
                ms[j + 1] = x;
            }
            int deg = 0;  // at most nnz <= kChainMaxNnz
            for (int i = 0; i < cnt; ++i) {
                const int m = ms[i];
                S.p.off[m] = (uint16_t)deg;
                deg += gld(rp, m + 1) - gld(rp, m);
            }
            if (deg > kChainMaxRow) s_bad = 1;
            M.l.rcount[a] = (deg + 3) & ~3;
        }
        __syncthreads();
        if (s_bad) {
            // a coarse row too long for one thread's accumulation: leave this
            // level to the grid kernels (its aggregates are discarded)
            stop_reason = 4;
            hd.agg_off = -1;
            if (tid == 0) J.hdr[k] = hd;
            break;
        }
        {
            const int all = chain_scan(
                nc, sh, [&](int a) { return M.l.rcount[a]; }, [&](int a, int q) { S.r.soff[a] = q; });
            if (tid == 0) S.r.soff[nc] = all;
        }
        int32_t* rpc = J.ai32 + i32_used + n;
        int32_t* colc = J.acol + cw_used;
        double* wc = J.aw + cw_used;
        // ---- Galerkin: every fine entry is a contribution to a coarse row,
        // in a slot of its row's (a multiple of four of them).  A slot's key
        // orders the row by coarse column, then fine CSR order (the members'
        // entries ascend with the members), so a slot's place is the number
        // of smaller keys in its row; the first slot of each column then adds
        // the column's contributions in that order.  A slot per thread, a
        // tile of rows at a time.  Bound by the LDS reads and compares of the
        // ranks (of one CU).  One thread per coarse row, matching each entry
        // against 12 register slots, left most lanes idle behind the longest
        // row: the levels from 992 vertices (3842 entries) on took 199 us in
        // all, from 6016 414 and from 7500 (75000) 700, now 91, 254 and 358.
        int nnzc = 0;
        __syncthreads();
        for (int a0 = 0; a0 < nc;) {
            const int s0 = S.r.soff[a0];
            int a1 = nc;
            if (S.r.soff[nc] - s0 > kChainTile) {
                int lo = a0 + 1;  // a row always fits
                while (a1 - lo > 1) {
                    const int mid = (lo + a1) >> 1;
                    if (S.r.soff[mid] - s0 <= kChainTile) lo = mid;
                    else a1 = mid;
                }
                a1 = lo;
            }
            const int cnt = S.r.soff[a1] - s0;
            for (int i = tid; i < cnt; i += T) R.key[i] = 0xffffffffu;
            __syncthreads();
            for (int v = tid; v < n; v += T) {
                const int a = S.u.a.agg[v];
                if (a < a0 || a >= a1) continue;
                const int base = S.r.soff[a] - s0 + S.p.off[v];
                const int e0 = gld(rp, v), e1 = gld(rp, v + 1);
                for (int e = e0; e < e1; e += 8) {
                    int c[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) c[q] = gld(col, min(e + q, e1 - 1));
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (e + q < e1) {
                            const uint32_t b = S.u.a.agg[c[q]];
                            R.key[base + (e - e0) + q] =
                                ((int)b == a ? kChainDrop : b << 19) | (uint32_t)(e + q);
                            R.row[base + (e - e0) + q] = (uint16_t)a;
                        }
                    }
                }
            }
            __syncthreads();
            uint32_t key[kChainTile / kChainThreads];
            int to[kChainTile / kChainThreads];
#pragma unroll
            for (int q = 0; q < kChainTile / kChainThreads; ++q) {
                const int i = tid + q * kChainThreads;
                to[q] = -1;
                if (i < cnt) {
                    key[q] = R.key[i];
                    if (key[q] != 0xffffffffu) {
                        const int a = R.row[i];
                        const int lo = S.r.soff[a] - s0, hi = S.r.soff[a + 1] - s0;
                        int less = 0;
#pragma unroll 2
                        for (int t = lo; t < hi; t += 4) {
                            const uint4 x = *(const uint4*)&R.key[t];
                            less += (x.x < key[q]) + (x.y < key[q]) + (x.z < key[q]) + (x.w < key[q]);
                        }
                        to[q] = lo + less;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kChainTile / kChainThreads; ++q)
                if (to[q] >= 0) R.key[to[q]] = key[q];
            __syncthreads();
            // the slots that open a coarse entry, numbered in slot order:
            // 64 slots of a wavefront by their ballot, the wavefronts' runs
            // by a scan of their counts
            uint32_t opens = 0, starts = 0;  // this thread's slots: a coarse entry, a row
#pragma unroll
            for (int q = 0; q < kChainTile / kChainThreads; ++q) {
                if (q * kChainThreads >= cnt) break;
                const int i = tid + q * kChainThreads;
                const int t = min(i, cnt - 1), t1 = max(t - 1, 0);
                const uint32_t x = R.key[t], x1 = R.key[t1];
                const int a = R.row[t], a_1 = R.row[t1];
                const bool real = i < cnt && x != 0xffffffffu;
                const bool open = real && x < kChainDrop && (i == 0 || (x >> 19) != (x1 >> 19) || a != a_1);
                starts |= real && t == S.r.soff[real ? a : a0] - s0 ? 1u << q : 0u;
                opens |= open ? 1u << q : 0u;
                const int c = __popcll(__ballot(open));
                if ((tid & 63) == 0) runs[q * (kChainThreads / 64) + (tid >> 6)] = c;
            }
            __syncthreads();
            const int nruns = (cnt + kChainThreads - 1) / kChainThreads * (kChainThreads / 64);
            const int heads = chain_scan(
                nruns, sh, [&](int i) { return runs[i]; }, [&](int i, int q) { runs[i] = q; });
#pragma unroll
            for (int q = 0; q < kChainTile / kChainThreads; ++q) {
                if (q * kChainThreads >= cnt) break;
                const int i = tid + q * kChainThreads;
                const bool open = (opens >> q) & 1;
                const int at = runs[q * (kChainThreads / 64) + (tid >> 6)] +
                               __popcll(__ballot(open) & ((1ull << (tid & 63)) - 1));
                if ((starts >> q) & 1) gst(rpc, (int)R.row[i], (int32_t)(nnzc + at));
                if (open) R.head[at] = (uint16_t)i;
            }
            __syncthreads();
            for (int q = tid; q < heads; q += T) {
                const int i = R.head[q];
                const uint32_t x = R.key[i];
                const int a = R.row[i];
                auto mine = [&](int t) { return t < cnt && (R.key[t] >> 19) == (x >> 19) && R.row[t] == a; };
                // most columns have at most four contributions: in flight together
                int m = 1;
                double y[4];
                y[0] = gld(w, (int)(x & 0x7ffffu));
#pragma unroll
                for (int t = 1; t < 4; ++t) {
                    if (m == t && mine(i + t)) m = t + 1;
                    y[t] = gld(w, (int)(R.key[i + (t < m ? t : 0)] & 0x7ffffu));
                }
                double sum = y[0];
#pragma unroll
                for (int t = 1; t < 4; ++t) sum = t < m ? sum + y[t] : sum;
                if (m == 4)
                    for (int t = i + 4; mine(t); ++t) sum += gld(w, (int)(R.key[t] & 0x7ffffu));
                gst(colc, nnzc + q, (int32_t)(x >> 19));
                gst(wc, nnzc + q, sum);
            }
            nnzc += heads;
            a0 = a1;
            __syncthreads();
        }
        if (tid == 0) rpc[nc] = nnzc;
        if (tid == 0) J.hdr[k] = hd;
        cur_rp_off = i32_used + n;
        cur_cw_off = cw_used;
        i32_used += n + nc + 1;
        cw_used += nnzc;
        __syncthreads();
        n = nc;
        nnz = nnzc;
        rp = rpc;
        col = colc;
        w = wc;
    }
    if (tid == 0) {
        J.out[0] = K;
        J.out[1] = collapsed;
        J.out[2] = stop_reason;
    }
}

}  // namespace

hipError_t launch_coarsen_chain(const ChainJob& job, hipStream_t s) {
    if (job.n0 > kChainMaxN) return hipErrorInvalidValue;
    // more than 64 KiB of LDS for one workgroup has to be asked for
    static const hipError_t asked = hipFuncSetAttribute(
        (const void*)k_coarsen_chain, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(ChainLds));
    if (asked != hipSuccess) return asked;
    hipLaunchKernelGGL(k_coarsen_chain, dim3(1), dim3(kChainThreads), sizeof(ChainLds), s, job);
    return hipGetLastError();
}

}  // namespace cmg
