// Setup of the small levels in one workgroup: for a chain of levels of at
// most kChainMaxN vertices, the row pass (Gershgorin shift, heaviest
// neighbours), HEC (Algorithm 2, in the round-synchronous form of the grid
// kernels in setup.hip) and the Galerkin coarse graph (Section 2, the
// Proposition on restriction) run level after level inside one launch,
// separated only by workgroup barriers.  The grid kernels need about 40
// launches and 7 host synchronisations per level; on small levels those
// gaps, not the work, set the setup time.
//
// The Galerkin product is formed per coarse row: the members of aggregate
// a are visited in increasing index and their entries in CSR order, so the
// contributions to each coarse entry (a, b) are added in fine CSR order,
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

// Columns a thread keeps in registers while it forms a coarse row.
constexpr int kChainSlots = 12;
// Longest fine row of a level this kernel coarsens (measured on MI355X:
// 3D-grid levels with 27-47 entries per row took 0.27-1.9 ms here against
// a few hundred microseconds on the grid kernels).
constexpr int kChainLongRow = 24;

// Everything per vertex or aggregate lives in LDS (16-bit ids, as a level
// has at most kChainMaxN = 8192 vertices); only the CSR arrays, the arenas
// of the levels produced and the rows that outgrow the register slots are
// in memory.  A phase is a handful of dependent accesses per thread, so its
// time is their latency: one workgroup on arrays in memory took 177 us for
// the four levels below 992 vertices and 459 us for the five below 6016.
// The 8-byte slots of the greedy rounds are dead once the matching stands,
// and their space then holds the arrays of the aggregates.
struct ChainLds {
    union {
        unsigned long long slot[kChainMaxN];
        struct {
            uint16_t rank[kChainMaxN];          // aggregate opened by a vertex
            uint16_t agg[kChainMaxN];
            int32_t astart[kChainMaxN / 2 + 1];  // first member of each aggregate
            int32_t acnt[kChainMaxN / 2];
        } a;
    } u;
    union {
        uint16_t h[kChainMaxN];
        uint16_t members[kChainMaxN];
    } v;
    union {
        uint16_t pair[kChainMaxN];
        int32_t afill[kChainMaxN / 2];
    } p;
    union {
        uint16_t root[kChainMaxN];
        int32_t soff[kChainMaxN / 2];  // scratch offset of a coarse row
    } r;
    union {
        struct {
            uint8_t live[kChainMaxN], state[kChainMaxN];
        } f;
        int32_t rcount[kChainMaxN / 2];
    } l;
};
static_assert(sizeof(ChainLds) <= 140 * 1024, "one workgroup's LDS");

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
    extern __shared__ double lds_raw[];
    ChainLds& S = *(ChainLds*)lds_raw;
    __shared__ int sh[17];
    __shared__ double sm[4 * 16];
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
            S.v.h[v] = (uint16_t)bc;
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
            S.l.f.live[v] = (hec_key(J.seed, level, v) < hec_key(J.seed, level, S.v.h[v])) ? 1 : 0;
            S.l.f.state[v] = 0;
            S.u.slot[v] = kNoKeyC;
        }
        __syncthreads();
        int rounds = 0;
        while (true) {
            for (int v = tid; v < n; v += T) {
                if (!S.l.f.live[v]) continue;
                const unsigned long long kv = hec_key(J.seed, level, v);
                atomicMin(&S.u.slot[v], kv);
                atomicMin(&S.u.slot[S.v.h[v]], kv);
            }
            __syncthreads();
            for (int v = tid; v < n; v += T) {
                if (!S.l.f.live[v]) continue;
                const unsigned long long kv = hec_key(J.seed, level, v);
                const int m = S.v.h[v];
                if (S.u.slot[v] == kv && S.u.slot[m] == kv) {
                    S.l.f.state[v] = kSeedC;
                    S.l.f.state[m] = kPartnerC;
                    S.p.pair[v] = (uint16_t)v;
                    S.p.pair[m] = (uint16_t)v;
                    S.l.f.live[v] = 0;
                }
            }
            __syncthreads();
            int alive = 0;
            for (int v = tid; v < n; v += T) {
                if (!S.l.f.live[v]) continue;
                const int m = S.v.h[v];
                if (S.l.f.state[v] != 0 || S.l.f.state[m] != 0) {
                    S.l.f.live[v] = 0;
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
            for (int guard = 0; guard < n && S.l.f.state[r] == 0; ++guard) r = S.v.h[r];
            S.r.root[v] = S.p.pair[r];
        }
        __syncthreads();
        // number the opening vertices (the slots are dead from here on)
        const int nc = chain_scan(
            n, sh, [&](int v) { return S.l.f.state[v] == kSeedC ? 1 : 0; },
            [&](int v, int q) { S.u.a.rank[v] = (uint16_t)q; });
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
            S.u.a.acnt[a] = 0;
            S.p.afill[a] = 0;
        }
        if (tid == 0) s_bad = 0;
        __syncthreads();
        // ---- members of each aggregate, in increasing vertex index
        for (int v = tid; v < n; v += T) {
            const int a = S.u.a.rank[S.r.root[v]];
            S.u.a.agg[v] = (uint16_t)a;
            gst(agg, v, (int32_t)a);
            atomicAdd(&S.u.a.acnt[a], 1);
        }
        __syncthreads();
        chain_scan(
            nc, sh, [&](int a) { return S.u.a.acnt[a]; }, [&](int a, int q) { S.u.a.astart[a] = q; });
        for (int v = tid; v < n; v += T) {
            const int a = S.u.a.agg[v];
            S.v.members[S.u.a.astart[a] + atomicAdd(&S.p.afill[a], 1)] = (uint16_t)v;
        }
        __syncthreads();
        for (int a = tid; a < nc; a += T) {
            uint16_t* ms = S.v.members + S.u.a.astart[a];
            const int cnt = S.u.a.acnt[a];
            for (int i = 1; i < cnt; ++i) {
                const uint16_t x = ms[i];
                int j = i - 1;
                while (j >= 0 && ms[j] > x) {
                    ms[j + 1] = ms[j];
                    --j;
                }
                ms[j + 1] = x;
            }
            int64_t deg = 0;
            for (int i = 0; i < cnt; ++i) deg += gld(rp, (int)ms[i] + 1) - gld(rp, (int)ms[i]);
            if (deg > kChainMaxRow) s_bad = 1;
            S.l.rcount[a] = (int32_t)deg;
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
        chain_scan(
            nc, sh, [&](int a) { return S.l.rcount[a]; }, [&](int a, int q) { S.r.soff[a] = q; });
        int32_t* rpc = J.ai32 + i32_used + n;
        int32_t* colc = J.acol + cw_used;
        double* wc = J.aw + cw_used;
        // ---- Galerkin: one thread per coarse row, contributions added in
        // fine CSR order, row sorted by coarse column.  The row is formed in
        // the thread's register slots; a row with more distinct columns
        // moves to its global scratch and goes on there.  Where every row
        // has a thread of its own it stays in the registers until the
        // row lengths are scanned; else it waits in the scratch.
        const bool once = nc <= T;
        int rb[kChainSlots];
        double rw[kChainSlots];
        int len = 0;
        bool in_regs = true;
        for (int a = tid; a < nc; a += T) {
            const uint16_t* ms = S.v.members + S.u.a.astart[a];
            const int cnt = S.u.a.acnt[a];
            int32_t* mb = J.mb + S.r.soff[a];
            double* mw = J.mw + S.r.soff[a];
            // the row in registers: columns rb[0..len) (unused: INT_MAX) and
            // their sums; every slot operation is unrolled and branch-free
#pragma unroll
            for (int q = 0; q < kChainSlots; ++q) {
                rb[q] = 0x7fffffff;
                rw[q] = 0.0;
            }
            len = 0;
            in_regs = true;
            for (int i = 0; i < cnt; ++i) {
                const int m = ms[i];
                chain_walk<4>(col, w, gld(rp, m), gld(rp, m + 1), [&](int c, double x) {
                    const int b = S.u.a.agg[c];
                    bool found = b == a;  // inside the aggregate: dropped
#pragma unroll
                    for (int q = 0; q < kChainSlots; ++q) {
                        const bool here = rb[q] == b;
                        rw[q] = here ? rw[q] + x : rw[q];
                        found = found || here;
                    }
#pragma unroll
                    for (int q = 0; q < kChainSlots; ++q) {
                        const bool here = !found && q == len;
                        rb[q] = here ? b : rb[q];
                        rw[q] = here ? x : rw[q];
                    }
                    len += found ? 0 : 1;
                });
            }
            if (len <= kChainSlots) {
                // odd-even transposition sort by column (unused slots last)
#pragma unroll
                for (int pass = 0; pass < kChainSlots; ++pass) {
#pragma unroll
                    for (int q = pass & 1; q + 1 < kChainSlots; q += 2) {
                        const bool swap = rb[q] > rb[q + 1];
                        const int tb = rb[q];
                        const double tw = rw[q];
                        rb[q] = swap ? rb[q + 1] : tb;
                        rb[q + 1] = swap ? tb : rb[q + 1];
                        rw[q] = swap ? rw[q + 1] : tw;
                        rw[q + 1] = swap ? tw : rw[q + 1];
                    }
                }
                if (!once) {
#pragma unroll
                    for (int q = 0; q < kChainSlots; ++q) {
                        if (q < len) {
                            gst(mb, q, (int32_t)rb[q]);
                            gst(mw, q, rw[q]);
                        }
                    }
                }
            } else {
                // more columns than slots: the row is formed again from its
                // first entry, in the scratch
                in_regs = false;
                len = 0;
                for (int i = 0; i < cnt; ++i) {
                    const int m = ms[i];
                    const int e1 = gld(rp, m + 1);
                    for (int e = gld(rp, m); e < e1; ++e) {
                        const int b = S.u.a.agg[gld(col, e)];
                        const double x = gld(w, e);
                        if (b == a) continue;
                        int q = 0;
                        while (q < len && mb[q] != b) ++q;
                        if (q == len) {
                            mb[len] = b;
                            mw[len] = x;
                            ++len;
                        } else {
                            mw[q] += x;
                        }
                    }
                }
                for (int i = 1; i < len; ++i) {
                    const int b = mb[i];
                    const double x = mw[i];
                    int j = i - 1;
                    while (j >= 0 && mb[j] > b) {
                        mb[j + 1] = mb[j];
                        mw[j + 1] = mw[j];
                        --j;
                    }
                    mb[j + 1] = b;
                    mw[j + 1] = x;
                }
            }
            S.l.rcount[a] = len;
        }
        __syncthreads();
        // row pointers, in memory and in place of the lengths' scratch use
        const int64_t nnzc = chain_scan(
            nc, sh, [&](int a) { return S.l.rcount[a]; },
            [&](int a, int q) {
                gst(rpc, a, (int32_t)q);
                S.p.afill[a] = q;
            });
        if (tid == 0) rpc[nc] = (int32_t)nnzc;
        for (int a = tid; a < nc; a += T) {
            const int base = S.p.afill[a];
            if (once && in_regs) {
#pragma unroll
                for (int q = 0; q < kChainSlots; ++q) {
                    if (q < len) {
                        gst(colc, base + q, (int32_t)rb[q]);
                        gst(wc, base + q, rw[q]);
                    }
                }
                continue;
            }
            const int32_t* mb = J.mb + S.r.soff[a];
            const double* mw = J.mw + S.r.soff[a];
            const int l = S.l.rcount[a];
            for (int q = 0; q < l; ++q) {
                gst(colc, base + q, gld(mb, q));
                gst(wc, base + q, gld(mw, q));
            }
        }
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
