// Coarse levels refined inside one workgroup (Algorithm 1, Step 3; power
// iteration, Algorithm 3): all steps of a level, and of several levels in a
// row, in one launch with the vectors in LDS, on rows held in registers or
// read from an LDS image of the level's CSR arrays.  The arithmetic of a
// step is that of refine.hip.
#include <algorithm>

#include "cmg_internal.h"
#include "jump.h"

namespace cmg {

namespace {

// ------------------------------------------------ single-workgroup levels

__device__ __forceinline__ size_t align8(size_t b) { return (b + 7) & ~(size_t)7; }

// a load or store through the LDS view (LDS) or the global view
template <bool LDS, typename T>
__device__ __forceinline__ T ldx(const T* p, int i) {
    if constexpr (LDS) return sld(p, i);
    else return gld(p, i);
}
template <bool LDS, typename T>
__device__ __forceinline__ void stx(T* p, int i, T v) {
    if constexpr (LDS) sst(p, i, v);
    else gst(p, i, v);
}

// Bytes of the LDS image of a level: two vectors, weights (FP32 when that
// is exact), row pointers, columns (uint16: an image that fits has fewer
// than 65536 rows).
__device__ __forceinline__ size_t staged_bytes(const LevelDev& L, int w32) {
    size_t b = align8(16 * (size_t)L.n);
    b += align8((size_t)L.nnz * (w32 ? 4 : 8));
    b += align8(4 * ((size_t)L.n + 1));
    b += align8((size_t)L.nnz * 2);
    return b;
}

// Levels up to this size run on one wavefront with no workgroup barrier.
constexpr int kWaveRows = 256;

// Sum of NV (<= 4) doubles over the active threads, identical in every
// thread.  Wave mode: wave sum.  Workgroup mode: waves post their sums
// (one barrier, alternating slots); each wave reads the posts with one LDS
// access per lane, adds them within rows of 16 lanes and reads row q.
template <int NV, bool WAVE>
__device__ __forceinline__ void small_sum(double (&v)[NV], double* red, int& parity) {
    const int lane = threadIdx.x & 63;
    if constexpr (WAVE) {
        // LDS writes of this step become visible to the other lanes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = group_sum_t<64>(v[q]);
    } else {
        const int wv = threadIdx.x >> 6;
        const int nw = blockDim.x >> 6;
        double* slot = red + parity * 64;
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = group_sum_t<64>(v[q]);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < NV; ++q) slot[q * 16 + wv] = v[q];
        }
        __syncthreads();
        double t = (lane < NV * 16 && (lane & 15) < nw) ? slot[lane] : 0.0;
        t = group_sum_t<16>(t);
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = read_lane(t, q * 16);
        parity ^= 1;
    }
}

// The four sums of a PI step over one wavefront, identical in every lane.
// Lanes trade halves of their partials so that each exchange adds one
// value per lane: after the two quad exchanges lane p of a quad holds the
// quad sum of value 2 (p & 1) + (p >> 1); rotations of each row by 4 and 8
// lanes, then the row and half swaps, complete the sums.
__device__ __forceinline__ void wave_sum4(double (&v)[4]) {
    const int lane = threadIdx.x & 63;
    const bool odd = (lane & 1) != 0;
    double k0 = odd ? v[2] : v[0];
    double k1 = odd ? v[3] : v[1];
    const double s0 = odd ? v[0] : v[2];
    const double s1 = odd ? v[1] : v[3];
    k0 += dpp_move<0xB1>(s0);
    k1 += dpp_move<0xB1>(s1);
    const bool hi = (lane & 2) != 0;
    double k = hi ? k1 : k0;
    k += dpp_move<0x4E>(hi ? k0 : k1);
    k += dpp_move<0x124>(k);
    k += dpp_move<0x128>(k);
    k = pair_sum_rows<16>(k);
    k = pair_sum_rows<32>(k);
    v[0] = read_lane(k, 0);
    v[2] = read_lane(k, 1);
    v[1] = read_lane(k, 2);
    v[3] = read_lane(k, 3);
}

// Sums of a PI step over the `nw` wavefronts that run the steps (the first
// nw of the workgroup), identical in each of their lanes.  nw == 1: no
// workgroup barrier.  Otherwise every such wave posts its four sums (one
// barrier, alternating slots) and adds the posts within rows of 16 lanes.
template <bool WAVE>
__device__ __forceinline__ void step_sum4(double (&v)[4], double* red, int& parity, int nw) {
    if constexpr (WAVE) {
        // LDS writes of this step become visible to the other lanes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        wave_sum4(v);
    } else {
        const int lane = threadIdx.x & 63;
        const int wv = threadIdx.x >> 6;
        double* slot = red + parity * 64;
        wave_sum4(v);
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) slot[q * 16 + wv] = v[q];
        }
        __syncthreads();
        double t = ((lane & 15) < nw) ? slot[lane] : 0.0;
        t = group_sum_t<16>(t);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = read_lane(t, q * 16);
        parity ^= 1;
    }
}

// A product of a jump on a single-workgroup level, as in JumpOp (the jump's
// sum is added up from the products' vectors by their own pass).
struct SmallJump {
    bool first;
    double be;
};

// One PI step (JUMP: one product of a jump) of a small level, rows shared by
// `nthr` threads in G-lane groups.  Pointers are either all LDS (staged
// modes) or all global.
template <int G, bool W32, bool LDS, bool JUMP>
__device__ __forceinline__ void pi_small(int n, int nthr, const int32_t* rp, const void* colp,
                                         const void* wp, double g, const double* win, double* wout,
                                         double mu, double s, const SmallJump& sj, double (&acc)[4]) {
    const int lane = threadIdx.x & (G - 1);
    const int ngroups = nthr / G;
    for (int i = (int)(threadIdx.x / G); i < n; i += ngroups) {
        const int a = ldx<LDS>(rp, i), b = ldx<LDS>(rp, i + 1);
        const double wi = ldx<LDS>(win, i);
        double z = 0.0;
        if constexpr (JUMP) {
            if (!sj.first) z = ldx<LDS>(wout, i);
        }
        double t = 0.0;
        int e = a + lane;
        // four entries per trip: their column and value loads, then their
        // gathers, are in flight together; the sum keeps the entry order
        for (; e + 3 * G < b; e += 4 * G) {
            int c[4];
            double wt[4], x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int f = e + q * G;
                if constexpr (LDS) c[q] = (int)ldx<LDS>((const uint16_t*)colp, f);
                else c[q] = ldx<LDS>((const int32_t*)colp, f);
                if constexpr (W32) wt[q] = (double)ldx<LDS>((const float*)wp, f);
                else wt[q] = ldx<LDS>((const double*)wp, f);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = ldx<LDS>(win, c[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) t += wt[q] * (x[q] - wi);
        }
        for (; e < b; e += G) {
            int c;
            double wt;
            if constexpr (LDS) c = (int)ldx<LDS>((const uint16_t*)colp, e);
            else c = ldx<LDS>((const int32_t*)colp, e);
            if constexpr (W32) wt = (double)ldx<LDS>((const float*)wp, e);
            else wt = ldx<LDS>((const double*)wp, e);
            t += wt * (ldx<LDS>(win, c) - wi);
        }
        t = group_sum_t<G>(t);
        if (lane == 0) {
            if constexpr (JUMP) {
                const double y = (sj.first ? wi : 2.0 * wi) + sj.be * t - z;
                stx<LDS>(wout, i, y);
                acc[0] += wi * y;
                acc[1] += y * y;
                acc[2] += wi * wi;
            } else {
                const double x = (wi - mu) * s;
                const double y = s * (g * (wi - mu) + t);
                stx<LDS>(wout, i, y);
                acc[0] += y;
                acc[1] += y * y;
                acc[2] += y * x;
                acc[3] += x;
            }
        }
    }
}

// the same for a run-time G
template <bool W32, bool LDS, bool JUMP>
__device__ __forceinline__ void pi_small_any(int G, int n, int nthr, const int32_t* rp, const void* colp,
                                             const void* wp, double g, const double* win, double* wout, double mu,
                                             double s, const SmallJump& sj, double (&acc)[4]) {
    switch (G) {
        case 1: pi_small<1, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        case 2: pi_small<2, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        case 4: pi_small<4, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        case 8: pi_small<8, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        case 16: pi_small<16, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        case 32: pi_small<32, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
        default: pi_small<64, W32, LDS, JUMP>(n, nthr, rp, colp, wp, g, win, wout, mu, s, sj, acc); break;
    }
}

constexpr int kJumpSums = 4;  // entries of a jump's sum that a thread keeps in registers

// Moments and samples of a jump, and its verdict.
struct JumpLds {
    double mom[kJumpMoments];
    double dl[kJumpSamples];
    int safe, next;
};

// After each barrier of the waves that run the steps: count it and tell the
// idle waves that more follow.
template <bool WAVE>
__device__ __forceinline__ void small_bar(int* stop_flag, int& bar) {
    ++bar;
    if (!WAVE && threadIdx.x == 0) stop_flag[bar & 1] = 0;
}

template <bool WAVE>
__device__ __forceinline__ void small_sync(double* red, int& parity, int* stop_flag, int& bar, int nw) {
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    step_sum4<WAVE>(z, red, parity, nw);
    small_bar<WAVE>(stop_flag, bar);
}

// Mean and norm of b0, each entry written by the thread that reads it here.
template <bool WAVE, bool LDS>
__device__ __forceinline__ void small_normalise(int n, int nact, const double* b0, double* red, int& parity,
                                                int* stop_flag, int& bar, int nw, double& mu, double& s) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < n; i += nact) v[0] += ldx<LDS>(b0, i);
    step_sum4<WAVE>(v, red, parity, nw);
    small_bar<WAVE>(stop_flag, bar);
    mu = v[0] / (double)n;
    v[0] = v[1] = v[2] = v[3] = 0.0;
    for (int i = threadIdx.x; i < n; i += nact) {
        const double d = ldx<LDS>(b0, i) - mu;
        v[0] += d * d;
    }
    step_sum4<WAVE>(v, red, parity, nw);
    small_bar<WAVE>(stop_flag, bar);
    s = 1.0 / sqrt(v[0]);
}

// Verdict on a jump whose products are done, the same in every running
// thread; the moments are in js.
template <bool WAVE>
__device__ __forceinline__ bool small_jump_end(int K, int d, double tol, JumpLds* js, double* red, int& parity,
                                               int* stop_flag, int& bar, int nw, int* more, int* hold) {
    if (tol < 0.0) {
        small_sync<WAVE>(red, parity, stop_flag, bar, nw);
        return jump_verdict(K, 0, 0, true, more, hold);
    }
    small_sync<WAVE>(red, parity, stop_flag, bar, nw);
    // a sample per running thread (at least 128, at most kJumpSamples)
    const int ns = min(kJumpSamples, max(64 * nw, 128));
    for (int q = threadIdx.x; q < ns; q += 64 * nw)
        js->dl[q] = jump_delta(js->mom, 2 * d + 1, jump_sample(q, ns, K));
    small_sync<WAVE>(red, parity, stop_flag, bar, nw);
    if (threadIdx.x < 64) {
        int safe, next;
        jump_judge(js->dl, ns, K, tol, &safe, &next);
        if (threadIdx.x == 0) {
            js->safe = safe;
            js->next = next;
        }
    }
    small_sync<WAVE>(red, parity, stop_flag, bar, nw);
    return jump_verdict(K, js->safe, js->next, false, more, hold);
}

struct SmallIn {
    const void* cbuf;  // final vector of the coarser level
    int cfp32;
    int uniform;
    double cm, cs;     // its transform (v - cm) * cs
    uint64_t seed;
    double tol;
    int maxit;
};

// Rows of a small level read from its CSR arrays every step (an LDS image
// or global memory), in G-lane groups with G = L.lanes.
// Rows of a small level held in registers for all its steps: each G-lane
// group owns R rows and each lane E entries of every such row (entry
// a + lane + m G in slot m; columns as uint16 pairs, weights as FP32 where
// the level's weights equal that exactly, else FP64), so a step is one
// round of independent gathers from the LDS vector.  Unused slots point at
// the row's own vertex with weight 0 and add an exact zero, which keeps the
// sum of a row bit for bit that of the CSR traversal with the same G.
// A row longer than G E keeps its further entries in an LDS list; the
// lanes take them as slots E, E + 1, ... of the same stride, so each lane
// still sums its entries in CSR order.
//
// A step is bound by the LDS gathers and the adds of all E slots, of which
// most are unused (rows of 5 to 15 entries beside one of 30), so the rows
// are dealt out by length, longest first, and a wavefront does only the
// slots (in fours) that its longest row of the round has.
template <int G, int R, int E, typename W>
struct RegRows {
    uint32_t c2[R][E / 2];
    W w[R][E];
    int row[R];
    int em[R];             // fours of slots of the wavefront's longest row (wave-uniform)
    int ooff[R], ocnt[R];  // the row's entries beyond G E: LDS list offset and count
    const uint64_t* ovl;
    int n;
    double g;

    // list words per entry: column and FP32 weight in one, or column and
    // FP64 weight in two
    static constexpr int kListWords = sizeof(W) == 4 ? 1 : 2;

    // order: the rows, longest first (LDS, uint16); ov: LDS list of ovcap
    // words, filled from *ofill (zero before the first call of the level);
    // a list that would overflow sets *bad
    __device__ __forceinline__ void load(const LevelDev& L, int nact, const uint16_t* order, int* bad, uint64_t* ov,
                                         int ovcap, int* ofill) {
        n = L.n;
        g = L.g;
        ovl = ov;
        const int lane = (int)threadIdx.x & (G - 1);
        const int lead = ((int)threadIdx.x & (kWave - 1)) & ~(G - 1);
        const int ngroups = nact / G;
        const int grp = (int)threadIdx.x / G;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int p = grp + r * ngroups;
            const int i = p < n ? (int)sld(order, p) : n;
            row[r] = i < n ? i : -1;
            int a = 0, b = 0;
            if (i < n) {
                a = gld(L.rp, i);
                b = gld(L.rp, i + 1);
            }
            int most = (min(b - a, G * E) + 4 * G - 1) / (4 * G);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, kWave));
            em[r] = __builtin_amdgcn_readfirstlane(most);
            // the same count in every lane of the group; its first lane
            // takes the list space for all of them
            int extra = max(b - a - G * E, 0);
            int off = 0;
            if (extra > 0 && lane == 0) off = atomicAdd(ofill, kListWords * extra);
            off = __shfl(off, lead, kWave);
            if (extra > 0 && (off < 0 || off > ovcap - kListWords * extra)) {
                if (lane == 0) *bad = 1;
                extra = 0;
            }
            ooff[r] = off;
            ocnt[r] = extra;
            for (int q = lane; q < extra; q += G) {
                const int e = a + G * E + q;
                if constexpr (sizeof(W) == 4) {
                    const uint64_t wb = __float_as_uint((float)gld(L.w64, e));
                    sst(ov, off + q, (uint64_t)(uint32_t)gld(L.col, e) | (wb << 32));
                } else {
                    sst(ov, off + 2 * q, (uint64_t)(uint32_t)gld(L.col, e));
                    sst(ov, off + 2 * q + 1, (uint64_t)__double_as_longlong(gld(L.w64, e)));
                }
            }
            const uint32_t self = i < n ? (uint32_t)i : 0u;
#pragma unroll
            for (int m = 0; m < E; ++m) {
                const int e = a + lane + m * G;
                uint32_t cv = self;
                W wv = (W)0;
                if (e < b) {
                    cv = (uint32_t)gld(L.col, e);
                    wv = (W)gld(L.w64, e);
                }
                if (m & 1) c2[r][m >> 1] |= cv << 16;
                else c2[r][m >> 1] = cv;
                w[r][m] = wv;
            }
        }
        // the list entries are read back by the lanes of the group that
        // wrote them, in the same wavefront
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // sum over the first M slots of row r
    template <int M>
    __device__ __forceinline__ double slot_sum(int r, const double* win, double wi) {
        double x[M];
#pragma unroll
        for (int m = 0; m < M; ++m) x[m] = sld(win, (int)((m & 1) ? (c2[r][m >> 1] >> 16) : (c2[r][m >> 1] & 0xffffu)));
        double t = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m) t += (double)w[r][m] * (x[m] - wi);
        return t;
    }

    // sum over row r's entries a (w_k - w_i), in every lane of the group
    __device__ __forceinline__ double row_sum(int r, const double* win, double wi) {
        const int lane = (int)threadIdx.x & (G - 1);
        const int i = row[r];
        if constexpr (R * E > 32) {
            // decode the columns and widen the weights every step:
            // hoisted out of the step loop they would not fit
#pragma unroll
            for (int q = 0; q < E / 2; ++q) asm volatile("" : "+v"(c2[r][q]));
            if constexpr (sizeof(W) == 4) {
#pragma unroll
                for (int q = 0; q < E; ++q) asm volatile("" : "+v"(w[r][q]));
            }
        }
        double t;
        if constexpr (E == 8) {
            t = em[r] <= 1 ? slot_sum<4>(r, win, wi) : slot_sum<8>(r, win, wi);
        } else {
            if (em[r] <= 2) t = em[r] <= 1 ? slot_sum<4>(r, win, wi) : slot_sum<8>(r, win, wi);
            else t = em[r] <= 3 ? slot_sum<12>(r, win, wi) : slot_sum<16>(r, win, wi);
        }
        // entries beyond G E, two per trip; the second of a trip past
        // the row's end is its own vertex with weight 0 (an exact zero)
        for (int q = lane; q < ocnt[r]; q += 2 * G) {
            const bool two = q + G < ocnt[r];
            int k0, k1 = i;
            double a0, a1 = 0.0;
            if constexpr (sizeof(W) == 4) {
                const uint64_t p0 = sld(ovl, ooff[r] + q);
                const uint64_t p1 = two ? sld(ovl, ooff[r] + q + G) : (uint64_t)(uint32_t)i;
                k0 = (int)(uint32_t)p0;
                k1 = (int)(uint32_t)p1;
                a0 = (double)__uint_as_float((uint32_t)(p0 >> 32));
                a1 = (double)__uint_as_float((uint32_t)(p1 >> 32));
            } else {
                k0 = (int)sld(ovl, ooff[r] + 2 * q);
                a0 = __longlong_as_double((long long)sld(ovl, ooff[r] + 2 * q + 1));
                if (two) {
                    k1 = (int)sld(ovl, ooff[r] + 2 * (q + G));
                    a1 = __longlong_as_double((long long)sld(ovl, ooff[r] + 2 * (q + G) + 1));
                }
            }
            const double x0 = sld(win, k0), x1 = sld(win, k1);
            t += a0 * (x0 - wi);
            t += a1 * (x1 - wi);
        }
        return group_sum_t<G>(t);
    }

    __device__ __forceinline__ void step(const double* win, double* wout, double mu, double s, double (&acc)[4]) {
        const int lane = (int)threadIdx.x & (G - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = row[r];
            const double wi = sld(win, i < 0 ? 0 : i);
            const double t = row_sum(r, win, wi);
            if (lane == 0 && i >= 0) {
                const double xv = (wi - mu) * s;
                const double y = s * (g * (wi - mu) + t);
                sst(wout, i, y);
                acc[0] += y;
                acc[1] += y * y;
                acc[2] += y * xv;
                acc[3] += xv;
            }
        }
    }

    // one product of a jump, as in JumpOp, with the jump's sum in registers
    __device__ __forceinline__ void product(const double* win, double* wout, bool first, double be, double cj,
                                            double (&jsum)[R], double* jback, double (&acc)[4]) {
        const int lane = (int)threadIdx.x & (G - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = row[r];
            const double wi = sld(win, i < 0 ? 0 : i);
            const double z = sld(wout, i < 0 ? 0 : i);
            const double t = row_sum(r, win, wi);
            const double y = (first ? wi : 2.0 * wi - z) + be * t;
            jsum[r] = (first ? wi : jsum[r]) + cj * y;
            if (lane == 0 && i >= 0) {
                if (first) gst(jback, i, wi);
                sst(wout, i, y);
                acc[0] += wi * y;
                acc[1] += y * y;
                acc[2] += wi * wi;
            }
        }
    }
};

// Prolongation, deflation, normalisation and PI steps of one small level
// read from its CSR arrays.  MODE 0: LDS image, one wavefront; 1: LDS
// image, whole workgroup; 2: global memory, whole workgroup.
template <int MODE, bool W32>
__device__ void small_level(const LevelDev& L, const SmallIn& in, double* lds, double* red, int& parity,
                            int* stop_flag, JumpLds* js, int nw_run, LevelState& out) {
    constexpr bool WAVE = (MODE == 0);
    constexpr bool LDS = (MODE != 2);
    const int n = L.n;
    const int nthr = WAVE ? 64 : (int)blockDim.x;
    double* b0;
    double* b1;
    const int32_t* rp;
    const void* colp;
    const void* wp;
    if constexpr (MODE != 2) {
        char* p = (char*)lds;
        b0 = (double*)p;
        b1 = b0 + n;
        p += align8(16 * (size_t)n);
        wp = p;
        p += align8((size_t)L.nnz * (W32 ? 4 : 8));
        rp = (const int32_t*)p;
        p += align8(4 * ((size_t)n + 1));
        colp = p;
    } else {
        b0 = (double*)L.buf0;
        b1 = (double*)L.buf1;
        rp = L.rp;
        colp = L.col;
        wp = L.w64;
    }
    double sum[1] = {0.0};
    if (in.uniform) {
        for (int i = threadIdx.x; i < n; i += nthr) {
            const double v = hashed_uniform(in.seed, i) - 0.5;
            stx<LDS>(b0, i, v);
            sum[0] += v;
        }
    } else {
        for (int i = threadIdx.x; i < n; i += nthr) {
            const double v = (ld_any(in.cbuf, in.cfp32, gld(L.agg, i)) - in.cm) * in.cs;
            stx<LDS>(b0, i, v);
            sum[0] += v;
        }
    }
    small_sum<1, WAVE>(sum, red, parity);
    double mu = sum[0] / (double)n;
    double ss[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += nthr) {
        const double d = ldx<LDS>(b0, i) - mu;
        ss[0] += d * d;
    }
    small_sum<1, WAVE>(ss, red, parity);
    double s = 1.0 / sqrt(ss[0]);
    int cur = 0, k = 0, hit = 0;
    double utv = 0.0, pmu = mu, ps = s;
    // The PI steps run on the first `nw` wavefronts; the others only keep
    // the barrier count: after each barrier they read the flag left after
    // the one before it, and the running waves end with one more barrier.
    const int nw = WAVE ? 1 : nw_run;
    const int nact = 64 * nw;
    // wave-uniform test, taken as a scalar branch
    if (WAVE || __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) < nw) {
        const bool jumps = L.jmom != nullptr && (in.tol < 0.0 || in.tol >= kJumpTolMin);
        int bar = 0;              // barriers passed
        int since = 0, hold = 0;  // plain steps since the last jump, and to take before the next estimate
        while (true) {
            const double* win = cur ? b1 : b0;
            double* wout = cur ? b0 : b1;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            pi_small_any<W32, LDS, false>(L.lanes, n, nact, rp, colp, wp, L.g, win, wout, mu, s, SmallJump{}, acc);
            step_sum4<WAVE>(acc, red, parity, nw);
            ++bar;
            const double mu2 = acc[0] / (double)n;
            const double s2 = 1.0 / sqrt(acc[1] - acc[0] * mu2);
            const double utvp = utv;
            utv = s2 * (acc[2] - mu2 * acc[3]);
            ++k;
            cur ^= 1;
            pmu = mu;
            ps = s;
            mu = mu2;
            s = s2;
            bool stop = !(utv < 1.0 - in.tol);
            if (!stop && k >= in.maxit) {
                hit = 1;
                stop = true;
            }
            if (!WAVE && threadIdx.x == 0) stop_flag[bar & 1] = stop ? 1 : 0;
            if (stop) break;
            if (hold > 0) {
                --hold;
                continue;
            }
            if (!jumps || !jump_due(++since)) continue;
            const double r = 1.0 / (s * L.g);
            int K = jump_plan(utv, utvp, in.tol, r, in.maxit - k - 1);
            while (K > 0) {
                const int d = jump_products(K);
                SmallJump sj;
                double cj = 2.0 * (double)K / (double)(K + 1);
                // the jump's sum: up to kJumpSums entries per thread in
                // registers, else in memory
                const bool regs = n <= kJumpSums * nact;
                double sums[kJumpSums];
                const double* src = cur ? b1 : b0;
#pragma unroll
                for (int q = 0; q < kJumpSums; ++q) {
                    const int i = (int)threadIdx.x + q * nact;
                    sums[q] = regs && i < n ? ldx<LDS>(src, i) : 0.0;
                }
                for (int i = threadIdx.x; i < n; i += nact) {
                    const double x = ldx<LDS>(src, i);
                    gst(L.jback, i, x);
                    if (!regs) gst(L.jsum, i, x);
                }
                for (int j = 0; j < d; ++j) {
                    sj.first = j == 0;
                    sj.be = (j == 0 ? 2.0 : 4.0) / L.g;
                    double sum4[4] = {0.0, 0.0, 0.0, 0.0};
                    double* dst = cur ? b0 : b1;
                    pi_small_any<W32, LDS, true>(L.lanes, n, nact, rp, colp, wp, L.g, cur ? b1 : b0, dst, mu, s, sj,
                                                 sum4);
                    step_sum4<WAVE>(sum4, red, parity, nw);
                    small_bar<WAVE>(stop_flag, bar);
                    if (threadIdx.x == 0) jump_moments(js->mom, j, sum4[0], sum4[1], sum4[2]);
                    if (regs) {
#pragma unroll
                        for (int q = 0; q < kJumpSums; ++q) {
                            const int i = (int)threadIdx.x + q * nact;
                            if (i < n) sums[q] += cj * ldx<LDS>((const double*)dst, i);
                        }
                    } else {
                        for (int i = threadIdx.x; i < n; i += nact)
                            gst(L.jsum, i, gld(L.jsum, i) + cj * ldx<LDS>((const double*)dst, i));
                    }
                    cj = jump_coef(cj, K, j + 1);
                    cur ^= 1;
                }
                int more = 0;
                const bool keep = small_jump_end<WAVE>(K, d, in.tol, js, red, parity, stop_flag, bar, nw, &more, &hold);
                if (regs && keep) {
#pragma unroll
                    for (int q = 0; q < kJumpSums; ++q) {
                        const int i = (int)threadIdx.x + q * nact;
                        if (i < n) stx<LDS>(b0, i, sums[q]);
                    }
                } else {
                    const double* from = keep ? L.jsum : L.jback;
                    for (int i = threadIdx.x; i < n; i += nact) stx<LDS>(b0, i, gld(from, i));
                }
                if (keep) {
                    k += K;
                    small_normalise<WAVE, LDS>(n, nact, b0, red, parity, stop_flag, bar, nw, mu, s);
                } else {
                    small_sync<WAVE>(red, parity, stop_flag, bar, nw);
                }
                cur = 0;
                since = 0;
                K = more > 0 ? jump_steps((double)more, r, in.maxit - k - 1) : 0;
            }
        }
        if constexpr (!WAVE) __syncthreads();
    } else {
        // the flag left after barrier q - 1 tells whether barrier q is the
        // closing one; the slot parity follows the barriers, as in the
        // running waves
        for (int q = 1;; ++q) {
            __syncthreads();
            if (q > 1 && stop_flag[(q - 1) & 1]) break;
            parity ^= 1;
        }
        return;  // the state is kept by thread 0
    }
    int fin = cur;
    if constexpr (MODE != 2) {
        // the LDS vectors are discarded: final vector to buf0, previous to buf1
        const double* src = cur ? b1 : b0;
        const double* prv = cur ? b0 : b1;
        double* g0 = (double*)L.buf0;
        double* g1 = (double*)L.buf1;
        for (int i = threadIdx.x; i < n; i += nact) {
            gst(g0, i, sld(src, i));
            gst(g1, i, sld(prv, i));
        }
        fin = 0;
    }
    out.mu = mu;
    out.s = s;
    out.mu_prev = pmu;
    out.s_prev = ps;
    out.utv = utv;
    out.margin = utv - (1.0 - in.tol);
    out.fin = fin;
    out.k = k;
    out.maxit = hit;
    out.err = 0;
    out.ticks = 0;
}

// Levels jhi down to jlo (all FP64, small) refined inside one workgroup:
// prolongation, deflation, normalisation and every PI step separated only
// by workgroup (or wavefront) barriers, so thousands of steps cost no
// launches.  A level whose CSR and two vectors fit in `lds_budget` bytes
// is first copied to LDS (columns as uint16, weights as
// FP32 when that is exact) and its steps touch no global memory; levels of
// LevelDev::bwaves = 1 then run on a single wavefront, the others on that
// many (0: one up to kWaveRows vertices, else all).  Larger levels stream from global
// memory (L2).  The final vector of each level goes to buf0 (its
// predecessor to buf1).
__global__ void __launch_bounds__(kBlockKernelThreads)
    k_block_jobs(const BlockJob* __restrict__ jobs, int lds_budget) {
    extern __shared__ double lds[];
    __shared__ double red[2 * 64];
    __shared__ double s_cm, s_cs;
    __shared__ int s_cfin;
    __shared__ int s_stop[2];
    __shared__ JumpLds s_jump;
    const BlockJob Jb = jobs[blockIdx.x];
    const LevelDev* __restrict__ lv = Jb.lv;
    int parity = 0;
    if (threadIdx.x == 0 && !Jb.uniform) {
        LevelState c = Jb.st[Jb.jhi + 1];
        s_cm = c.mu;
        s_cs = c.s;
        s_cfin = c.fin;
    }
    __syncthreads();
    for (int j = Jb.jhi; j >= Jb.jlo; --j) {
        const long long t_start = wall_clock64();
        const LevelDev L = lv[j];
        const int n = L.n;
        const int nwmax = (int)(blockDim.x >> 6);
        const int nw = L.bwaves > 0 ? min(L.bwaves, nwmax) : (n <= kWaveRows ? 1 : nwmax);
        const int w32 = L.w32exact ? 1 : 0;
        const size_t need = staged_bytes(L, w32);
        const bool staged = need <= (size_t)lds_budget;
        const int mode = staged ? (nw == 1 ? 0 : 1) : 2;
        if (staged) {
            char* p = (char*)lds + align8(16 * (size_t)n);
            void* wdst = p;
            p += align8((size_t)L.nnz * (w32 ? 4 : 8));
            int32_t* rdst = (int32_t*)p;
            p += align8(4 * ((size_t)n + 1));
            void* cdst = p;
            for (int i = threadIdx.x; i <= n; i += blockDim.x) sst(rdst, i, gld(L.rp, i));
            for (int e = threadIdx.x; e < (int)L.nnz; e += blockDim.x) {
                const int cv = gld(L.col, e);
                const double wv = gld(L.w64, e);
                sst((uint16_t*)cdst, e, (uint16_t)cv);
                if (w32) sst((float*)wdst, e, (float)wv);
                else sst((double*)wdst, e, wv);
            }
            __syncthreads();
        }
        SmallIn in;
        in.uniform = (Jb.uniform && j == Jb.jhi) ? 1 : 0;
        if (!in.uniform) {
            const LevelDev C = lv[j + 1];
            in.cbuf = s_cfin ? C.buf1 : C.buf0;
            in.cfp32 = C.fp32;
        } else {
            in.cbuf = nullptr;
            in.cfp32 = 0;
        }
        in.cm = s_cm;
        in.cs = s_cs;
        in.seed = Jb.seed;
        in.tol = L.kfix > 0 ? -1.0 : Jb.tol;  // a fixed schedule never passes the test
        in.maxit = L.kfix > 0 ? L.kfix : Jb.maxit;
        LevelState o;
        if (mode == 0) {
            if (threadIdx.x < 64) {
                if (w32) small_level<0, true>(L, in, lds, red, parity, s_stop, &s_jump, 1, o);
                else small_level<0, false>(L, in, lds, red, parity, s_stop, &s_jump, 1, o);
            }
        } else if (mode == 1) {
            if (w32) small_level<1, true>(L, in, lds, red, parity, s_stop, &s_jump, nw, o);
            else small_level<1, false>(L, in, lds, red, parity, s_stop, &s_jump, nw, o);
        } else {
            small_level<2, false>(L, in, lds, red, parity, s_stop, &s_jump, nw, o);
        }
        if (threadIdx.x == 0) {
            o.ticks = wall_clock64() - t_start;
            Jb.st[j] = o;
            s_cm = o.mu;
            s_cs = o.s;
            s_cfin = o.fin;
        }
        __syncthreads();
    }
}

// The rows of a level by the number of slots (in fours) that a lane needs
// for them, longest first, in index order among equals: a counting sort
// over wavefront ballots, the same for every run.  chunks: an LDS word per
// class and 64 rows.
constexpr int kRowChunks = kBlockRegsThreads * 4 / 64;  // R <= 4 rows per thread
template <int G, int E>
__device__ __forceinline__ void rows_by_length(const LevelDev& L, int nact, uint16_t* order, int* chunks, double* red,
                                               int& parity, int* stop_flag, int& bar, int nw) {
    constexpr int C = E / 4;
    const int n = L.n;
    const int lane = (int)threadIdx.x & 63;
    const int nch = (n + 63) / 64;
    // class 0 holds the longest rows
    auto cls = [&](int i) {
        const int len = min(gld(L.rp, i + 1) - gld(L.rp, i), G * E);
        return C - max((len + 4 * G - 1) / (4 * G), 1);
    };
    for (int i = threadIdx.x; i < nch * 64; i += nact) {
        const int q = i < n ? cls(i) : -1;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int cnt = __popcll(__ballot(q == c));
            if (lane == 0) chunks[c * nch + (i >> 6)] = cnt;
        }
    }
    small_sync<false>(red, parity, stop_flag, bar, nw);
    for (int i = threadIdx.x; i < nch * 64; i += nact) {
        const int q = i < n ? cls(i) : -1;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const unsigned long long m = __ballot(q == c);
            if (m == 0ull) continue;
            // rows of longer classes, then of this class in earlier chunks
            int before = 0;
            const int upto = c * nch + (i >> 6);
            for (int k = lane; k < upto; k += 64) before += chunks[k];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
            if (q == c) sst(order, before + __popcll(m & ((1ull << lane) - 1ull)), (uint16_t)i);
        }
    }
    small_sync<false>(red, parity, stop_flag, bar, nw);
}

// One level on register rows with both vectors in LDS (and the entries of
// rows longer than the layout in the LDS list ov of ovcap entries, filled
// from *ofill).  nw == 1: on wavefront 0 alone with no workgroup barrier
// (the caller keeps the other waves out); else the first nw waves run the
// steps and the others keep the barrier count as in the CSR traversal.
template <int G, int R, int E, typename W>
__device__ void reg_level(const LevelDev& L, const SmallIn& in, double* b0, double* b1, uint64_t* ov, int ovcap,
                          int* ofill, int* chunks, double* red, int& parity, int* stop_flag, JumpLds* js, int* bad,
                          int nw, LevelState& out) {
    const bool wave = (nw == 1);
    const int n = L.n;
    const int nthr = wave ? 64 : (int)blockDim.x;
    double sum[1] = {0.0};
    if (in.uniform) {
        for (int i = threadIdx.x; i < n; i += nthr) {
            const double v = hashed_uniform(in.seed, i) - 0.5;
            sst(b0, i, v);
            sum[0] += v;
        }
    } else {
        for (int i = threadIdx.x; i < n; i += nthr) {
            const double v = (ld_any(in.cbuf, in.cfp32, gld(L.agg, i)) - in.cm) * in.cs;
            sst(b0, i, v);
            sum[0] += v;
        }
    }
    if (wave) small_sum<1, true>(sum, red, parity);
    else small_sum<1, false>(sum, red, parity);
    double mu = sum[0] / (double)n;
    double ss[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += nthr) {
        const double d = sld(b0, i) - mu;
        ss[0] += d * d;
    }
    if (wave) small_sum<1, true>(ss, red, parity);
    else small_sum<1, false>(ss, red, parity);
    double s = 1.0 / sqrt(ss[0]);
    int cur = 0, k = 0, hit = 0;
    double utv = 0.0, pmu = mu, ps = s;
    const int nact = 64 * nw;
    if (!(wave || __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) < nw)) {
        // counts the barriers along, as in the CSR traversal
        for (int q = 1;; ++q) {
            __syncthreads();
            if (q > 1 && stop_flag[(q - 1) & 1]) break;
            parity ^= 1;
        }
        return;  // the state is kept by thread 0
    }
    int bar = 0;  // barriers passed
    // the rows in the order they are dealt out, in b1 (not written before
    // the first step)
    uint16_t* order = (uint16_t*)b1;
    if (wave) {
        for (int i = threadIdx.x; i < n; i += 64) sst(order, i, (uint16_t)i);
        small_sync<true>(red, parity, stop_flag, bar, 1);
    } else {
        rows_by_length<G, E>(L, nact, order, chunks, red, parity, stop_flag, bar, nw);
    }
    RegRows<G, R, E, W> rows;
    rows.load(L, nact, order, bad, ov, ovcap, ofill);
    if (wave) small_sync<true>(red, parity, stop_flag, bar, 1);
    else small_sync<false>(red, parity, stop_flag, bar, nw);
    const bool jumps = L.jmom != nullptr && (in.tol < 0.0 || in.tol >= kJumpTolMin);
    const double inv_n = 1.0 / (double)n;
    int since = 0, hold = 0;  // plain steps since the last jump, and to take before the next estimate
    while (true) {
        const double* win = cur ? b1 : b0;
        double* wout = cur ? b0 : b1;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        rows.step(win, wout, mu, s, acc);
        if (wave) step_sum4<true>(acc, red, parity, 1);
        else step_sum4<false>(acc, red, parity, nw);
        ++bar;
        // (a division and a square root less: 0.1 us of a step)
        const double mu2 = acc[0] * inv_n;
        const double s2 = fast_rsq(acc[1] - acc[0] * mu2);
        const double utvp = utv;
        utv = s2 * (acc[2] - mu2 * acc[3]);
        ++k;
        cur ^= 1;
        pmu = mu;
        ps = s;
        mu = mu2;
        s = s2;
        bool stop = !(utv < 1.0 - in.tol);
        if (!stop && k >= in.maxit) {
            hit = 1;
            stop = true;
        }
        if (!wave && threadIdx.x == 0) stop_flag[bar & 1] = stop ? 1 : 0;
        if (stop) break;
        if (hold > 0) {
            --hold;
            continue;
        }
        if (!jumps || !jump_due(++since)) continue;
        const double r = 1.0 / (s * L.g);
        int K = jump_plan(utv, utvp, in.tol, r, in.maxit - k - 1);
        while (K > 0) {
            const int d = jump_products(K);
            double cj = 2.0 * (double)K / (double)(K + 1);
            double jsum[R];
#pragma unroll
            for (int q = 0; q < R; ++q) jsum[q] = 0.0;
            for (int j = 0; j < d; ++j) {
                double sum4[4] = {0.0, 0.0, 0.0, 0.0};
                rows.product(cur ? b1 : b0, cur ? b0 : b1, j == 0, (j == 0 ? 2.0 : 4.0) / L.g, cj, jsum, L.jback, sum4);
                if (wave) step_sum4<true>(sum4, red, parity, 1);
                else step_sum4<false>(sum4, red, parity, nw);
                if (wave) small_bar<true>(stop_flag, bar);
                else small_bar<false>(stop_flag, bar);
                if (threadIdx.x == 0) jump_moments(js->mom, j, sum4[0], sum4[1], sum4[2]);
                cj = jump_coef(cj, K, j + 1);
                cur ^= 1;
            }
            int more = 0;
            const bool keep =
                wave ? small_jump_end<true>(K, d, in.tol, js, red, parity, stop_flag, bar, 1, &more, &hold)
                     : small_jump_end<false>(K, d, in.tol, js, red, parity, stop_flag, bar, nw, &more, &hold);
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (((int)threadIdx.x & (G - 1)) == 0 && rows.row[q] >= 0)
                    sst(b0, rows.row[q], keep ? jsum[q] : gld(L.jback, rows.row[q]));
            if (wave) small_sync<true>(red, parity, stop_flag, bar, 1);
            else small_sync<false>(red, parity, stop_flag, bar, nw);
            if (keep) {
                k += K;
                if (wave) small_normalise<true, true>(n, 64, b0, red, parity, stop_flag, bar, 1, mu, s);
                else small_normalise<false, true>(n, nact, b0, red, parity, stop_flag, bar, nw, mu, s);
            }
            cur = 0;
            since = 0;
            K = more > 0 ? jump_steps((double)more, r, in.maxit - k - 1) : 0;
        }
    }
    if (!wave) __syncthreads();
    // the LDS vectors are discarded: final vector to buf0, previous to buf1
    const double* src = cur ? b1 : b0;
    const double* prv = cur ? b0 : b1;
    double* g0 = (double*)L.buf0;
    double* g1 = (double*)L.buf1;
    for (int i = threadIdx.x; i < n; i += nact) {
        gst(g0, i, sld(src, i));
        gst(g1, i, sld(prv, i));
    }
    if (wave) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    out.mu = mu;
    out.s = s;
    out.mu_prev = pmu;
    out.s_prev = ps;
    out.utv = utv;
    out.margin = utv - (1.0 - in.tol);
    out.fin = 0;
    out.k = k;
    out.maxit = hit;
    out.err = *bad;
    out.ticks = 0;
}

// Levels jhi down to jlo refined inside one workgroup on register rows of
// G lanes per row, R rows per lane group and E slots per lane and row
// (every level of the job has that layout and LevelDev::bwaves waves;
// weights exact in W; rows longer than G E keep the rest in the LDS left
// after the two vectors).  A level whose layout does not fit is skipped
// with err = 2 in its state; err = 1 if the entries beyond the layout do
// not fit the LDS left.
template <int G, int R, int E, typename W>
__global__ void __launch_bounds__(kBlockRegsThreads)
    k_block_regs(const BlockJob* __restrict__ jobs, int lds_budget) {
    extern __shared__ double lds[];
    __shared__ double red[2 * 64];
    __shared__ double s_cm, s_cs;
    __shared__ int s_cfin;
    __shared__ int s_stop[2];
    __shared__ JumpLds s_jump;
    __shared__ int s_chunks[(E / 4) * kRowChunks];
    __shared__ int s_bad;
    __shared__ int s_ofill;
    const BlockJob Jb = jobs[blockIdx.x];
    const LevelDev* __restrict__ lv = Jb.lv;
    int parity = 0;
    if (threadIdx.x == 0 && !Jb.uniform) {
        LevelState c = Jb.st[Jb.jhi + 1];
        s_cm = c.mu;
        s_cs = c.s;
        s_cfin = c.fin;
    }
    __syncthreads();
    for (int j = Jb.jhi; j >= Jb.jlo; --j) {
        const long long t_start = wall_clock64();
        const LevelDev L = lv[j];
        const int n = L.n;
        const int nw = max(1, min(L.bwaves, (int)(blockDim.x >> 6)));
        const bool fits = L.lanes == G && L.bregs == R && L.bslots == E && (sizeof(W) == 8 || L.w32exact) && n >= 1 && n <= 65536 &&
                          16 * (size_t)n <= (size_t)lds_budget && n <= R * (64 * nw / G) &&
                          (nw > 1 || (G == 1 && R == 1));
        if (threadIdx.x == 0) {
            s_bad = 0;
            s_ofill = 0;
        }
        // list of the entries beyond the layout: the LDS left after the vectors
        uint64_t* ov = (uint64_t*)(lds + 2 * (size_t)n);
        const int ovcap = fits ? (int)(((size_t)lds_budget - 16 * (size_t)n) / 8) : 0;
        SmallIn in;
        in.uniform = (Jb.uniform && j == Jb.jhi) ? 1 : 0;
        if (!in.uniform) {
            const LevelDev C = lv[j + 1];
            in.cbuf = s_cfin ? C.buf1 : C.buf0;
            in.cfp32 = C.fp32;
        } else {
            in.cbuf = nullptr;
            in.cfp32 = 0;
        }
        in.cm = s_cm;
        in.cs = s_cs;
        in.seed = Jb.seed;
        in.tol = L.kfix > 0 ? -1.0 : Jb.tol;  // a fixed schedule never passes the test
        in.maxit = L.kfix > 0 ? L.kfix : Jb.maxit;
        LevelState o{};
        if (!fits) {
            o.err = 2;
        } else if (nw == 1) {
            if (threadIdx.x < 64)
                reg_level<G, R, E, W>(L, in, lds, lds + n, ov, ovcap, &s_ofill, s_chunks, red, parity, s_stop, &s_jump, &s_bad, 1, o);
        } else {
            reg_level<G, R, E, W>(L, in, lds, lds + n, ov, ovcap, &s_ofill, s_chunks, red, parity, s_stop, &s_jump, &s_bad, nw, o);
        }
        if (threadIdx.x == 0) {
            o.ticks = wall_clock64() - t_start;
            Jb.st[j] = o;
            s_cm = o.mu;
            s_cs = o.s;
            s_cfin = o.fin;
        }
        __syncthreads();
    }
}

// -------------------------------------------------- dense small levels
//
// A level of at most kDenseBlockN vertices holds B' = (gI - L)/g - 1 1^T/n
// (the step with its deflation) as a dense matrix and works on sixteen
// iterates at once: X = [x, B'x, .., B'^15 x] becomes the next sixteen by
// one product with M = B'^16, formed by four squarings at the start (whose
// intermediate powers also give the first sixteen).  The products are
// matrix instructions (v_mfma_f64_16x16x4: a wave per 16 rows, its rows of M
// in registers, X in LDS); the stopping quantity of every one of the
// sixteen steps comes from the columns' norms and the products of
// neighbouring columns, so the level ends at the same step as step by step.
// Per step that is n/4 matrix-instruction latencies (64 cycles) and two
// barriers over 16, against a chain of gathers, sums over the workgroup and
// a square root: 0.35 to 0.8 us a step before.
//
// The powers are symmetric, so only the 16 x 16 tiles on and below the
// diagonal are kept and formed (half the products, and 11 tiles a side fit
// the LDS); the entries of a tile are swizzled so that its rows and its
// columns are both read without bank conflicts.
typedef double v4d __attribute__((ext_vector_type(4)));

template <int NT>
struct DenseTiles {
    double* p;
    // entry (r, c) of tile (i, j)
    __device__ __forceinline__ static int at(int i, int j, int r, int c) {
        return i >= j ? ((i * (i + 1)) / 2 + j) * 256 + r * 16 + (c ^ r) : ((j * (j + 1)) / 2 + i) * 256 + c * 16 + (r ^ c);
    }
    __device__ __forceinline__ double get(int i, int j, int r, int c) const { return sld(p, at(i, j, r, c)); }
    __device__ __forceinline__ void put(int i, int j, int r, int c, double v) { sst(p, at(i, j, r, c), v); }
};

template <int NT>
__device__ void dense_level(const LevelDev& L, const SmallIn& in, double* lds, double* red, double* part,
                            LevelState& out) {
    constexpr int N = 16 * NT;                    // rows, padded with zeros
    constexpr int NTILE = NT * (NT + 1) / 2;
    constexpr int RT = NT > 8 ? 2 : 1;            // row tiles of a wavefront
    constexpr int CW = NT <= 4 ? 4 : NT < 8 ? 2 : 8;  // wavefronts that check, with no tile of their own if NT < 8
    constexpr int C0 = NT < 8 ? 8 - CW : 0;       // the first of them
    constexpr int MAXT = (NTILE + 7) / 8;         // tiles of a wavefront in a squaring
    DenseTiles<NT> M{lds};
    double* X0 = lds + NTILE * 256;  // N x 16
    double* X1 = lds;                // N x 16, over the matrix once that is in registers
    const int n = L.n;
    const int tid = (int)threadIdx.x, T = (int)blockDim.x;
    const int lane = tid & 63, l16 = lane & 15, l4 = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // B' and the start vector
    const double inv_n = 1.0 / (double)n, inv_g = 1.0 / L.g;
    for (int t = tid; t < NTILE * 256; t += T) {
        int i = 0;
        while ((i + 1) * (i + 2) / 2 <= (t >> 8)) ++i;
        const int j = (t >> 8) - i * (i + 1) / 2, r = (t >> 4) & 15, c = (t & 15) ^ r;
        sst(lds, t, 16 * i + r < n && 16 * j + c < n ? -inv_n : 0.0);
    }
    for (int t = tid; t < N * 16; t += T) sst(X0, t, 0.0);
    double v = 0.0;
    if (tid < n) {
        if (in.uniform) v = hashed_uniform(in.seed, tid) - 0.5;
        else v = (ld_any(in.cbuf, in.cfp32, gld(L.agg, tid)) - in.cm) * in.cs;
    }
    double sum[1] = {v};
    block_sum<1>(sum, red);
    const double mu = sum[0] / (double)n;
    const double dv = tid < n ? v - mu : 0.0;
    double ss[1] = {dv * dv};
    block_sum<1>(ss, red);
    if (tid < n) {
        sst(X0, tid * 16, dv * (1.0 / sqrt(ss[0])));
        double d = 0.0;
        const int a = gld(L.rp, tid), b = gld(L.rp, tid + 1);
        for (int e = a; e < b; e += 4) {
            int c[4];
            double w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = gld(L.col, min(e + q, b - 1));
                w[q] = gld(L.w64, min(e + q, b - 1));
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (e + q >= b) continue;
                d += w[q];
                // columns below the diagonal fill the lower triangle (and
                // both halves of a diagonal tile)
                if ((c[q] >> 4) > (tid >> 4)) continue;
                const int t = M.at(tid >> 4, c[q] >> 4, tid & 15, c[q] & 15);
                sst(lds, t, w[q] * inv_g - inv_n);
            }
        }
        M.put(tid >> 4, tid >> 4, tid & 15, tid & 15, (L.g - d) * inv_g - inv_n);
    }
    __syncthreads();
    // the first sixteen iterates and M = B'^16
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        v4d y[RT];
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            const int i = wv + 8 * u;
            y[u] = v4d{0.0, 0.0, 0.0, 0.0};
            if (i >= NT) continue;
#pragma unroll 2
            for (int k = 0; k < NT; ++k) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    y[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                        M.get(i, k, l16, 4 * t + l4), sld(X0, (16 * k + 4 * t + l4) * 16 + l16), y[u], 0, 0, 0);
            }
        }
        // the square's tiles, dealt out over the wavefronts
        v4d c[MAXT];
#pragma unroll
        for (int q = 0; q < MAXT; ++q) {
            const int tile = wv + 8 * q;
            c[q] = v4d{0.0, 0.0, 0.0, 0.0};
            if (tile >= NTILE) continue;
            int i = 0;
            while ((i + 1) * (i + 2) / 2 <= tile) ++i;
            const int j = tile - i * (i + 1) / 2;
#pragma unroll 2
            for (int k = 0; k < NT; ++k) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    c[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(M.get(i, k, l16, 4 * t + l4),
                                                                M.get(k, j, 4 * t + l4, l16), c[q], 0, 0, 0);
            }
        }
        __syncthreads();
        const int done = 1 << p;  // columns there are
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            const int i = wv + 8 * u;
            if (i >= NT || l16 >= done) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) sst(X0, (16 * i + 4 * q + l4) * 16 + l16 + done, y[u][q]);
        }
#pragma unroll
        for (int q = 0; q < MAXT; ++q) {
            const int tile = wv + 8 * q;
            if (tile >= NTILE) continue;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int r = 4 * h + l4;
                sst(lds, tile * 256 + r * 16 + (l16 ^ r), c[q][h]);
            }
        }
        __syncthreads();
    }
    double af[RT][4 * NT];
#pragma unroll
    for (int u = 0; u < RT; ++u) {
        if (wv + 8 * u >= NT) continue;
#pragma unroll
        for (int t = 0; t < 4 * NT; ++t) af[u][t] = M.get(wv + 8 * u, t >> 2, l16, 4 * (t & 3) + l4);
    }
    __syncthreads();  // the matrix is read before the second block overwrites it
    // blocks of sixteen steps: step 16 b + c is column c of block b
    double* X = X0;
    double* Y = X1;
    int first = 1;       // first step of the block with a test
    int k0 = 0, k = 0;   // step of column 0; the step that ends the level
    int col = 0, hit = 0;
    double plast = 0.0;  // 1 / norm of the last column of the block before
    double utv = 0.0, sc = 1.0, sp = 1.0;
    while (true) {
        // norms of the columns and products with the one before
        if (wv >= C0) {
            double a0 = 0.0, a1 = 0.0;
#pragma unroll 4
            for (int r = 4 * (wv - C0) + l4; r < N; r += 4 * CW) {
                const double x = sld(X, r * 16 + l16);
                const double z = l16 > 0 ? sld(X, r * 16 + l16 - 1) : sld(Y, r * 16 + 15);
                a0 += x * x;
                a1 += x * z;
            }
            a0 = pair_sum_rows<32>(pair_sum_rows<16>(a0));
            a1 = pair_sum_rows<32>(pair_sum_rows<16>(a1));
            if (lane < 16) {
                sst(part, (wv - C0) * 32 + l16, a0);
                sst(part, (wv - C0) * 32 + 16 + l16, a1);
            }
        }
        // the next block meanwhile
        v4d y[RT];
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            y[u] = v4d{0.0, 0.0, 0.0, 0.0};
            if (wv + 8 * u >= NT) continue;
#pragma unroll
            for (int t = 0; t < 4 * NT; ++t)
                y[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[u][t], sld(X, (4 * t + l4) * 16 + l16), y[u], 0, 0, 0);
        }
        __syncthreads();
        double n2 = 0.0, dd = 0.0;
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            n2 += sld(part, q * 32 + l16);
            dd += sld(part, q * 32 + 16 + l16);
        }
        const double rn = fast_rsq(n2);
        const double rb = __shfl_up(rn, 1, 16);
        const double rp = l16 > 0 ? rb : plast;
        const double uv = dd * rn * rp;
        const bool end = l16 >= first && (!(uv < 1.0 - in.tol) || k0 + l16 >= in.maxit);
        const unsigned m = (unsigned)(__ballot(end) & 0xffffull);
        if (m != 0u) {
            col = __ffs(m) - 1;
            k = k0 + col;
            utv = read_lane(uv, col);
            sc = read_lane(rn, col);
            sp = col > 0 ? read_lane(rn, col - 1) : plast;
            hit = utv < 1.0 - in.tol ? 1 : 0;
            break;
        }
        // scaled by a power of two against underflow
        const double last = read_lane(n2, 15);
        plast = read_lane(rn, 15);
        const double scale = last < 0x1p-200 ? 0x1p+100 : 1.0;
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            if (wv + 8 * u >= NT) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) sst(Y, (16 * (wv + 8 * u) + 4 * q + l4) * 16 + l16, y[u][q] * scale);
        }
        __syncthreads();
        double* const t = X;
        X = Y;
        Y = t;
        k0 += 16;
        first = 0;
    }
    // final vector to buf0, the one before to buf1
    if (tid < n) {
        gst((double*)L.buf0, tid, sld(X, tid * 16 + col));
        gst((double*)L.buf1, tid, col > 0 ? sld(X, tid * 16 + col - 1) : sld(Y, tid * 16 + 15));
    }
    __syncthreads();
    out.mu = 0.0;
    out.s = sc;
    out.mu_prev = 0.0;
    out.s_prev = sp;
    out.utv = utv;
    out.margin = utv - (1.0 - in.tol);
    out.fin = 0;
    out.k = k;
    out.maxit = hit;
    out.err = 0;
    out.ticks = 0;
}

// tiles a side of the kernel that takes a level of nt
__host__ __device__ constexpr int dense_tiles(int nt) {
    return nt <= 2 ? 2 : nt <= 4 ? nt : nt <= 6 ? 6 : nt <= 8 ? 8 : nt <= 9 ? 9 : 11;
}
// its LDS: the lower triangle of tiles (or a block, if larger) and a block
__host__ __device__ constexpr int dense_lds_bytes(int nt) { return 8 * (nt * (nt + 1) / 2 * 256 + 16 * nt * 16); }

// Levels jhi down to jlo, each of at most kDenseBlockN vertices, as dense
// matrices in one workgroup (err = 2 on a level that does not fit).
__global__ void __launch_bounds__(kBlockRegsThreads)
    k_block_dense(const BlockJob* __restrict__ jobs, int lds_budget) {
    extern __shared__ double lds[];
    __shared__ double red[16 + 8];
    __shared__ double part[8 * 32];
    __shared__ double s_cm, s_cs;
    __shared__ int s_cfin;
    const BlockJob Jb = jobs[blockIdx.x];
    const LevelDev* __restrict__ lv = Jb.lv;
    if (threadIdx.x == 0 && !Jb.uniform) {
        LevelState c = Jb.st[Jb.jhi + 1];
        s_cm = c.mu;
        s_cs = c.s;
        s_cfin = c.fin;
    }
    __syncthreads();
    for (int j = Jb.jhi; j >= Jb.jlo; --j) {
        const long long t_start = wall_clock64();
        const LevelDev L = lv[j];
        SmallIn in;
        in.uniform = (Jb.uniform && j == Jb.jhi) ? 1 : 0;
        if (!in.uniform) {
            const LevelDev C = lv[j + 1];
            in.cbuf = s_cfin ? C.buf1 : C.buf0;
            in.cfp32 = C.fp32;
        } else {
            in.cbuf = nullptr;
            in.cfp32 = 0;
        }
        in.cm = s_cm;
        in.cs = s_cs;
        in.seed = Jb.seed;
        in.tol = L.kfix > 0 ? -1.0 : Jb.tol;  // a fixed schedule never passes the test
        in.maxit = L.kfix > 0 ? L.kfix : Jb.maxit;
        LevelState o{};
        const int nt = (L.n + 15) / 16;
        if (L.n < 1 || nt > 11 || dense_lds_bytes(dense_tiles(nt)) > lds_budget) o.err = 2;
        else if (nt <= 2) dense_level<2>(L, in, lds, red, part, o);
        else if (nt == 3) dense_level<3>(L, in, lds, red, part, o);
        else if (nt == 4) dense_level<4>(L, in, lds, red, part, o);
        else if (nt <= 6) dense_level<6>(L, in, lds, red, part, o);
        else if (nt <= 8) dense_level<8>(L, in, lds, red, part, o);
        else if (nt == 9) dense_level<9>(L, in, lds, red, part, o);
        else dense_level<11>(L, in, lds, red, part, o);
        if (threadIdx.x == 0) {
            o.ticks = wall_clock64() - t_start;
            Jb.st[j] = o;
            s_cm = o.mu;
            s_cs = o.s;
            s_cfin = o.fin;
        }
        __syncthreads();
    }
}

}  // namespace

namespace {
template <int G, int E, typename W>
const void* block_regs_kernel(int ri) {
    return ri == 0 ? (const void*)k_block_regs<G, 1, E, W> : ri == 1 ? (const void*)k_block_regs<G, 2, E, W>
                                                                    : (const void*)k_block_regs<G, 4, E, W>;
}
template <typename W>
const void* block_layout_kernel(int l, int ri) {
    switch (l) {
        case 0: return block_regs_kernel<1, 8, W>(ri);
        case 1: return block_regs_kernel<2, 8, W>(ri);
        case 2: return block_regs_kernel<4, 8, W>(ri);
        case 3: return block_regs_kernel<8, 8, W>(ri);
        case 4: return block_regs_kernel<1, 16, W>(ri);
        case 5: return block_regs_kernel<2, 16, W>(ri);
        default: return block_regs_kernel<4, 16, W>(ri);
    }
}
// kind 0: CSR traversal; 1 + 3 l + log2(R): register rows of layout l, the
// kinds after those with FP64 weights; the last dense
const void* block_kernel(int kind) {
    if (kind <= 0) return (const void*)k_block_jobs;
    if (kind == kBlockDense) return (const void*)k_block_dense;
    const int q = (kind - 1) % (3 * kRegLayouts);
    return kind - 1 < 3 * kRegLayouts ? block_layout_kernel<float>(q / 3, q % 3)
                                      : block_layout_kernel<double>(q / 3, q % 3);
}
}  // namespace

int refine_block_lds_budget() {
    static int budget = -1;
    if (budget < 0) {
        int dev = 0, maxsh = 65536;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&maxsh, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
        size_t stat = 0;
        for (int r = 0; r < kBlockDense; ++r) {
            hipFuncAttributes fa;
            if (hipFuncGetAttributes(&fa, block_kernel(r)) == hipSuccess) stat = std::max(stat, fa.sharedSizeBytes);
        }
        long b = std::min<long>(kBlockLdsMax, (long)maxsh - (long)stat - 256);
        b = std::max<long>(b, 0);
        for (int r = 0; r < kBlockDense; ++r) {
            if (b > 65536 - (long)stat - 256 &&
                hipFuncSetAttribute(block_kernel(r), hipFuncAttributeMaxDynamicSharedMemorySize, (int)b) != hipSuccess) {
                (void)hipGetLastError();
                b = std::max<long>(0, 65536 - (long)stat - 256);
            }
        }
        budget = (int)(b & ~7L);
    }
    return budget;
}

// The dense kernel asks for LDS beyond the other kernels' budget.
int dense_block_budget() {
    static const int budget = [] {
        int dev = 0, maxsh = 65536;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&maxsh, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, (const void*)k_block_dense) != hipSuccess) return 0;
        const int b = std::min(maxsh - (int)fa.sharedSizeBytes, dense_lds_bytes(dense_tiles(kDenseBlockN / 16)));
        if (hipFuncSetAttribute((const void*)k_block_dense, hipFuncAttributeMaxDynamicSharedMemorySize, b) !=
            hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        return b;
    }();
    return budget;
}

bool dense_block_fits(int n) {
    return n <= kDenseBlockN && dense_lds_bytes(dense_tiles((n + 15) / 16)) <= dense_block_budget();
}

hipError_t launch_block_jobs(const BlockJob* jobs, int njobs, int kind, hipStream_t s) {
    if (kind < 0 || kind >= kBlockKinds) return hipErrorInvalidValue;
    const int budget = kind == kBlockDense ? dense_block_budget() : refine_block_lds_budget();
    void* args[] = {(void*)&jobs, (void*)&budget};
    return hipLaunchKernel(block_kernel(kind), dim3(njobs), dim3(kind ? kBlockRegsThreads : kBlockKernelThreads), args,
                           (size_t)budget, s);
}

}  // namespace cmg
