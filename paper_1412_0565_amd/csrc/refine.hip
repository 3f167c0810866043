// Coarsest solve and cascadic refinement kernels (Algorithm 1, Steps 2-3;
// power iteration, Algorithm 3).
//
// Power iteration on B_g = gI - L with the constant vector deflated.  The
// kernels never normalise a vector in place: a level keeps an unnormalised
// vector w plus scalars (mu, s) with the current iterate
// v = (w - mu) * s, deflated and of unit norm.  One step computes
//   y_i = ((gI - L) v)_i = s * ( g (w_i - mu) + sum_k a_ik (w_k - w_i) )
// (mu cancels in the Laplacian part because L 1 = 0) and, in the same pass,
// the FP64 sums  Sy = sum y, Syy = sum y^2, Syx = sum y v, Sx = sum v.
// From them:  mu' = Sy/n,  ||y - mu'||^2 = Syy - Sy mu',  s' = 1/||.||,
// and the stopping quantity (u, v) = s' (Syx - mu' Sx) for u = (y-mu')s'.
// Every reduction has a fixed order, so results are reproducible bitwise.
#include <algorithm>
#include <mutex>

#include "cmg_internal.h"
#include "jump.h"

namespace cmg {

namespace {

__device__ __forceinline__ double ld_agent(const double* p) {
    unsigned long long b =
        __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __longlong_as_double((long long)b);
}

__device__ __forceinline__ void st_agent(double* p, double v) {
    __hip_atomic_store((unsigned long long*)p, (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup b runs on XCD b % 8; give each XCD a contiguous range of row
// blocks so neighbouring rows (and their x gathers) share one L2.  XCD x
// runs the blocks x, x + 8, ... of [0, nb): nb / 8 of them, one more for the
// first nb % 8 XCDs.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    const int q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

// ~2 s at the 100 MHz constant clock: a safety bound, never reached when
// the grid is co-resident (launches are sized to the measured residency).
constexpr long long kSpinTicks = 200000000LL;

// Grids up to this many workgroups use the all-read form below (measured
// on MI355X: 88 and 112 workgroups 7% and 3% faster per level than with
// the broadcast, 184 workgroups 17% slower).
constexpr int kAllReadMax = 128;

// Spin until *p == e.  The abort flag and the time bound are checked only
// every 64 polls: the flag shares one line that every waiter would hit.
// Returns false (after raising the abort flag, recording the first
// timeout) if the wait was given up.
__device__ __forceinline__ bool spin_until(const unsigned long long* p, unsigned long long e,
                                           GridSync* gs, int nb, int tag) {
    const long long t0 = wall_clock64();
    unsigned polls = 0;
    while (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != e) {
        __builtin_amdgcn_s_sleep(1);
        if ((++polls & 63u) == 0u &&
            (__hip_atomic_load(&gs->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
             wall_clock64() - t0 > kSpinTicks)) {
            if (atomicOr(&gs->abort, 1u) == 0u) {
                gs->where = (unsigned)nb | ((unsigned)(tag + 2) << 16);
                gs->abort_epoch = e;
            }
            return false;
        }
    }
    return true;
}

__device__ __forceinline__ GridSlot* bcast_line(GridSlot* bcast, int q) {
    return (GridSlot*)((char*)bcast + (size_t)q * kBcastStride);
}

// Grid-wide sum of NV (<= 7) doubles with a barrier, free of contended
// atomics: every workgroup writes its block sums and the barrier epoch into
// its own 64-byte slot (release); slots alternate between two banks by
// epoch parity, so a slot is rewritten only after every workgroup has
// passed the barrier in between.
//  * Small grids (nb <= kAllReadMax): every workgroup polls all slots and
//    adds them itself (one memory round trip less).
//  * Larger grids: workgroup 0 polls all slots, adds them and publishes
//    the totals with the epoch on kBcastLines lines that sit on different
//    memory channels (release); workgroup b waits on line b % kBcastLines,
//    so no line has more than nb / kBcastLines pollers.
// Either way the totals are the slot values added in slot order by the
// same fixed tree, so they do not depend on which workgroup adds them or
// on arrival order.  Returns false if the barrier timed out or was aborted;
// then every workgroup leaves.
template <int NV>
__device__ bool grid_allreduce_impl(double (&v)[NV], GridSync* gs, GridSlot* slots, GridSlot* bcast,
                                    unsigned long long& epoch, int vb, int lb, int nb, double* red,
                                    int tag) {
    __shared__ double s_tot[NV];
    __shared__ int s_ok;
    const unsigned long long e = ++epoch;
    GridSlot* bank = slots + (e & 1ull) * (unsigned long long)nb;
    const bool master = vb == 0;
    block_sum<NV>(v, red);
    if (threadIdx.x == 0) {
        GridSlot* my = bank + lb;
#pragma unroll
        for (int q = 0; q < NV; ++q) my->v[q] = v[q];
        __hip_atomic_store(&my->epoch, e, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        s_ok = 1;
    }
    __syncthreads();
    const bool allread = nb <= kAllReadMax;
    if (allread || master) {
        double acc[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] = 0.0;
        for (int b = threadIdx.x; b < nb; b += blockDim.x) {
            if (!spin_until(&bank[b].epoch, e, gs, nb, tag)) {
                s_ok = 0;
                break;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[q] += ld_agent(&bank[b].v[q]);
        }
        block_sum<NV>(acc, red);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int q = 0; q < NV; ++q) s_tot[q] = acc[q];
        }
        if (master && s_ok) {
            if (allread) {
                if (threadIdx.x == 0)
                    __hip_atomic_store(&gs->epoch, e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else if (threadIdx.x < kBcastLines) {
                GridSlot* line = bcast_line(bcast, threadIdx.x);
#pragma unroll
                for (int q = 0; q < NV; ++q) st_agent(&line->v[q], acc[q]);
                __hip_atomic_store(&line->epoch, e, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                if (threadIdx.x == 0)
                    __hip_atomic_store(&gs->epoch, e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else if (threadIdx.x == 0) {
        GridSlot* line = bcast_line(bcast, vb % kBcastLines);
        if (!spin_until(&line->epoch, e, gs, nb, tag)) s_ok = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#pragma unroll
        for (int q = 0; q < NV; ++q) s_tot[q] = ld_agent(&line->v[q]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = s_tot[q];
    const bool ok = s_ok != 0;
    __syncthreads();
    return ok;
}

__device__ __forceinline__ unsigned long long start_epoch(GridSync* gs) {
    return __hip_atomic_load(&gs->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One power-iteration step on rows [r0, r1) with G lanes per row.  Lane 0
// of each group owns the row: writes y and adds {y, y^2, y v, v} to acc.
template <int G, typename T>
__device__ __forceinline__ void pi_rows(const LevelDev& L, const T* __restrict__ win,
                                        T* __restrict__ wout, double mu, double s, int r0, int r1,
                                        double (&acc)[4]) {
    const int lane = threadIdx.x & (G - 1);
    const int ngroups = blockDim.x / G;
    const T* __restrict__ wv = (const T*)(sizeof(T) == 4 ? (const void*)L.w32 : (const void*)L.w64);
    const int32_t* __restrict__ rp = L.rp;
    const int32_t* __restrict__ col = L.col;
    const double g = L.g;
    for (int i = r0 + (int)(threadIdx.x / G); i < r1; i += ngroups) {
        const int a = rp[i], b = rp[i + 1];
        const double wi = (double)win[i];
        double t = 0.0;
        for (int e = a + lane; e < b; e += G) t += (double)wv[e] * ((double)win[col[e]] - wi);
        t = group_sum_t<G>(t);
        if (lane == 0) {
            const double x = (wi - mu) * s;
            const T ys = (T)(s * (g * (wi - mu) + t));
            wout[i] = ys;
            const double yd = (double)ys;
            acc[0] += yd;
            acc[1] += yd * yd;
            acc[2] += yd * x;
            acc[3] += x;
        }
    }
}

template <typename T>
__device__ __forceinline__ void pi_rows_dispatch(int G, const LevelDev& L, const T* win, T* wout,
                                                 double mu, double s, int r0, int r1,
                                                 double (&acc)[4]) {
    switch (G) {
        case 1: pi_rows<1, T>(L, win, wout, mu, s, r0, r1, acc); break;
        case 2: pi_rows<2, T>(L, win, wout, mu, s, r0, r1, acc); break;
        case 4: pi_rows<4, T>(L, win, wout, mu, s, r0, r1, acc); break;
        case 8: pi_rows<8, T>(L, win, wout, mu, s, r0, r1, acc); break;
        case 16: pi_rows<16, T>(L, win, wout, mu, s, r0, r1, acc); break;
        case 32: pi_rows<32, T>(L, win, wout, mu, s, r0, r1, acc); break;
        default: pi_rows<64, T>(L, win, wout, mu, s, r0, r1, acc); break;
    }
}

// ---------------------------------------------------------- coarsest

// coarsest levels up to this size keep A and V in LDS (2 n^2 doubles)
constexpr int kDenseLds = 48;

// Sweeps of the Jacobi iteration in the parallel round-robin
// ("tournament") order on the m x m matrix A (m even, row-major), rotations
// collected in V: m/2 disjoint plane rotations per step, m - 1 steps per
// sweep (disjoint rotations commute, so a step equals applying them one
// after another), until the off-diagonal norm is <= 1e-14 fro.  A step is
// two barriers: the pairs' rotations, then every 2 x 2 block of J^T A J (a
// thread per pair of pairs) and every row of V J.  It is bound by the
// latency of the rotation (estimates in place of two divisions and two
// square roots) and of its LDS trips: n = 25 measured 372 us with rows,
// columns and eigenvalue order in turn.
__device__ __forceinline__ void jacobi_sweeps(double* A, double* V, int m, double fro, double* red, double* cs,
                                              double* sn, int* pp, int* qq) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int np = m / 2;
    const float inv = 1.0f / (float)np;
    for (int sweep = 0; sweep < 50; ++sweep) {
        double o[1] = {0.0};
        for (int t = tid; t < m * m; t += nt)
            if (t / m != t % m) o[0] += A[t] * A[t];
        block_sum<1>(o, red);
        if (sqrt(o[0]) <= 1e-14 * fro) break;
        for (int step = 0; step < m - 1; ++step) {
            for (int i = tid; i < np; i += nt) {
                int a = 0, b = step + 1;
                if (i > 0) {
                    a = step + i >= m - 1 ? step + i - (m - 1) + 1 : step + i + 1;
                    b = step - i < 0 ? step - i + (m - 1) + 1 : step - i + 1;
                }
                const int p = min(a, b), q = max(a, b);
                const double apq = A[p * m + q];
                double c = 1.0, s = 0.0;
                if (fabs(apq) > 1e-30 * fro) {
                    const double tau = 0.5 * (A[q * m + q] - A[p * m + p]) * fast_rcp(apq);
                    const double w = 1.0 + tau * tau;
                    const double t = copysign(fast_rcp(fabs(tau) + w * fast_rsq(w)), tau);
                    c = fast_rsq(1.0 + t * t);
                    s = t * c;
                }
                pp[i] = p;
                qq[i] = q;
                cs[i] = c;
                sn[i] = s;
            }
            __syncthreads();
            for (int t = tid; t < np * np + np * m; t += nt) {
                // t / np by a float product (t < 2^14, exact half-way off an integer)
                const int tq = (int)(((float)t + 0.5f) * inv);
                if (t < np * np) {  // rows of pair i, columns of pair j
                    const int i = tq, j = t - i * np;
                    const int ri = pp[i] * m, rq = qq[i] * m, cj = pp[j], cq = qq[j];
                    const double ci = cs[i], si = sn[i], c = cs[j], s = sn[j];
                    const double x = A[ri + cj], y = A[ri + cq], z = A[rq + cj], w = A[rq + cq];
                    const double x1 = ci * x - si * z, y1 = ci * y - si * w;
                    const double z1 = si * x + ci * z, w1 = si * y + ci * w;
                    A[ri + cj] = c * x1 - s * y1;
                    A[ri + cq] = s * x1 + c * y1;
                    A[rq + cj] = c * z1 - s * w1;
                    A[rq + cq] = s * z1 + c * w1;
                } else {  // row k of V
                    const int k = tq - np, j = t - tq * np;
                    const int cj = k * m + pp[j], cq = k * m + qq[j];
                    const double c = cs[j], s = sn[j];
                    const double x = V[cj], y = V[cq];
                    V[cj] = c * x - s * y;
                    V[cq] = s * x + c * y;
                }
            }
            __syncthreads();
        }
    }
}

// Dense coarsest solve in one workgroup: L^J assembled densely (a zero row
// and column make an odd order even), its eigenvectors by Jacobi iteration.
// The vector is the normalised projection of the ramp z_i = i - (n-1)/2
// onto the eigenspace of all eigenvalues (above the smallest) within
// 1e-10 ||A||_F of lambda_2; a hashed uniform vector replaces z if that
// projection is tiny.
__global__ void __launch_bounds__(256) k_coarse_jobs(const CoarseJob* __restrict__ jobs) {
    extern __shared__ double dyn[];
    const CoarseJob& Jb = jobs[blockIdx.x];
    const LevelDev L = Jb.L;
    LevelState* st = Jb.st;
    double* Vg = Jb.V;
    const uint64_t seed = Jb.seed;
    FinishOut* fo = Jb.fo;
    __shared__ double red[16 * 2 + 8];
    __shared__ double cs_c[64], cs_s[64], ev[128], dots[128];
    __shared__ int pr_p[64], pr_q[64], idx[128];
    const int n = L.n;
    const int m = n + (n & 1);
    const int tid = threadIdx.x, nt = blockDim.x;
    const bool lds = n <= kDenseLds;
    double* A = lds ? dyn : Jb.A;
    double* V = lds ? dyn + m * m : Vg;
    for (int t = tid; t < m * m; t += nt) {
        A[t] = 0.0;
        V[t] = ((t / m) == (t % m)) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int i = tid; i < n; i += nt) {
        double d = 0.0;
        for (int e = L.rp[i]; e < L.rp[i + 1]; ++e) {
            A[i * m + L.col[e]] = -L.w64[e];
            d += L.w64[e];
        }
        A[i * m + i] = d;
    }
    __syncthreads();
    double f[1] = {0.0};
    for (int t = tid; t < m * m; t += nt) f[0] += A[t] * A[t];
    block_sum<1>(f, red);
    const double fro = sqrt(f[0]);
    if (lds) jacobi_sweeps(dyn, dyn + m * m, m, fro, red, cs_c, cs_s, pr_p, pr_q);
    else jacobi_sweeps(Jb.A, Vg, m, fro, red, cs_c, cs_s, pr_p, pr_q);
    // ascending eigenvalues, the lower index first on ties
    // (every index stays valid where a value is not a number)
    for (int k = tid; k < n; k += nt) {
        ev[k] = A[k * m + k];
        idx[k] = k;
    }
    __syncthreads();
    for (int k = tid; k < n; k += nt) {
        const double e = ev[k];
        int rank = 0;
        for (int i = 0; i < n; ++i) rank += (ev[i] < e || (ev[i] == e && i < k)) ? 1 : 0;
        idx[rank] = k;
        Jb.ev[k] = e;
    }
    __syncthreads();
    for (int k = tid; k < n; k += nt) Jb.idx[k] = idx[k];
    const double l2 = ev[idx[1]];
    double* y = (double*)L.buf0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        // dots over the cluster
        for (int r = tid; r < n; r += nt) {
            const int k = idx[r];
            double d = 0.0;
            if (r >= 1 && fabs(ev[k] - l2) <= 1e-10 * fro) {
                for (int i = 0; i < n; ++i) {
                    double z = attempt == 0 ? (double)i - 0.5 * (double)(n - 1)
                                            : hashed_uniform(seed, i) - 0.5;
                    d += V[i * m + k] * z;
                }
            }
            dots[r] = d;
        }
        __syncthreads();
        double acc[2] = {0.0, 0.0};
        for (int i = tid; i < n; i += nt) {
            double yi = 0.0;
            for (int r = 1; r < n; ++r) yi += dots[r] * V[i * m + idx[r]];
            y[i] = yi;
            acc[0] += yi * yi;
            double z = attempt == 0 ? (double)i - 0.5 * (double)(n - 1) : hashed_uniform(seed, i) - 0.5;
            acc[1] += z * z;
        }
        block_sum<2>(acc, red);
        if (sqrt(acc[0]) >= 1e-8 * sqrt(acc[1]) || attempt == 1) {
            double inv = 1.0 / sqrt(acc[0]);
            for (int i = tid; i < n; i += nt) y[i] *= inv;
            break;
        }
        __syncthreads();
    }
    // the eigenvectors are left in Vg with rows of n (several-eigenpair
    // starts read them), from global memory by way of A
    if (lds) {
        for (int t = tid; t < n * n; t += nt) Vg[t] = V[(t / n) * m + t % n];
    } else if (m != n) {
        for (int t = tid; t < n * n; t += nt) Jb.A[t] = V[(t / n) * m + t % n];
        __syncthreads();
        for (int t = tid; t < n * n; t += nt) Vg[t] = Jb.A[t];
    }
    if (tid == 0) {
        int mult = 0;
        for (int r = 1; r < n; ++r)
            if (fabs(ev[idx[r]] - l2) <= 1e-10 * fro) ++mult;
        LevelState s0;
        s0.mu = 0.0;
        s0.s = 1.0;
        s0.mu_prev = 0.0;
        s0.s_prev = 1.0;
        s0.utv = 1.0;
        s0.margin = 0.0;
        s0.fin = 0;
        s0.k = -1;
        s0.maxit = 0;
        s0.err = 0;
        s0.ticks = 0;
        *st = s0;
        fo->coarse_lambda2 = l2;
        fo->coarse_mult = mult;
    }
}

// ------------------------------------------------------- grid levels

// A job's view of the launch: jobs of a packed launch own disjoint ranges
// of workgroups; a single-graph launch is one job.  Every job has its own
// barrier state, so graphs refined together never wait for each other.
struct GridCtx {
    GridSync* gs;
    GridSlot* slots;
    GridSlot* bcast;
    unsigned long long epoch;
    int nb;  // workgroups of the job
    int vb;  // this workgroup within the job
    int lb;  // row block of this workgroup
    int tag;
};

template <int NV>
__device__ __forceinline__ bool job_allreduce(double (&v)[NV], GridCtx& c, double* red) {
    return grid_allreduce_impl<NV>(v, c.gs, c.slots, c.bcast, c.epoch, c.vb, c.lb, c.nb, red, c.tag);
}

// ---- per-row operations fed by the two traversal drivers
//
// Edge weights are read through WRead<W>: W = double or float (an FP32
// copy, used only where every weight of the level is exact in FP32),
// uint8_t or uint16_t (a copy where every weight is an integer in 1..255
// or 1..65535), or
// WUnit where every weight is 1 and nothing is read.  The value is the
// same double in all of them, so results do not depend on the storage.
struct WUnit {};
template <typename W, bool LDS = false>
struct WRead {
    const W* __restrict__ p;
    __device__ __forceinline__ double operator[](int e) const {
        if constexpr (LDS) return (double)sld(p, e);
        else return (double)gld(p, e);
    }
};
template <bool LDS>
struct WRead<WUnit, LDS> {
    const void* p;
    __device__ __forceinline__ double operator[](int) const { return 1.0; }
};
// storage type of kind WK for iterates of type T
template <typename T, int WK>
struct WStore {
    using type = T;
};
template <typename T>
struct WStore<T, kWF32> {
    using type = float;
};
template <typename T>
struct WStore<T, kWUnit> {
    using type = WUnit;
};
template <typename T>
struct WStore<T, kWU8> {
    using type = uint8_t;
};
template <typename T>
struct WStore<T, kWU16> {
    using type = uint16_t;
};
// the level's weights of kind WK for iterates of type T
template <typename T, int WK>
__device__ __forceinline__ WRead<typename WStore<T, WK>::type> weights_of(const LevelDev& L) {
    WRead<typename WStore<T, WK>::type> r;
    if constexpr (WK == kWUnit) r.p = nullptr;
    else if constexpr (WK == kWU8) r.p = L.w8;
    else if constexpr (WK == kWU16) r.p = L.w16;
    else if constexpr (WK == kWF32 || sizeof(T) == 4) r.p = L.w32;
    else r.p = L.w64;
    return r;
}
// the finishing pass reads FP64 weights, or the exact FP32 copy, or none
template <int WK>
using FinW = WRead<typename WStore<double, WK>::type>;
template <int WK>
__device__ __forceinline__ FinW<WK> fin_weights(const LevelDev& L) {
    return weights_of<double, WK>(L);
}

// One PI step: y_i = s (g (w_i - mu) + sum_k a_ik (w_k - w_i)), stored as
// T; acc += {y, y^2, y v, v} with v = (w_i - mu) s.
// Rows and entries are numbered from the arrays the traversal reads (the
// level's, or with STG a workgroup's LDS stage); vector index = row + roff.
template <typename T, int WK, bool STG = false>
struct PiOp {
    const int32_t* __restrict__ col;
    WRead<typename WStore<T, WK>::type, STG> wv;
    const T* __restrict__ win;
    T* __restrict__ wout;
    int roff;
    double mu, s, g;
    double acc[4];
    __device__ __forceinline__ double xi(int i) const { return (double)gld(win, roff + i); }
    __device__ __forceinline__ int vidx(int i) const { return roff + i; }
    // an entry's term split into its loads (column and weight, then the
    // gathered vector value) and its arithmetic, so a traversal can issue
    // the loads of several entries before it adds their terms in order
    __device__ __forceinline__ int colof(int e) const {
        if constexpr (STG) return sld(col, e);
        else return gld(col, e);
    }
    __device__ __forceinline__ double wof(int e) const { return wv[e]; }
    __device__ __forceinline__ double xk(int c) const { return (double)gld(win, c); }
    __device__ __forceinline__ double term(double xc, double wt, double x) const { return wt * (xc - x); }
    __device__ __forceinline__ double entry(int e, double x) const { return term(xk(colof(e)), wof(e), x); }
    __device__ __forceinline__ double entry_cw(int c, double wt, double x) const { return term(xk(c), wt, x); }
    __device__ __forceinline__ void row(int i, double x, double t) {
        const double v = (x - mu) * s;
        const T ys = (T)(s * (g * (x - mu) + t));
        gst(wout, roff + i, ys);
        const double yd = (double)ys;
        acc[0] += yd;
        acc[1] += yd * yd;
        acc[2] += yd * v;
        acc[3] += v;
    }
};

// One product of a jump (jump.h): y_i = al x_i + be (-L x)_i - ga z_i with z
// the vector before x, which y replaces (the first product has ga = 0 and
// keeps x in jback); jsum += cj y; acc = {(x, y), (y, y), (x, x)}.
template <int WK, bool STG = false>
struct JumpOp {
    const int32_t* __restrict__ col;
    WRead<typename WStore<double, WK>::type, STG> wv;
    const double* __restrict__ win;
    double* wout;
    double* jsum;
    double* jback;
    int roff;
    bool first;
    double be, cj;
    double acc[3];
    __device__ __forceinline__ double xi(int i) const { return gld(win, roff + i); }
    __device__ __forceinline__ int vidx(int i) const { return roff + i; }
    __device__ __forceinline__ int colof(int e) const {
        if constexpr (STG) return sld(col, e);
        else return gld(col, e);
    }
    __device__ __forceinline__ double wof(int e) const { return wv[e]; }
    __device__ __forceinline__ double xk(int c) const { return gld(win, c); }
    __device__ __forceinline__ double term(double xc, double wt, double x) const { return wt * (xc - x); }
    __device__ __forceinline__ double entry(int e, double x) const { return term(xk(colof(e)), wof(e), x); }
    __device__ __forceinline__ double entry_cw(int c, double wt, double x) const { return term(xk(c), wt, x); }
    __device__ __forceinline__ void row(int i, double x, double t) {
        const int q = roff + i;
        double y, sum;
        if (first) {
            y = x + be * t;
            sum = x;
            gst(jback, q, x);
        } else {
            const double z = gld(wout, q);
            sum = gld(jsum, q);
            y = 2.0 * x + be * t - z;
        }
        gst(wout, q, y);
        gst(jsum, q, sum + cj * y);
        acc[0] += x * y;
        acc[1] += y * y;
        acc[2] += x * x;
    }
};

// FP64 recomputation of a step from a (possibly FP32) iterate.
template <int WK>
struct RedoOp {
    const int32_t* __restrict__ col;
    FinW<WK> w;
    const void* src;
    int f32;
    double* __restrict__ dst;
    double mu, s, g;
    double acc[2];
    __device__ __forceinline__ double xi(int i) const { return ld_any(src, f32, i); }
    __device__ __forceinline__ int vidx(int i) const { return i; }
    __device__ __forceinline__ int colof(int e) const { return gld(col, e); }
    __device__ __forceinline__ double wof(int e) const { return w[e]; }
    __device__ __forceinline__ double xk(int c) const { return ld_any(src, f32, c); }
    __device__ __forceinline__ double term(double xc, double wt, double x) const { return wt * (xc - x); }
    __device__ __forceinline__ double entry(int e, double x) const { return term(xk(colof(e)), wof(e), x); }
    __device__ __forceinline__ double entry_cw(int c, double wt, double x) const { return term(xk(c), wt, x); }
    __device__ __forceinline__ void row(int i, double x, double t) {
        const double y = s * (g * (x - mu) + t);
        gst(dst, i, y);
        acc[0] += y;
        acc[1] += y * y;
    }
};

// Sums of u = (src - mu) s and the edge form sum_k a_ik ((src_k - src_i) s)^2.
template <int WK>
struct EdgeOp {
    const int32_t* __restrict__ col;
    FinW<WK> w;
    const void* src;
    int f32;
    double mu, s;
    double acc[3];
    __device__ __forceinline__ double xi(int i) const { return ld_any(src, f32, i); }
    __device__ __forceinline__ int vidx(int i) const { return i; }
    __device__ __forceinline__ int colof(int e) const { return gld(col, e); }
    __device__ __forceinline__ double wof(int e) const { return w[e]; }
    __device__ __forceinline__ double xk(int c) const { return ld_any(src, f32, c); }
    __device__ __forceinline__ double term(double xc, double wt, double x) const {
        const double d = (xc - x) * s;
        return wt * d * d;
    }
    __device__ __forceinline__ double entry(int e, double x) const { return term(xk(colof(e)), wof(e), x); }
    __device__ __forceinline__ double entry_cw(int c, double wt, double x) const { return term(xk(c), wt, x); }
    __device__ __forceinline__ void row(int i, double x, double t) {
        const double u = (x - mu) * s;
        acc[0] += u;
        acc[1] += u * u;
        acc[2] += t;
    }
};

// Output y = (u - mean)/nrm and residual terms (L y - lambda y)_i.
template <int WK>
struct ResidualOp {
    const int32_t* __restrict__ col;
    FinW<WK> w;
    const void* src;
    int f32;
    double mu, s, mean_u, nrm, lam;
    double* __restrict__ yout;
    double acc[1];
    __device__ __forceinline__ double xi(int i) const { return ld_any(src, f32, i); }
    __device__ __forceinline__ int vidx(int i) const { return i; }
    __device__ __forceinline__ int colof(int e) const { return gld(col, e); }
    __device__ __forceinline__ double wof(int e) const { return w[e]; }
    __device__ __forceinline__ double xk(int c) const { return ld_any(src, f32, c); }
    __device__ __forceinline__ double term(double xc, double wt, double x) const { return wt * (x - xc); }
    __device__ __forceinline__ double entry(int e, double x) const { return term(xk(colof(e)), wof(e), x); }
    __device__ __forceinline__ double entry_cw(int c, double wt, double x) const { return term(xk(c), wt, x); }
    __device__ __forceinline__ void row(int i, double x, double t) {
        const double yi = ((x - mu) * s - mean_u) / nrm;
        const double r = t * s / nrm - lam * yi;
        acc[0] += r * r;
        gst(yout, i, yi);
    }
};

// ---- traversal driver 1: G lanes per row (G = 64: a wavefront per row)
//
// Each lane group takes two rows at a time (rows i and i + ngroups) so the
// loads of both are in flight together; the rows are still emitted in the
// order i, i + ngroups, i + 2 ngroups, ... of a one-row loop.
//
// Rows with more than lmin entries (the hubs of a skewed degree
// distribution; lrows lists them in ascending order after their count) are
// left out of the groups' loop and summed afterwards by the whole
// workgroup, one after the other in ascending order, so a hub row no longer
// holds one lane group while the others idle.  `red` is block_sum scratch;
// rows r of the traversal are rows r + loff of the list (an LDS stage).

__device__ __forceinline__ int lower_bound_i32(const int32_t* __restrict__ a, int n, int v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (gld(a, mid) < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The first kRowBatch entries of each lane in a row are loaded before any
// of them is added: all column and weight loads of both rows are issued,
// then all their vector gathers, then the terms are added in entry order
// (so the sums are those of the plain loop), and a row with more entries
// finishes in the loop.  Without the batch a lane waits for a column and
// then its gather once per entry.  The loads are unconditional, so no
// loaded value passes through a branch (which would make the compiler wait
// for it early): a slot past the row's end reads the entry before the row
// end (a valid index whenever the level has entries; the term is then
// dropped) and gathers the row's own vector value.
constexpr int kRowBatch = 2;

template <int U, int G, class Op>
__device__ __forceinline__ void rows_batch(const Op& op, int lane, int self1, int a1, int b1, double x1, double& t1,
                                           int self2, int a2, int b2, double x2, double& t2) {
    int c1[U], c2[U];
    double w1[U], w2[U], y1[U], y2[U];
    const int z1 = max(b1 - 1, 0), z2 = max(b2 - 1, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e1 = a1 + lane + u * G, e2 = a2 + lane + u * G;
        const int q1 = e1 < b1 ? e1 : z1, q2 = e2 < b2 ? e2 : z2;
        c1[u] = op.colof(q1);
        w1[u] = op.wof(q1);
        c2[u] = op.colof(q2);
        w2[u] = op.wof(q2);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        y1[u] = op.xk(a1 + lane + u * G < b1 ? c1[u] : self1);
        y2[u] = op.xk(a2 + lane + u * G < b2 ? c2[u] : self2);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const double v1 = op.term(y1[u], w1[u], x1);
        const double v2 = op.term(y2[u], w2[u], x2);
        t1 = a1 + lane + u * G < b1 ? t1 + v1 : t1;
        t2 = a2 + lane + u * G < b2 ? t2 + v2 : t2;
    }
}

// SRP: the row pointers are an LDS stage (else global memory).
template <bool SRP>
__device__ __forceinline__ int ld_rp(const int32_t* rp, int i) {
    if constexpr (SRP) return sld(rp, i);
    else return gld(rp, i);
}

// A lane's entries e, e + G, ... of a row up to b, four per trip, while
// four remain: e is left at the first entry not taken.
template <int G, typename Op>
__device__ __forceinline__ void row_rest4(const Op& op, int& e, int b, double x, double& t) {
    for (; e + 3 * G < b; e += 4 * G) {
        int c[4];
        double w[4], v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = op.colof(e + q * G);
            w[q] = op.wof(e + q * G);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = op.xk(c[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) t += op.term(v[q], w[q], x);
    }
}

// the long rows of [r0, r1) (listed in lrows), each summed by the whole
// workgroup
template <bool SRP = false, bool HUB4 = false, typename Op>
__device__ __forceinline__ void drive_long_rows(const int32_t* __restrict__ rp, int r0, int r1, Op& op,
                                                const int32_t* __restrict__ lrows, double* red, int loff = 0) {
    const int cnt = gld(lrows, 0);
    const int32_t* lr = lrows + 1;
    const int q1 = lower_bound_i32(lr, cnt, r1 + loff);
    for (int q = lower_bound_i32(lr, cnt, r0 + loff); q < q1; ++q) {
        const int r = gld(lr, q) - loff;
        const int a = ld_rp<SRP>(rp, r), b = ld_rp<SRP>(rp, r + 1);
        const double x = op.xi(r);
        double t[1] = {0.0};
        // HUB4: each thread's entries four per trip, their loads in flight
        // together (a hub row holds one workgroup while the grid waits)
        const int bd = (int)blockDim.x;
        int e = a + (int)threadIdx.x;
        for (; HUB4 && e + 3 * bd < b; e += 4 * bd) {
            int c[4];
            double w[4], v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = op.colof(e + q * bd);
                w[q] = op.wof(e + q * bd);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = op.xk(c[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[0] += op.term(v[q], w[q], x);
        }
        for (; e < b; e += bd) t[0] += op.entry(e, x);
        block_sum<1>(t, red);
        if (threadIdx.x == 0) op.row(r, x, t[0]);
    }
}

template <int G, bool SRP = false, bool REST4 = false, class Op>
__device__ __forceinline__ void drive_rows(const int32_t* __restrict__ rp, int r0, int r1, Op& op,
                                           const int32_t* __restrict__ lrows = nullptr, int lmin = 0x7fffffff,
                                           double* red = nullptr, int loff = 0) {
    const int lane = threadIdx.x & (G - 1);
    const int ngroups = blockDim.x / G;
    int i = r0 + (int)(threadIdx.x / G);
    for (; i + ngroups < r1; i += 2 * ngroups) {
        const int i2 = i + ngroups;
        const int a1 = ld_rp<SRP>(rp, i), a2 = ld_rp<SRP>(rp, i2);
        int b1 = ld_rp<SRP>(rp, i + 1), b2 = ld_rp<SRP>(rp, i2 + 1);
        const bool l1 = b1 - a1 > lmin, l2 = b2 - a2 > lmin;
        if (l1) b1 = a1;
        if (l2) b2 = a2;
        const double x1 = op.xi(i), x2 = op.xi(i2);
        double t1 = 0.0, t2 = 0.0;
        rows_batch<kRowBatch, G>(op, lane, op.vidx(i), a1, b1, x1, t1, op.vidx(i2), a2, b2, x2, t2);
        int e1 = a1 + lane + kRowBatch * G, e2 = a2 + lane + kRowBatch * G;
        if constexpr (REST4) {
            // rows of hundreds of entries: each lane's rest in trips of
            // four, their columns and weights, then their gathers, in
            // flight together (the sum keeps the entry order); only where
            // the registers allow it (the step kernels: the persistent
            // kernels' cap would spill)
            row_rest4<G>(op, e1, b1, x1, t1);
            row_rest4<G>(op, e2, b2, x2, t2);
        }
        while (e1 < b1 || e2 < b2) {
            if (e1 < b1) {
                t1 += op.entry(e1, x1);
                e1 += G;
            }
            if (e2 < b2) {
                t2 += op.entry(e2, x2);
                e2 += G;
            }
        }
        t1 = group_sum_t<G>(t1);
        t2 = group_sum_t<G>(t2);
        if (lane == 0) {
            if (!l1) op.row(i, x1, t1);
            if (!l2) op.row(i2, x2, t2);
        }
    }
    if (i < r1) {
        const int a = ld_rp<SRP>(rp, i), b = ld_rp<SRP>(rp, i + 1);
        if (b - a <= lmin) {
            const double x = op.xi(i);
            double t = 0.0;
            for (int e = a + lane; e < b; e += G) t += op.entry(e, x);
            t = group_sum_t<G>(t);
            if (lane == 0) op.row(i, x, t);
        }
    }
    // levels of 32 or 64 lanes per row (skewed degrees, hub rows) batch the
    // hub rows' loads; on the others the extra registers would spill
    if (lrows != nullptr) drive_long_rows<SRP, (G >= 32)>(rp, r0, r1, op, lrows, red, loff);
}

// ---- traversal driver 2: merge path
//
// The block's rows [r0, r1) and entries are merged into one sequence
// (the entries of a row followed by its row end) that is cut into equal
// pieces of kMergeIPT items per thread, so a row of any length is shared
// by many threads and a chunk of short rows by few (Merrill & Garland,
// "Merge-based parallel sparse matrix-vector multiplication", SC 2016).
// Per chunk the row ends and the chunk's entries (columns and weights, a
// contiguous range starting where the previous chunk's ended) are copied to
// LDS with coalesced loads, every thread finds its start by binary search
// on its diagonal and walks its items from there, and the partial sums of
// rows split across threads are combined by a segmented scan in thread
// order (deterministic), then added by the thread that completes the row.
// The entry arithmetic is the operation's own, so staging changes no
// result.
constexpr int kMergeIPT = 8;
constexpr int kMergeChunk = kGridBlock * kMergeIPT;

struct MergeShared {
    int win[kMergeChunk + 2];  // row starts/ends of rows ia .. ia + W (relative to the block's first entry)
    int scol[kMergeChunk];     // entries js .. js + kMergeChunk (relative to the block's first entry)
    double sw[kMergeChunk];
    int crow[kGridBlock];
    double cval[kGridBlock];
    int wrow[16];
    int wfirst[16];
    double wtail[16];
    int inrow[17];
    double inval[17];
    int s_ia, s_js;
};

template <class Op>
__device__ __forceinline__ void drive_merge(const int32_t* __restrict__ rp, int r0, int r1, Op& op,
                                            MergeShared& sh) {
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
    const int e0 = gld(rp, r0);
    const int nrows = r1 - r0;
    const int nent = gld(rp, r1) - e0;
    const int total = nrows + nent;
    int carry_row = -1;
    double carry_val = 0.0;
    int ia = 0, js = 0;
    for (int d0 = 0; d0 < total; d0 += kMergeChunk) {
        const int dl_end = min(kMergeChunk, total - d0);
        const int W = min(kMergeChunk + 1, nrows - ia);  // rows whose ends can lie in this chunk
        for (int q = tid; q <= W; q += blockDim.x) sh.win[q] = gld(rp, r0 + ia + q) - e0;
        // the chunk's entries start where the previous chunk's ended and
        // are at most kMergeChunk (those past its end serve the next one)
        const int ns = min(kMergeChunk, nent - js);
        for (int q = tid; q < ns; q += blockDim.x) {
            sh.scol[q] = op.colof(e0 + js + q);
            sh.sw[q] = op.wof(e0 + js + q);
        }
        __syncthreads();
        // start coordinate (i, j) on my diagonal: i rows completed, j entries consumed
        const int dl = min(tid * kMergeIPT, dl_end);
        const int diag = d0 + dl;
        int lo = max(ia, diag - nent), hi = min(ia + W, diag);
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sh.win[mid - ia + 1] <= diag - mid - 1) lo = mid + 1;
            else hi = mid;
        }
        int i = lo, j = diag - lo;
        const int steps = min(dl + kMergeIPT, dl_end) - dl;
        double x = (i < nrows) ? op.xi(r0 + i) : 0.0;
        double part = 0.0;
        int frow = -1;
        double fx = 0.0, fpart = 0.0;
        for (int q = 0; q < steps; ++q) {
            if (i < nrows && j < sh.win[i - ia + 1]) {
                part += op.entry_cw(sh.scol[j - js], sh.sw[j - js], x);
                ++j;
            } else {
                if (frow < 0) {
                    frow = i;
                    fx = x;
                    fpart = part;
                } else {
                    op.row(r0 + i, x, part);
                }
                part = 0.0;
                ++i;
                x = (i < nrows) ? op.xi(r0 + i) : 0.0;
            }
        }
        if (tid * kMergeIPT < dl_end && min(tid * kMergeIPT + kMergeIPT, dl_end) == dl_end) {
            sh.s_ia = i;
            sh.s_js = j;
        }
        // inclusive segmented scan of the carries (rows are non-decreasing in tid)
        int myrow = i;
        double v = part;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int ro = __shfl_up(myrow, o, 64);
            const double vo = __shfl_up(v, o, 64);
            if (lane >= o && ro == myrow) v += vo;
        }
        const int first_in_wave = __shfl(myrow, 0, 64);
        if (lane == 63) {
            sh.wrow[wv] = myrow;
            sh.wtail[wv] = v;
            sh.wfirst[wv] = first_in_wave;
        }
        __syncthreads();
        if (tid == 0) {
            int r = carry_row;
            double cv = carry_val;
            for (int w = 0; w < nw; ++w) {
                sh.inrow[w] = r;
                sh.inval[w] = cv;
                const bool whole = sh.wfirst[w] == sh.wrow[w];
                const double tail = sh.wtail[w] + ((whole && r == sh.wrow[w]) ? cv : 0.0);
                r = sh.wrow[w];
                cv = tail;
            }
            sh.inrow[nw] = r;
            sh.inval[nw] = cv;
        }
        __syncthreads();
        if (myrow == first_in_wave && myrow == sh.inrow[wv]) v += sh.inval[wv];
        sh.crow[tid] = myrow;
        sh.cval[tid] = v;
        __syncthreads();
        if (frow >= 0) {
            double cin = 0.0;
            if (tid == 0) {
                if (carry_row == frow) cin = carry_val;
            } else if (sh.crow[tid - 1] == frow) {
                cin = sh.cval[tid - 1];
            }
            op.row(r0 + frow, fx, fpart + cin);
        }
        carry_row = sh.inrow[nw];
        carry_val = sh.inval[nw];
        ia = sh.s_ia;
        js = sh.s_js;
        __syncthreads();
    }
}

// ---- merge path, a workgroup's share held in registers
//
// A jump multiplies by the same matrix some 60 to 400 times.  Where a
// workgroup's share is at most kMergeHeld items and kMergeRegRows rows,
// every thread keeps the columns and weights of its own items, and the
// rows' vector values and sums stay in LDS, so a product is one batch of
// gathers, the walk, the scan and the rows' update; nothing but the vector
// is read from memory.  Bound by those latencies (7 us at 4000 items) and
// the grid barrier (8 us at 200 workgroups).  drive_merge reads everything
// again behind the barrier, which invalidates the L2: 28700 rows of 759000
// entries took 24 us a product, this way 15.5.  Shares for more workgroups
// than CUs were slower: two on one CU take twice as long as the others.
constexpr int kMergeRegIPT = kMergeHeld / kGridBlock;
constexpr int kMergeRowsPer = 3;  // own rows per thread
constexpr int kMergeRegRows = kMergeRowsPer * kGridBlock;
static_assert(2 * kMergeRegRows <= kMergeChunk, "both in MergeShared::sw; the others half as long each");

template <int WK>
struct MergeRegs {
    using W = std::conditional_t<WK == kWNative, double, float>;  // exact for every other storage
    int c[kMergeRegIPT];   // columns of the items that are entries
    W w[kMergeRegIPT];
    uint32_t ents, ends;   // items that are entries / row ends
    int row0, row;         // first row, and the row after the last item (of the workgroup's)
};

// False (in every thread) where the share is larger.
template <int WK>
__device__ __forceinline__ bool merge_regs_load(const LevelDev& L, int r0, int r1, const double* win, MergeRegs<WK>& m,
                                                MergeShared& sh) {
    const int tid = (int)threadIdx.x;
    const int e0 = gld(L.rp, r0);
    const int nrows = r1 - r0;
    const int nent = gld(L.rp, r1) - e0;
    const int total = nrows + nent;
    if (total > kMergeHeld || nrows > kMergeRegRows || nrows < 1) return false;
    const auto wv = weights_of<double, WK>(L);
    const int diag = min(tid * kMergeRegIPT, total);
    int lo = max(0, diag - nent), hi = min(nrows, diag);
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (gld(L.rp, r0 + mid + 1) - e0 <= diag - mid - 1) lo = mid + 1;
        else hi = mid;
    }
    int i = lo, e = e0 + diag - lo;
    m.row0 = i;
    m.ents = m.ends = 0;
    int end = i < nrows ? gld(L.rp, r0 + i + 1) : e;
#pragma unroll
    for (int q = 0; q < kMergeRegIPT; ++q) {
        m.c[q] = r0;  // a vector value that is there; the item drops it
        m.w[q] = 0;
        if (diag + q >= total) continue;
        if (e < end) {
            m.ents |= 1u << q;
            m.c[q] = gld(L.col, e);
            m.w[q] = (typename MergeRegs<WK>::W)wv[e];
            ++e;
        } else {
            m.ends |= 1u << q;
            ++i;
            if (i < nrows) end = gld(L.rp, r0 + i + 1);
        }
    }
    m.row = i;
#pragma unroll
    for (int t = 0; t < kMergeRowsPer; ++t) {
        const int r = tid + t * kGridBlock;
        if (r < nrows) sh.sw[r] = gld(win, r0 + r);
    }
    __syncthreads();
    return true;
}

// Product of a jump (as JumpOp with drive_merge): y = T_{j+1} to op.wout.
template <int WK>
__device__ __forceinline__ void merge_regs_product(JumpOp<WK>& op, int r0, int nrows, bool last, MergeRegs<WK>& m,
                                                   MergeShared& sh) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // own rows: T_j, the sums of the entries, T_{j-1} and the jump's sum (the
    // grid barrier before each product orders them)
    double* rx = sh.sw;
    double* rs = sh.sw + kMergeRegRows;
    double* rz = (double*)sh.win;
    double* rj = (double*)sh.scol;
    double y[kMergeRegIPT];
#pragma unroll
    for (int q = 0; q < kMergeRegIPT; ++q) y[q] = op.xk(m.c[q]);
    int i = m.row0, frow = -1;
    double part = 0.0, fpart = 0.0;
    double x = i < nrows ? rx[i] : 0.0;
#pragma unroll
    for (int q = 0; q < kMergeRegIPT; ++q) {
        if ((m.ents >> q) & 1) part += op.term(y[q], (double)m.w[q], x);
        if ((m.ends >> q) & 1) {
            if (frow < 0) {
                frow = i;
                fpart = part;
            } else {
                rs[i] = part;
            }
            part = 0.0;
            ++i;
            x = i < nrows ? rx[i] : 0.0;
        }
    }
    // inclusive segmented scan of the carries (rows are non-decreasing in tid)
    const int myrow = m.row;
    double v = part;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int ro = __shfl_up(myrow, o, 64);
        const double vo = __shfl_up(v, o, 64);
        if (lane >= o && ro == myrow) v += vo;
    }
    const int first = __shfl(myrow, 0, 64);
    if (lane == 63) {
        sh.wrow[wv] = myrow;
        sh.wtail[wv] = v;
        sh.wfirst[wv] = first;
    }
    __syncthreads();
    // what the wavefronts before carry into this one
    int crow = -1;
    double cval = 0.0;
#pragma unroll
    for (int w = 0; w < kGridBlock / 64; ++w) {
        const int rw = sh.wrow[w];
        const double tail = sh.wtail[w] + (sh.wfirst[w] == rw && crow == rw ? cval : 0.0);
        if (w < wv) {
            crow = rw;
            cval = tail;
        }
    }
    if (myrow == first && myrow == crow) v += cval;
    int prow = __shfl_up(myrow, 1, 64);
    double pval = __shfl_up(v, 1, 64);
    if (lane == 0) {
        prow = crow;
        pval = cval;
    }
    if (frow >= 0) rs[frow] = fpart + (prow == frow ? pval : 0.0);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kMergeRowsPer; ++t) {
        const int r = tid + t * kGridBlock;
        if (r >= nrows) continue;
        const double xr = rx[r], s = rs[r];
        double yr, sum;
        if (op.first) {
            yr = xr + op.be * s;
            sum = xr;
            gst(op.jback, r0 + r, xr);
        } else {
            yr = 2.0 * xr + op.be * s - rz[r];
            sum = rj[r];
        }
        gst(op.wout, r0 + r, yr);
        sum += op.cj * yr;
        if (last) gst(op.jsum, r0 + r, sum);
        rj[r] = sum;
        rz[r] = xr;
        rx[r] = yr;
        op.acc[0] += xr * yr;
        op.acc[1] += yr * yr;
        op.acc[2] += xr * xr;
    }
}

// TRAV = 0: merge path; TRAV = G > 0: G lanes per row.
template <int TRAV, class Op>
__device__ __forceinline__ void drive(const LevelDev& L, int r0, int r1, Op& op, MergeShared* sh, double* red) {
    if constexpr (TRAV == 0) {
        drive_merge(L.rp, r0, r1, op, *sh);
    } else {
        drive_rows<TRAV>(L.rp, r0, r1, op, L.lrows, L.lmin, red);
    }
}

// ---- a workgroup's rows staged in LDS
//
// A grid barrier's acquire invalidates the L2, so on a level whose
// workgroup shares are small every step would fetch the row pointers,
// columns and weights again before it can gather.  When a workgroup's rows
// and entries fit the LDS stage (FP64 levels, G lanes per row) they are
// copied there once per level and the steps read them from LDS through the
// same traversal; only the vector gathers go to memory.  Rows and entries
// are visited in the same order, so the sums are bit for bit those of the
// global traversal.
constexpr int kStageRows = kGridStageRows;
constexpr int kStageEnts = 3840;
struct StageLds {
    int32_t rp[kStageRows + 1];  // row pointers relative to the first entry
    int32_t col[kStageEnts];
    double w[kStageEnts];
};

// ---- the products of a jump over K steps (jump.h) from buf[cur], whose sum
// is left in jsum, and the verdict's inputs: the first workgroup keeps the
// moments, samples (u, v) over the jump and sends the result to the others.
// Rows are shared as in the plain steps (see refine_level).
template <int TRAV, int WK>
__device__ __forceinline__ bool jump_products_run(const LevelDev& L, GridCtx& c, int K, double tol, int cur,
                                                  bool staged, StageLds* stg, MergeShared* sh, double* red, int r0,
                                                  int r1, int x0, int x1, int xp, int np, int& safe, int& next) {
    using WT = typename WStore<double, WK>::type;
    const int d = jump_products(K);
    double cj = 2.0 * (double)K / (double)(K + 1);
    double* bufs[2] = {(double*)L.buf0, (double*)L.buf1};
    const double be1 = 2.0 / L.g;
    MergeRegs<WK> mr;
    bool held = false;
    if constexpr (TRAV == 0) held = merge_regs_load<WK>(L, r0, r1, bufs[cur], mr, *sh);
    for (int j = 0; j < d; ++j) {
        double acc[3];
        if (TRAV > 0 && staged) {
            if constexpr (TRAV > 0) {
                JumpOp<WK, true> op;
                op.col = stg->col;
                if constexpr (WK != kWUnit) op.wv.p = (const WT*)stg->w;
                op.win = cur ? bufs[1] : bufs[0];
                op.wout = cur ? bufs[0] : bufs[1];
                op.jsum = L.jsum;
                op.jback = L.jback;
                op.roff = r0;
                op.first = j == 0;
                op.be = j == 0 ? be1 : 2.0 * be1;
                op.cj = cj;
                op.acc[0] = op.acc[1] = op.acc[2] = 0.0;
                drive_rows<TRAV, true>(stg->rp, 0, r1 - r0, op, L.lrows, L.lmin, red, r0);
#pragma unroll
                for (int q = 0; q < 3; ++q) acc[q] = op.acc[q];
            }
        } else {
            JumpOp<WK> op;
            op.col = L.col;
            op.wv = weights_of<double, WK>(L);
            op.win = cur ? bufs[1] : bufs[0];
            op.wout = cur ? bufs[0] : bufs[1];
            op.jsum = L.jsum;
            op.jback = L.jback;
            op.roff = 0;
            op.first = j == 0;
            op.be = j == 0 ? be1 : 2.0 * be1;
            op.cj = cj;
            op.acc[0] = op.acc[1] = op.acc[2] = 0.0;
            if constexpr (TRAV == 0) {
                if (held) merge_regs_product<WK>(op, r0, r1 - r0, j == d - 1, mr, *sh);
                else drive_merge(L.rp, r0, r1, op, *sh);
            } else if (L.ileave) {
                const int cw = 4 * ((int)blockDim.x / TRAV);
                for (int a = x0 + xp * cw; a < x1; a += np * cw)
                    drive_rows<TRAV>(L.rp, a, min(a + cw, x1), op, nullptr, L.lmin, red);
                if (L.lrows != nullptr) drive_long_rows<false, (TRAV >= 32)>(L.rp, r0, r1, op, L.lrows, red);
            } else {
                drive_rows<TRAV>(L.rp, r0, r1, op, L.lrows, L.lmin, red);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[q] = op.acc[q];
        }
        if (!job_allreduce<3>(acc, c, red)) return false;
        if (c.vb == 0 && threadIdx.x == 0) jump_moments(L.jmom, j, acc[0], acc[1], acc[2]);
        cj = jump_coef(cj, K, j + 1);
        cur ^= 1;
    }
    double vd[2] = {0.0, 0.0};
    if (c.vb == 0 && tol >= 0.0) {
        double* dl = L.jmom + kJumpMoments;
        __syncthreads();
        for (int q = threadIdx.x; q < kJumpSamples; q += blockDim.x)
            dl[q] = jump_delta(L.jmom, 2 * d + 1, jump_sample(q, kJumpSamples, K));
        __syncthreads();
        if (threadIdx.x < 64) {
            int sf, nx;
            jump_judge(dl, kJumpSamples, K, tol, &sf, &nx);
            if (threadIdx.x == 0) {
                vd[0] = (double)sf;
                vd[1] = (double)nx;
            }
        }
    }
    if (!job_allreduce<2>(vd, c, red)) return false;
    safe = (int)vd[0];
    next = (int)vd[1];
    return true;
}

// ---- refinement of one level by a job's workgroups

template <typename T, int TRAV, int WK>
__device__ void refine_level(const GridJob& J, GridCtx& c, double* red, MergeShared* sh, StageLds* stg) {
    const LevelDev& L = J.L;
    const double tol = J.tol;
    const int maxit = J.maxit;
    const uint64_t seed = J.seed;
    const int r0 = L.part[c.lb], r1 = L.part[c.lb + 1];
    T* b0 = (T*)L.buf0;
    T* b1 = (T*)L.buf1;
    const double n = (double)L.n;
    // traversal arrays of the PI steps: the level's, or the LDS stage
    // (weights staged in their storage type; none where all are 1)
    using WT = typename WStore<T, WK>::type;
    PiOp<T, WK> op;
    op.col = L.col;
    op.wv = weights_of<T, WK>(L);
    op.roff = 0;
    op.g = L.g;
    PiOp<T, WK, true> ops;
    bool staged = false;
    if constexpr (TRAV > 0 && sizeof(T) == 8) {
        const int a0 = gld(L.rp, r0), a1 = gld(L.rp, r1);
        // the same in every thread of the workgroup
        if (stg != nullptr && L.stage && !L.ileave && r1 - r0 <= kStageRows && a1 - a0 <= kStageEnts) {
            for (int i = threadIdx.x; i <= r1 - r0; i += blockDim.x) stg->rp[i] = gld(L.rp, r0 + i) - a0;
            for (int e = threadIdx.x; e < a1 - a0; e += blockDim.x) {
                stg->col[e] = gld(L.col, a0 + e);
                if constexpr (WK != kWUnit) ((WT*)stg->w)[e] = gld(op.wv.p, a0 + e);
            }
            __syncthreads();
            ops.col = stg->col;
            if constexpr (WK != kWUnit) ops.wv.p = (const WT*)stg->w;
            ops.roff = r0;
            ops.g = L.g;
            staged = true;
        }
    }
    // interleaved steps: this workgroup's XCD holds parts xl0 .. xl0 + np - 1
    // (the grouping of xcd_remap); their rows [x0, x1) go in chunks of four
    // passes, chunk q to the workgroup at position q mod np
    int x0 = r0, x1 = r1, xp = 0, np = 1;
    if (TRAV > 0 && L.ileave) {
        const int q = c.nb >> 3, rr = c.nb & 7, x = c.vb & 7;
        const int xl0 = x * q + min(x, rr);
        np = q + (x < rr ? 1 : 0);
        xp = c.vb >> 3;
        x0 = gld(L.part, xl0);
        x1 = gld(L.part, xl0 + np);
    }
    // prolongation from level j+1 (or the hashed uniform start)
    double sum[1] = {0.0};
    if (J.uniform) {
        for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
            const T v = (T)(hashed_uniform(seed, i) - 0.5);
            gst(b0, i, v);
            sum[0] += (double)v;
        }
    } else {
        const LevelState cst = *J.stc;
        const void* cb = cst.fin ? J.C.buf1 : J.C.buf0;
        for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
            const T v = (T)((ld_any(cb, J.C.fp32, gld(L.agg, i)) - cst.mu) * cst.s);
            gst(b0, i, v);
            sum[0] += (double)v;
        }
    }
    // mean and norm of the vector in b0, whose sum the workgroups hold
    double mu = 0.0, s = 0.0;
    auto normalise = [&](double (&sm)[1]) -> bool {
        if (!job_allreduce<1>(sm, c, red)) return false;
        mu = sm[0] / n;
        double ss[1] = {0.0};
        for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
            const double d = (double)gld(b0, i) - mu;
            ss[0] += d * d;
        }
        if (!job_allreduce<1>(ss, c, red)) return false;
        s = 1.0 / sqrt(ss[0]);
        return true;
    };
    if (!normalise(sum)) return;
    int cur = 0, k = 0, hit = 0;
    double utv = 0.0, pmu = mu, ps = s;
    const bool jumps = sizeof(T) == 8 && L.jmom != nullptr && (tol < 0.0 || tol >= kJumpTolMin);
    int since = 0, hold = 0;  // plain steps since the last jump, and to take before the next estimate
    while (true) {
        double acc[4];
        if (TRAV > 0 && staged) {
            ops.win = cur ? b1 : b0;
            ops.wout = cur ? b0 : b1;
            ops.mu = mu;
            ops.s = s;
            ops.acc[0] = ops.acc[1] = ops.acc[2] = ops.acc[3] = 0.0;
            if constexpr (TRAV > 0 && sizeof(T) == 8)
                drive_rows<TRAV, true>(stg->rp, 0, r1 - r0, ops, L.lrows, L.lmin, red, r0);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = ops.acc[q];
        } else {
            op.win = cur ? b1 : b0;
            op.wout = cur ? b0 : b1;
            op.mu = mu;
            op.s = s;
            op.acc[0] = op.acc[1] = op.acc[2] = op.acc[3] = 0.0;
            if constexpr (TRAV == 0) {
                drive_merge(L.rp, r0, r1, op, *sh);
            } else if (L.ileave) {
                const int cw = 4 * ((int)blockDim.x / TRAV);
                for (int a = x0 + xp * cw; a < x1; a += np * cw)
                    drive_rows<TRAV>(L.rp, a, min(a + cw, x1), op, nullptr, L.lmin, red);
                if (L.lrows != nullptr) drive_long_rows<false, (TRAV >= 32)>(L.rp, r0, r1, op, L.lrows, red);
            } else {
                drive_rows<TRAV>(L.rp, r0, r1, op, L.lrows, L.lmin, red);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = op.acc[q];
        }
        if (!job_allreduce<4>(acc, c, red)) return;
        const double mu2 = acc[0] / n;
        const double s2 = 1.0 / sqrt(acc[1] - acc[0] * mu2);
        const double utvp = utv;
        utv = s2 * (acc[2] - mu2 * acc[3]);
        ++k;
        cur ^= 1;
        pmu = mu;
        ps = s;
        mu = mu2;
        s = s2;
        if (!(utv < 1.0 - tol)) break;
        if (k >= maxit) {
            hit = 1;
            break;
        }
        if constexpr (sizeof(T) == 8) {
            if (hold > 0) {
                --hold;
                continue;
            }
            if (!jumps || !jump_due(++since)) continue;
            const double r = 1.0 / (s * L.g);
            int K = jump_plan(utv, utvp, tol, r, maxit - k - 1);
            while (K > 0) {
                int safe = 0, next = 0;
                if (!jump_products_run<TRAV, WK>(L, c, K, tol, cur, staged, stg, sh, red, r0, r1, x0, x1, xp, np, safe,
                                                 next))
                    return;
                int more = 0;
                double sm[1] = {0.0};
                since = 0;
                cur = 0;
                if (jump_verdict(K, safe, next, tol < 0.0, &more, &hold)) {
                    k += K;
                    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
                        const double v = gld(L.jsum, i);
                        gst((double*)L.buf0, i, v);
                        sm[0] += v;
                    }
                    if (!normalise(sm)) return;
                } else {
                    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x)
                        gst((double*)L.buf0, i, gld(L.jback, i));
                    if (!job_allreduce<1>(sm, c, red)) return;
                }
                K = more > 0 ? jump_steps((double)more, r, maxit - k - 1) : 0;
            }
        }
    }
    if (c.vb == 0 && threadIdx.x == 0) {
        LevelState o;
        o.mu = mu;
        o.s = s;
        o.mu_prev = pmu;
        o.s_prev = ps;
        o.utv = utv;
        o.margin = utv - (1.0 - tol);
        o.fin = cur;
        o.k = k;
        o.maxit = hit;
        o.err = 0;
        o.ticks = 0;
        *J.st = o;
    }
}

// ---- finishing pass on the finest level
//
// With `redo` = 1 (mixed precision) the last power-iteration step is
// recomputed in FP64 from the FP32 iterate before it, so the step count
// equals the FP64 path and only that earlier iterate carries FP32
// rounding.  Then the output y = deflated, normalised iterate, the
// edge-form Rayleigh quotient r = sum_edges w (y_i - y_k)^2 and the
// residual ||L y - r y||, all in FP64.
template <int TRAV, int WK>
__device__ void finish_level(const GridJob& J, GridCtx& c, double* red, MergeShared* sh) {
    const LevelDev& L = J.L;
    const int r0 = L.part[c.lb], r1 = L.part[c.lb + 1];
    const double n = (double)L.n;
    const LevelState st = *J.stc;
    const void* src = st.fin ? L.buf1 : L.buf0;
    int f32 = L.fp32;
    double mu = st.mu, s = st.s;
    if (J.redo && st.k > 0) {
        RedoOp<WK> op;
        op.col = L.col;
        op.w = fin_weights<WK>(L);
        op.src = st.fin ? L.buf0 : L.buf1;
        op.f32 = f32;
        op.dst = J.fa;
        op.mu = st.mu_prev;
        op.s = st.s_prev;
        op.g = L.g;
        op.acc[0] = op.acc[1] = 0.0;
        drive<TRAV>(L, r0, r1, op, sh, red);
        if (!job_allreduce<2>(op.acc, c, red)) return;
        mu = op.acc[0] / n;
        s = 1.0 / sqrt(op.acc[1] - op.acc[0] * mu);
        src = J.fa;
        f32 = 0;
    }
    EdgeOp<WK> eo;
    eo.col = L.col;
    eo.w = fin_weights<WK>(L);
    eo.src = src;
    eo.f32 = f32;
    eo.mu = mu;
    eo.s = s;
    eo.acc[0] = eo.acc[1] = eo.acc[2] = 0.0;
    drive<TRAV>(L, r0, r1, eo, sh, red);
    if (!job_allreduce<3>(eo.acc, c, red)) return;
    const double mean_u = eo.acc[0] / n;
    const double nrm2 = eo.acc[1] - eo.acc[0] * mean_u;
    const double nrm = sqrt(nrm2);
    const double lam = 0.5 * eo.acc[2] / nrm2;
    ResidualOp<WK> ro;
    ro.col = L.col;
    ro.w = fin_weights<WK>(L);
    ro.src = src;
    ro.f32 = f32;
    ro.mu = mu;
    ro.s = s;
    ro.mean_u = mean_u;
    ro.nrm = nrm;
    ro.lam = lam;
    ro.yout = J.yout;
    ro.acc[0] = 0.0;
    drive<TRAV>(L, r0, r1, ro, sh, red);
    if (!job_allreduce<1>(ro.acc, c, red)) return;
    if (c.vb == 0 && threadIdx.x == 0) {
        J.fo->lambda = lam;
        J.fo->residual = sqrt(ro.acc[0]);
        J.fo->sum_u = eo.acc[0];
        J.fo->sum_uu = eo.acc[1];
        J.fo->edge = eo.acc[2];
    }
}

// Which job owns this workgroup (jobs sorted by first workgroup).
__device__ __forceinline__ int find_job(const GridJob* jobs, int njobs) {
    int lo = 0, hi = njobs - 1;
    const int b = blockIdx.x;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].b0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ GridCtx make_ctx(const GridJob& J) {
    GridCtx c;
    c.gs = J.gs;
    c.slots = J.slots;
    c.bcast = J.bcast;
    c.nb = J.L.grid;
    c.vb = (int)blockIdx.x - J.b0;
    c.lb = xcd_remap(c.vb, c.nb);
    c.epoch = start_epoch(J.gs);
    c.tag = J.tag;
    return c;
}

// nslots: the slot array holds two banks of nslots
__global__ void k_raise_abort(GridSync* gs) {
    if (threadIdx.x == 0) atomicOr(&gs->abort, 1u);
}

__global__ void k_reset_sync(GridSync* gs, GridSlot* slots, int nslots, GridSlot* bcast) {
    nslots *= 2;
    for (int b = threadIdx.x; b < nslots; b += blockDim.x) {
        for (int q = 0; q < 7; ++q) slots[b].v[q] = 0.0;
        slots[b].epoch = 0ull;
    }
    if (threadIdx.x < kBcastLines) {
        GridSlot* line = bcast_line(bcast, threadIdx.x);
        for (int q = 0; q < 7; ++q) line->v[q] = 0.0;
        line->epoch = 0ull;
    }
    if (threadIdx.x == 0) {
        gs->epoch = 0ull;
        gs->abort = 0u;
        gs->where = 0u;
        gs->abort_epoch = 0ull;
    }
}

// Residency count: each workgroup counts itself in, raises the recorded
// peak, stays `hold` ticks and counts itself out.  The peak is how many
// workgroups of this kernel the device keeps resident at once.
__device__ void residency_count(const GridJob& J) {
    if (threadIdx.x == 0) {
        const unsigned now = atomicAdd(J.count, 1u) + 1u;
        atomicMax(J.count + 1, now);
    }
    __syncthreads();
    const long long t0 = wall_clock64();
    while (wall_clock64() - t0 < J.hold) __builtin_amdgcn_s_sleep(2);
    __syncthreads();
    if (threadIdx.x == 0) atomicSub(J.count, 1u);
}

// One launch refines one level of each job (one graph per job).  Kernels
// are specialised by traversal (merge path, or G lanes per row) and
// storage precision to keep registers low; a packed launch holds one kind.
template <int TRAV, typename T, int WK>
__device__ __forceinline__ void refine_entry(const GridJob* __restrict__ jobs, int njobs, double* red,
                                             MergeShared* sh, StageLds* stg) {
    const GridJob J = jobs[find_job(jobs, njobs)];
    if (J.tag == kResidencyTag) {
        residency_count(J);
        return;
    }
    GridCtx c = make_ctx(J);
    if (c.vb < 0 || c.vb >= c.nb) return;
    refine_level<T, TRAV, WK>(J, c, red, sh, stg);
}

// At most 128 VGPRs: two workgroups of 512 threads per CU.
template <typename T, int WK>
__global__ void __launch_bounds__(kGridBlock) __attribute__((amdgpu_waves_per_eu(4)))
k_refine_merge(const GridJob* __restrict__ jobs, int njobs) {
    __shared__ double red[16 * 5 + 8];
    __shared__ MergeShared msh;
    refine_entry<0, T, WK>(jobs, njobs, red, &msh, nullptr);
}

// G lanes per row.  Held to 6 waves per SIMD (at most 80 VGPRs): grids
// run at most 3 workgroups of 512 threads per CU.
template <int G, typename T, int WK>
__global__ void __launch_bounds__(kGridBlock) __attribute__((amdgpu_waves_per_eu(6, 6)))
k_refine_rows(const GridJob* __restrict__ jobs, int njobs) {
    __shared__ double red[16 * 5 + 8];
    StageLds* stg = nullptr;
    if constexpr (sizeof(T) == 8) {
        __shared__ StageLds st;
        stg = &st;
    }
    refine_entry<G, T, WK>(jobs, njobs, red, nullptr, stg);
}

// One launch finishes the finest level of each job.
template <int TRAV, int WK>
__global__ void __launch_bounds__(kGridBlock) k_finish_jobs(const GridJob* __restrict__ jobs, int njobs) {
    __shared__ double red[16 * 5 + 8];
    MergeShared* sh = nullptr;
    if constexpr (TRAV == 0) {
        __shared__ MergeShared msh;
        sh = &msh;
    }
    const GridJob J = jobs[find_job(jobs, njobs)];
    if (J.tag == kResidencyTag) {
        residency_count(J);
        return;
    }
    GridCtx c = make_ctx(J);
    if (c.vb < 0 || c.vb >= c.nb) return;
    finish_level<TRAV, WK>(J, c, red, sh);
}

// ------------------------------------------ large levels: a launch per step
//
// The same arithmetic as refine_level, with the grid-wide sums formed by a
// one-workgroup kernel after each launch instead of a grid barrier inside
// it: each workgroup posts its block sums, the check kernel adds the posts
// in workgroup order, applies the stopping test and leaves (mu, s) for the
// next step.  A step launched after the test passed returns at once.

constexpr int kCheckThreads = 1024;

template <int NV>
__device__ __forceinline__ void post_part(double (&v)[NV], double* red, double* part, int slot) {
    block_sum<NV>(v, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) part[4 * (size_t)slot + q] = v[q];
    }
}

// fixed-order total of the posts of nb workgroups, in every thread
template <int NV>
__device__ __forceinline__ void sum_parts(const double* part, int nb, double (&v)[NV], double* red) {
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] += part[4 * (size_t)b + q];
    }
    block_sum<NV>(v, red);
}

// prolongation (or the hashed uniform start) into buf0; posts its sum
template <typename T>
__global__ void __launch_bounds__(kStepBlock) k_step_prolong(const StepJob* __restrict__ jp) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    const LevelDev& L = J.L;
    const int lb = xcd_remap((int)blockIdx.x, (int)gridDim.x);  // row block, posted in row order
    const int r0 = L.part[lb], r1 = L.part[lb + 1];
    T* b0 = (T*)L.buf0;
    double sum[1] = {0.0};
    if (J.uniform) {
        for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
            const T v = (T)(hashed_uniform(J.seed, i) - 0.5);
            gst(b0, i, v);
            sum[0] += (double)v;
        }
    } else {
        const LevelState cst = *J.stc;
        const void* cb = cst.fin ? J.C.buf1 : J.C.buf0;
        for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
            const T v = (T)((ld_any(cb, J.C.fp32, gld(L.agg, i)) - cst.mu) * cst.s);
            gst(b0, i, v);
            sum[0] += (double)v;
        }
    }
    post_part<1>(sum, red, J.part, lb);
}

// mean of the start vector
__global__ void __launch_bounds__(kCheckThreads) k_step_mean(const StepJob* __restrict__ jp, int nb) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    double v[1];
    sum_parts<1>(J.part, nb, v, red);
    if (threadIdx.x == 0) J.ctl->mu = v[0] / (double)J.L.n;
}

// squared distance of the start vector from its mean
template <typename T>
__global__ void __launch_bounds__(kStepBlock) k_step_sumsq(const StepJob* __restrict__ jp) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    const LevelDev& L = J.L;
    const int lb = xcd_remap((int)blockIdx.x, (int)gridDim.x);  // row block, posted in row order
    const int r0 = L.part[lb], r1 = L.part[lb + 1];
    const T* b0 = (const T*)L.buf0;
    const double mu = J.ctl->mu;
    double ss[1] = {0.0};
    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
        const double d = (double)gld(b0, i) - mu;
        ss[0] += d * d;
    }
    post_part<1>(ss, red, J.part, lb);
}

// normalisation of the start vector; arms the step loop
__global__ void __launch_bounds__(kCheckThreads) k_step_norm(const StepJob* __restrict__ jp, int nb) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    double v[1];
    sum_parts<1>(J.part, nb, v, red);
    if (threadIdx.x == 0) {
        StepCtl* c = J.ctl;
        const double mu = c->mu;
        const double s = 1.0 / sqrt(v[0]);
        c->s = s;
        c->pmu = mu;
        c->ps = s;
        c->utv = 0.0;
        c->k = 0;
        c->cur = 0;
        c->done = 0;
        c->hit = 0;
        c->mode = 0;
        c->since = c->hold = c->more = 0;
    }
}

// one power-iteration step: buf[cur] -> buf[cur ^ 1], posts {y, y^2, y v, v}
template <int G, typename T, int WK>
__global__ void __launch_bounds__(kStepBlock) k_step_spmv(const StepJob* __restrict__ jp) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    const StepCtl c = *J.ctl;
    if (c.done) return;
    const LevelDev& L = J.L;
    const int lb = xcd_remap((int)blockIdx.x, (int)gridDim.x);  // row block, posted in row order
    const int r0 = L.part[lb], r1 = L.part[lb + 1];
    if constexpr (sizeof(T) == 8) {
        if (c.mode > 2) {  // the end of a jump (StepCtl)
            double* b0 = (double*)L.buf0;
            const double* src = c.mode == 3 ? L.jsum : c.mode == 4 ? b0 : L.jback;
            double sum[3] = {0.0, 0.0, 0.0};
            for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
                const double v = gld(src, i);
                if (c.mode != 4) gst(b0, i, v);
                sum[0] += c.mode == 4 ? (v - c.mu) * (v - c.mu) : v;
            }
            post_part<3>(sum, red, J.part, lb);
            return;
        }
        if (c.mode > 0) {  // a product of a jump
            JumpOp<WK> op;
            op.col = L.col;
            op.wv = weights_of<double, WK>(L);
            op.win = (const double*)(c.cur ? L.buf1 : L.buf0);
            op.wout = (double*)(c.cur ? L.buf0 : L.buf1);
            op.jsum = L.jsum;
            op.jback = L.jback;
            op.roff = 0;
            op.first = c.mode == 1;
            op.be = (c.mode == 1 ? 2.0 : 4.0) / L.g;
            op.cj = c.cj;
            op.acc[0] = op.acc[1] = op.acc[2] = 0.0;
            drive_rows<G, false, (G >= 32)>(L.rp, r0, r1, op, L.lrows, L.lmin, red);
            post_part<3>(op.acc, red, J.part, lb);
            return;
        }
    }
    PiOp<T, WK> op;
    op.col = L.col;
    op.wv = weights_of<T, WK>(L);
    op.roff = 0;
    op.g = L.g;
    op.win = (const T*)(c.cur ? L.buf1 : L.buf0);
    op.wout = (T*)(c.cur ? L.buf0 : L.buf1);
    op.mu = c.mu;
    op.s = c.s;
    op.acc[0] = op.acc[1] = op.acc[2] = op.acc[3] = 0.0;
    drive_rows<G, false, (G >= 32)>(L.rp, r0, r1, op, L.lrows, L.lmin, red);
    post_part<4>(op.acc, red, J.part, lb);
}

// arms a jump of K steps (0: plain steps)
__device__ __forceinline__ void step_arm(StepCtl& c, int K) {
    c.mode = K > 0 ? 1 : 0;
    c.j = 0;
    c.K = K;
    c.d = jump_products(K);
    c.cj = 2.0 * (double)K / (double)(K + 1);
}

// sums of the step, stopping test, state for the next step; writes the
// level state when the level is done
__global__ void __launch_bounds__(kCheckThreads) k_step_check(const StepJob* __restrict__ jp, int nb) {
    __shared__ double red[16 * 5 + 8];
    const StepJob J = *jp;
    StepCtl c = *J.ctl;
    if (c.done) return;
    const double n = (double)J.L.n;
    double acc[4];
    sum_parts<4>(J.part, nb, acc, red);
    if (c.mode == 0) {
        if (threadIdx.x != 0) return;
        const double mu2 = acc[0] / n;
        const double s2 = 1.0 / sqrt(acc[1] - acc[0] * mu2);
        c.utvp = c.utv;
        c.utv = s2 * (acc[2] - mu2 * acc[3]);
        ++c.k;
        c.cur ^= 1;
        c.pmu = c.mu;
        c.ps = c.s;
        c.mu = mu2;
        c.s = s2;
        if (!(c.utv < 1.0 - J.tol)) {
            c.done = 1;
        } else if (c.k >= J.maxit) {
            c.done = 1;
            c.hit = 1;
        } else if (c.hold > 0) {
            --c.hold;
        } else if (J.L.jmom != nullptr && J.tol >= kJumpTolMin && jump_due(++c.since)) {
            c.r = 1.0 / (c.s * J.L.g);
            step_arm(c, jump_plan(c.utv, c.utvp, J.tol, c.r, J.maxit - c.k - 1));
        }
        *J.ctl = c;
        if (c.done) {
            LevelState o;
            o.mu = c.mu;
            o.s = c.s;
            o.mu_prev = c.pmu;
            o.s_prev = c.ps;
            o.utv = c.utv;
            o.margin = c.utv - (1.0 - J.tol);
            o.fin = c.cur;
            o.k = c.k;
            o.maxit = c.hit;
            o.err = 0;
            o.ticks = 0;
            *J.st = o;
        }
        return;
    }
    if (c.mode <= 2) {
        double* mom = J.L.jmom;
        if (threadIdx.x == 0) jump_moments(mom, c.j, acc[0], acc[1], acc[2]);
        ++c.j;
        c.cj = jump_coef(c.cj, c.K, c.j);
        c.cur ^= 1;
        c.mode = 2;
        if (c.j == c.d) {  // the last product: sample (u, v) over the jump
            double* dl = mom + kJumpMoments;
            __syncthreads();
            for (int q = threadIdx.x; q < kJumpSamples; q += blockDim.x)
                dl[q] = jump_delta(mom, 2 * c.d + 1, jump_sample(q, kJumpSamples, c.K));
            __syncthreads();
            if (threadIdx.x >= 64) return;
            int safe, next;
            jump_judge(dl, kJumpSamples, c.K, J.tol, &safe, &next);
            c.since = 0;
            const bool keep = jump_verdict(c.K, safe, next, false, &c.more, &c.hold);
            if (keep) c.k += c.K;
            c.mode = keep ? 3 : 5;
        }
    } else if (c.mode == 3) {
        c.mu = acc[0] / n;
        c.mode = 4;
    } else {
        if (c.mode == 4) c.s = 1.0 / sqrt(acc[0]);
        c.cur = 0;
        step_arm(c, c.more > 0 ? jump_steps((double)c.more, c.r, J.maxit - c.k - 1) : 0);
    }
    if (threadIdx.x == 0) *J.ctl = c;
}

}  // namespace

// ================================================================ launchers

hipError_t launch_coarse_jobs(const CoarseJob* jobs, int njobs, hipStream_t s) {
    const size_t shmem = sizeof(double) * 2 * kDenseLds * kDenseLds;
    hipLaunchKernelGGL(k_coarse_jobs, dim3(njobs), dim3(256), shmem, s, jobs);
    return hipGetLastError();
}

namespace {
// kind = 16 wk + 2 t + fp32 with t = 0 (merge path) or 1 + log2(G) and wk
// the weight storage (FP32 iterates have no kWF32 form: FP32 is their own)
template <int TRAV, int WK>
const void* refine_kernel_w(int fp32) {
    if constexpr (TRAV == 0) {
        if constexpr (WK == kWF32) return (const void*)k_refine_merge<double, kWF32>;
        else return fp32 ? (const void*)k_refine_merge<float, WK> : (const void*)k_refine_merge<double, WK>;
    } else if constexpr (WK == kWF32) {
        return (const void*)k_refine_rows<TRAV, double, kWF32>;
    } else {
        return fp32 ? (const void*)k_refine_rows<TRAV, float, WK> : (const void*)k_refine_rows<TRAV, double, WK>;
    }
}
template <int TRAV>
const void* refine_kernel_t(int fp32, int wk) {
    return wk == kWUnit ? refine_kernel_w<TRAV, kWUnit>(fp32)
           : wk == kWF32 ? refine_kernel_w<TRAV, kWF32>(fp32)
           : wk == kWU8  ? refine_kernel_w<TRAV, kWU8>(fp32)
           : wk == kWU16 ? refine_kernel_w<TRAV, kWU16>(fp32)
                         : refine_kernel_w<TRAV, kWNative>(fp32);
}
const void* refine_kernel(int kind) {
    const int fp32 = kind & 1, wk = kind >> 4;
    switch ((kind >> 1) & 7) {
        case 0: return refine_kernel_t<0>(fp32, wk);
        case 1: return refine_kernel_t<1>(fp32, wk);
        case 2: return refine_kernel_t<2>(fp32, wk);
        case 3: return refine_kernel_t<4>(fp32, wk);
        case 4: return refine_kernel_t<8>(fp32, wk);
        case 5: return refine_kernel_t<16>(fp32, wk);
        case 6: return refine_kernel_t<32>(fp32, wk);
        default: return refine_kernel_t<64>(fp32, wk);
    }
}
template <int TRAV>
const void* finish_kernel_t(int wk) {
    return wk == kWUnit ? (const void*)k_finish_jobs<TRAV, kWUnit>
           : wk == kWF32 ? (const void*)k_finish_jobs<TRAV, kWF32>
           : wk == kWU8  ? (const void*)k_finish_jobs<TRAV, kWU8>
           : wk == kWU16 ? (const void*)k_finish_jobs<TRAV, kWU16>
                         : (const void*)k_finish_jobs<TRAV, kWNative>;
}
const void* finish_kernel(int kind) {
    const int wk = kind >> 4;
    switch ((kind >> 1) & 7) {
        case 0: return finish_kernel_t<0>(wk);
        case 1: return finish_kernel_t<1>(wk);
        case 2: return finish_kernel_t<2>(wk);
        case 3: return finish_kernel_t<4>(wk);
        case 4: return finish_kernel_t<8>(wk);
        case 5: return finish_kernel_t<16>(wk);
        case 6: return finish_kernel_t<32>(wk);
        default: return finish_kernel_t<64>(wk);
    }
}
// Workgroups of kernel `k` that can be resident at once.  The occupancy
// query alone can promise more than the device delivers (for kernels at
// 64 VGPRs and about 90 SGPRs it reports 4 workgroups of 512 threads per CU
// where 3 are resident), and a grid barrier over workgroups that are not
// all resident never completes.  So the kernel itself is launched once in
// residency-count mode at the queried size and the observed peak is used,
// rounded down to a multiple of 8.  Returns 0 on any error.
thread_local MeasureBuffers t_meas{nullptr, nullptr, nullptr};

int max_blocks_ptr(const void* k) {
    int dev = 0, ncu = 0, occ = 0, khz = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, kGridBlock, 0) != hipSuccess) return 0;
    const int want = occ * ncu;
    if (want <= 0) return 0;
    unsigned* cnt = nullptr;
    GridJob* dj = nullptr;
    hipStream_t s = nullptr;
    unsigned peak[2] = {0u, 0u};
    const bool own = t_meas.cnt == nullptr;  // else buffers and stream given by the caller
    // the count needs an idle device: work already queued (a coarsest solve
    // launched during setup, another thread's solve) finishes first
    bool ok = hipDeviceSynchronize() == hipSuccess;
    if (ok && own) {
        ok = hipMalloc((void**)&cnt, 2 * sizeof(unsigned)) == hipSuccess &&
             hipMalloc((void**)&dj, sizeof(GridJob)) == hipSuccess &&
             hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess;
    } else if (ok) {
        cnt = t_meas.cnt;
        dj = t_meas.job;
        s = t_meas.stream;
    }
    if (ok) {
        GridJob j{};
        j.tag = kResidencyTag;
        j.count = cnt;
        j.hold = (long long)khz;  // 1 ms: dispatch of the grid takes microseconds
        j.b0 = 0;
        int njobs = 1;
        void* args[] = {(void*)&dj, &njobs};
        ok = hipMemsetAsync(cnt, 0, 2 * sizeof(unsigned), s) == hipSuccess &&
             hipMemcpyAsync(dj, &j, sizeof(GridJob), hipMemcpyHostToDevice, s) == hipSuccess &&
             hipLaunchKernel(k, dim3(want), dim3(kGridBlock), args, 0, s) == hipSuccess &&
             hipMemcpyAsync(peak, cnt, 2 * sizeof(unsigned), hipMemcpyDeviceToHost, s) == hipSuccess &&
             hipStreamSynchronize(s) == hipSuccess;
    }
    if (own) {
        if (s) (void)hipStreamDestroy(s);
        if (dj) (void)hipFree(dj);
        if (cnt) (void)hipFree(cnt);
    }
    if (!ok) {
        (void)hipGetLastError();
        return 0;
    }
    const int got = std::min<int>(want, (int)peak[1]);
    return got >= 8 ? (got / 8) * 8 : got;
}
}  // namespace

void set_measure_buffers(const MeasureBuffers* b) { t_meas = b ? *b : MeasureBuffers{nullptr, nullptr, nullptr}; }

int job_kind(int variant, int lanes, int fp32, int wk) {
    int t = 0;
    if (variant != 2) {
        t = 1;
        for (int g = lanes; g > 1 && t < 7; g >>= 1) ++t;
    }
    // FP32 iterates read FP32 weights (their native storage)
    if (fp32 && wk == kWF32) wk = kWNative;
    return 16 * wk + 2 * t + (fp32 ? 1 : 0);
}

namespace {
std::mutex g_cap_mutex;
int g_refine_cap[kJobKinds];
int g_finish_cap[kJobKinds];
bool g_caps_init = false;
}  // namespace

// Measured once per kernel and process (the first call launches it).
void caps_init() {
    if (g_caps_init) return;
    for (int k = 0; k < kJobKinds; ++k) g_refine_cap[k] = g_finish_cap[k] = -1;
    g_caps_init = true;
}

int refine_jobs_max_blocks(int kind) {
    std::lock_guard<std::mutex> lock(g_cap_mutex);
    caps_init();
    if (g_refine_cap[kind] < 0) g_refine_cap[kind] = max_blocks_ptr(refine_kernel(kind));
    return g_refine_cap[kind];
}

int finish_jobs_max_blocks(int kind) {
    std::lock_guard<std::mutex> lock(g_cap_mutex);
    caps_init();
    if (g_finish_cap[kind] < 0) g_finish_cap[kind] = max_blocks_ptr(finish_kernel(kind));
    return g_finish_cap[kind];
}

// Grid launches are plain launches of at most the measured co-resident
// workgroup count: on an otherwise idle device every workgroup is resident
// at once, which is all the grid barrier needs.  (A cooperative launch
// costs about 17 us more per launch on MI355X and gave no protection from
// kernels on other streams either; the barrier's bounded wait turns such
// a case into CMG_E_DEVICE.)
hipError_t launch_refine_jobs(const GridJob* jobs, int njobs, int nblocks, int kind, hipStream_t s) {
    void* args[] = {(void*)&jobs, &njobs};
    return hipLaunchKernel(refine_kernel(kind), dim3(nblocks), dim3(kGridBlock), args, 0, s);
}

hipError_t launch_finish_jobs(const GridJob* jobs, int njobs, int nblocks, int kind, hipStream_t s) {
    void* args[] = {(void*)&jobs, &njobs};
    return hipLaunchKernel(finish_kernel(kind), dim3(nblocks), dim3(kGridBlock), args, 0, s);
}

hipError_t launch_step_begin(const StepJob* job, int nblocks, int kind, hipStream_t s) {
    if (kind & 1) {
        hipLaunchKernelGGL(k_step_prolong<float>, dim3(nblocks), dim3(kStepBlock), 0, s, job);
        hipLaunchKernelGGL(k_step_mean, dim3(1), dim3(kCheckThreads), 0, s, job, nblocks);
        hipLaunchKernelGGL(k_step_sumsq<float>, dim3(nblocks), dim3(kStepBlock), 0, s, job);
    } else {
        hipLaunchKernelGGL(k_step_prolong<double>, dim3(nblocks), dim3(kStepBlock), 0, s, job);
        hipLaunchKernelGGL(k_step_mean, dim3(1), dim3(kCheckThreads), 0, s, job, nblocks);
        hipLaunchKernelGGL(k_step_sumsq<double>, dim3(nblocks), dim3(kStepBlock), 0, s, job);
    }
    hipLaunchKernelGGL(k_step_norm, dim3(1), dim3(kCheckThreads), 0, s, job, nblocks);
    return hipGetLastError();
}

namespace {
template <int G, int WK>
void step_spmv_w(const StepJob* job, int nblocks, int fp32, hipStream_t s) {
    if constexpr (WK == kWF32) {
        hipLaunchKernelGGL((k_step_spmv<G, double, WK>), dim3(nblocks), dim3(kStepBlock), 0, s, job);
    } else {
        if (fp32) hipLaunchKernelGGL((k_step_spmv<G, float, WK>), dim3(nblocks), dim3(kStepBlock), 0, s, job);
        else hipLaunchKernelGGL((k_step_spmv<G, double, WK>), dim3(nblocks), dim3(kStepBlock), 0, s, job);
    }
}
template <int G>
void step_spmv_g(const StepJob* job, int nblocks, int fp32, int wk, hipStream_t s) {
    if (wk == kWUnit) step_spmv_w<G, kWUnit>(job, nblocks, fp32, s);
    else if (wk == kWF32) step_spmv_w<G, kWF32>(job, nblocks, fp32, s);
    else if (wk == kWU8) step_spmv_w<G, kWU8>(job, nblocks, fp32, s);
    else if (wk == kWU16) step_spmv_w<G, kWU16>(job, nblocks, fp32, s);
    else step_spmv_w<G, kWNative>(job, nblocks, fp32, s);
}
}  // namespace

hipError_t launch_step_pi(const StepJob* job, int nblocks, int kind, hipStream_t s) {
    const int fp32 = kind & 1, wk = kind >> 4;
    switch ((kind >> 1) & 7) {
        case 1: step_spmv_g<1>(job, nblocks, fp32, wk, s); break;
        case 2: step_spmv_g<2>(job, nblocks, fp32, wk, s); break;
        case 3: step_spmv_g<4>(job, nblocks, fp32, wk, s); break;
        case 4: step_spmv_g<8>(job, nblocks, fp32, wk, s); break;
        case 5: step_spmv_g<16>(job, nblocks, fp32, wk, s); break;
        case 6: step_spmv_g<32>(job, nblocks, fp32, wk, s); break;
        case 7: step_spmv_g<64>(job, nblocks, fp32, wk, s); break;
        default: return hipErrorInvalidValue;  // the merge path has no step form
    }
    hipLaunchKernelGGL(k_step_check, dim3(1), dim3(kCheckThreads), 0, s, job, nblocks);
    return hipGetLastError();
}

hipError_t launch_reset_sync(GridSync* gs, GridSlot* slots, int nslots, GridSlot* bcast, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_sync, dim3(1), dim3(256), 0, s, gs, slots, nslots, bcast);
    return hipGetLastError();
}

hipError_t launch_raise_abort(GridSync* gs, hipStream_t s) {
    hipLaunchKernelGGL(k_raise_abort, dim3(1), dim3(64), 0, s, gs);
    return hipGetLastError();
}

}  // namespace cmg
