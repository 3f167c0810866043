// Several eigenpairs at once (the Remark after Algorithm 4: start from p
// approximate eigenpairs of the coarsest level, smooth every vector on each
// level, orthogonalise them and take Rayleigh quotients).
//
// A level keeps an n x P row-major block W plus a column mean mu and an
// upper-triangular R^{-1}; the current orthonormal block is
// V = (W - 1 mu^T) R^{-1}.  One step computes, row by row,
//   Z_i = ( g (W_i - mu) + sum_k a_ik (W_k - W_i) ) R^{-1}  (= (B_g V)_i,
// since L 1 = 0) and, in the same pass, the FP64 sums 1^T Z, Z^T Z and
// Z^T V.  From them the next mean, the Gram matrix of the deflated Z, its
// Cholesky factor R' (Cholesky QR: the same orthonormal block as
// Gram-Schmidt in column order, exactly so in exact arithmetic) and the
// stopping quantities (u_c, v_c) = (R'^{-T} Z^T V)_cc (V is deflated, so
// Z needs no mean there).  All sums have a fixed order, so results are
// reproducible bitwise.  Small levels run inside one workgroup, larger ones
// one launch per step plus a one-workgroup check.
#include "cmg_internal.h"

namespace cmg {

namespace {

constexpr int kBlkThreads = 256;
constexpr int kBlkCheck = 1024;

// v = (w - mu) R^{-1} for one row (R^{-1} upper triangular, row-major)
template <int P>
__device__ __forceinline__ void to_v(const double* __restrict__ w, const double* mu, const double* rinv,
                                     double (&v)[P]) {
    double d[P];
#pragma unroll
    for (int r = 0; r < P; ++r) d[r] = w[r] - mu[r];
#pragma unroll
    for (int c = 0; c < P; ++c) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r <= c; ++r) s += d[r] * rinv[r * P + c];
        v[c] = s;
    }
}

// Totals of the per-workgroup partial sums, in workgroup order, in every thread.
template <int NV>
__device__ __forceinline__ void blk_totals(const double* part, int nb, double (&v)[NV], double* red) {
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] += part[(size_t)NV * b + q];
    }
    block_sum<NV>(v, red);
}

template <int NV>
__device__ __forceinline__ void blk_post(double (&v)[NV], double* red, double* part) {
    block_sum<NV>(v, red);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) part[(size_t)NV * blockIdx.x + q] = v[q];
    }
}

// ---- coarsest level: p vectors from the dense eigensolve
//
// E = the eigenvectors above the smallest eigenvalue whose eigenvalue is at
// most lambda_{P+1} + 1e-10 ||L||_F (whole clusters: independent of the
// eigensolver's basis).  Start c = U(seed ^ (c+1) 0xD1B54A32D192ED03, i) - 1/2
// is projected onto E; the P projections are orthonormalised in column order
// (mean removed, modified Gram-Schmidt, normalised).
template <int P>
__global__ void __launch_bounds__(kBlkThreads) k_blk_coarse(BlkJob J, const double* __restrict__ V,
                                                            const double* __restrict__ ev,
                                                            const int32_t* __restrict__ idx) {
    __shared__ double y[P][128];
    __shared__ double red[16 * 2 + 8];
    const int n = J.n;
    // ||L^J||_F from the coarsest CSR: degrees on the diagonal, weights off it
    double f[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        double d = 0.0, o = 0.0;
        for (int e = J.rp[i]; e < J.rp[i + 1]; ++e) {
            d += J.w[e];
            o += J.w[e] * J.w[e];
        }
        f[0] += d * d + o;
    }
    block_sum<1>(f, red);
    const double fro = sqrt(f[0]);
    const double top = ev[idx[P]];
    // projections: y_c = sum_{r in E} (q_r . z_c) q_r
    for (int c = 0; c < P; ++c) {
        const uint64_t sc = J.seed ^ ((uint64_t)(c + 1) * 0xD1B54A32D192ED03ull);
        for (int i = threadIdx.x; i < n; i += blockDim.x) y[c][i] = 0.0;
        __syncthreads();
        for (int r = 1; r < n; ++r) {
            const int k = idx[r];
            if (ev[k] > top + 1e-10 * fro) continue;
            double d[1] = {0.0};
            for (int i = threadIdx.x; i < n; i += blockDim.x) d[0] += V[i * n + k] * (hashed_uniform(sc, i) - 0.5);
            block_sum<1>(d, red);
            for (int i = threadIdx.x; i < n; i += blockDim.x) y[c][i] += d[0] * V[i * n + k];
            __syncthreads();
        }
    }
    // orthonormalise in column order
    for (int c = 0; c < P; ++c) {
        double m[1] = {0.0};
        for (int i = threadIdx.x; i < n; i += blockDim.x) m[0] += y[c][i];
        block_sum<1>(m, red);
        const double mean = m[0] / (double)n;
        for (int i = threadIdx.x; i < n; i += blockDim.x) y[c][i] -= mean;
        __syncthreads();
        for (int d = 0; d < c; ++d) {
            double t[1] = {0.0};
            for (int i = threadIdx.x; i < n; i += blockDim.x) t[0] += y[d][i] * y[c][i];
            block_sum<1>(t, red);
            for (int i = threadIdx.x; i < n; i += blockDim.x) y[c][i] -= t[0] * y[d][i];
            __syncthreads();
        }
        double q[1] = {0.0};
        for (int i = threadIdx.x; i < n; i += blockDim.x) q[0] += y[c][i] * y[c][i];
        block_sum<1>(q, red);
        const double nr = sqrt(q[0]);
        for (int i = threadIdx.x; i < n; i += blockDim.x) y[c][i] /= nr;
        __syncthreads();
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        for (int c = 0; c < P; ++c) J.W0[(size_t)i * P + c] = y[c][i];
    if (threadIdx.x == 0) {
        BlkCtl s{};
        for (int r = 0; r < P * P; ++r) s.rinv[r] = (r / P == r % P) ? 1.0 : 0.0;
        s.k = -1;
        s.cur = 0;
        s.done = 1;
        *J.ctl = s;
        for (int c = 0; c < P; ++c) J.out->coarse[c] = ev[idx[c + 1]];
    }
}

// ------------------------------------------------ rows, sums and factors of a step
//
// A row is spread over Q lanes, one per column: each lane sums its column's
// entries, takes the other columns' values from its neighbours, and adds up
// 2 Q + 1 products (1^T Z, Z^T Z and Z^T V, all that the test reads; 1^T V
// is zero to rounding), which are folded across the wavefront by halves.
template <int P>
struct BlkSums {
    static constexpr int Q = P == 1 ? 1 : P == 2 ? 2 : 4;  // lanes per row
    static constexpr int kSums = 2 * Q * Q + Q;            // by column: Z^T Z, Z^T V; then 1^T Z
    static constexpr int kSlot = (kSums + 3) & ~3;
    static constexpr int kLeft = Q == 4 ? 2 : 1;           // a lane's sums after two folds
};

// lane r's value in every lane of an aligned group of Q
template <int Q, int R>
__device__ __forceinline__ double blk_lane(double v) {
    if constexpr (Q == 1) return v;
    else if constexpr (Q == 2) return dpp_move<R == 0 ? 0xA0 : 0xF5>(v);
    else return dpp_move<R * 0x55>(v);
}
template <int Q>
__device__ __forceinline__ void blk_lanes(double v, double (&out)[Q]) {
    out[0] = blk_lane<Q, 0>(v);
    if constexpr (Q >= 2) out[1] = blk_lane<Q, 1>(v);
    if constexpr (Q == 4) {
        out[2] = blk_lane<Q, 2>(v);
        out[3] = blk_lane<Q, 3>(v);
    }
}

// Sum over the lanes l and l ^ ROWS: of a where bit ROWS of l is clear, of b
// where it is set.
template <int ROWS>
__device__ __forceinline__ double blk_fold(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const unsigned xl = (unsigned)(x & 0xffffffffll), xh = (unsigned)(x >> 32);
    const unsigned yl = (unsigned)(y & 0xffffffffll), yh = (unsigned)(y >> 32);
    if constexpr (ROWS == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
        return __longlong_as_double(((long long)h[0] << 32) | (long long)l[0]) +
               __longlong_as_double(((long long)h[1] << 32) | (long long)l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
        return __longlong_as_double(((long long)h[0] << 32) | (long long)l[0]) +
               __longlong_as_double(((long long)h[1] << 32) | (long long)l[1]);
    }
}

// sum over the groups of Q lanes within 16 lanes
template <int Q>
__device__ __forceinline__ double blk_row16(double v) {
    if constexpr (Q == 1) v += dpp_move<0xB1>(v);
    if constexpr (Q <= 2) v += dpp_move<0x4E>(v);
    v += dpp_move<0x124>(v);
    v += dpp_move<0x128>(v);
    return v;
}

__device__ __forceinline__ void blk_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront's sums of every lane's column, v = {Z^T Z, Z^T V} and
// cs = 1^T Z, to its slot.
template <int P>
__device__ __forceinline__ void blk_post_wave(double (&v)[2 * BlkSums<P>::Q], double cs, double* slot) {
    using B = BlkSums<P>;
    constexpr int Q = B::Q;
    const int lane = threadIdx.x & 63;
    double f[Q], h[B::kLeft];
#pragma unroll
    for (int q = 0; q < Q; ++q) f[q] = blk_fold<32>(v[q], v[q + Q]);
    if constexpr (Q == 1) h[0] = pair_sum_rows<16>(f[0]);
    else {
#pragma unroll
        for (int q = 0; q < Q / 2; ++q) h[q] = blk_fold<16>(f[q], f[q + Q / 2]);
    }
#pragma unroll
    for (int q = 0; q < B::kLeft; ++q) h[q] = blk_row16<Q>(h[q]);
    cs = blk_row16<Q>(pair_sum_rows<32>(pair_sum_rows<16>(cs)));
    const int c = lane & (Q - 1);
    if ((lane & 15) < Q) {
        double* at = slot + c * 2 * Q + (lane >= 32 ? Q : 0) + ((lane & 16) ? Q / 2 : 0);
#pragma unroll
        for (int q = 0; q < B::kLeft; ++q) sst(at, q, h[q]);
        if (lane < Q) sst(slot, 2 * Q * Q + c, cs);
    }
}

// From the totals: mu = 1^T Z / n, the Cholesky factor R of the Gram matrix
// of Z - 1 mu^T, and this lane's column of R^{-1} in rc (zero below the
// diagonal and in lanes without a column).  Reciprocal square roots in place
// of square roots and divisions.  False if the matrix is not positive
// definite.
template <int P>
__device__ __forceinline__ bool blk_chol(const double* tot, double n, double inv_n, double (&mu)[P],
                                               double (&rc)[BlkSums<P>::Q]) {
    constexpr int Q = BlkSums<P>::Q;
    const int c = threadIdx.x & (Q - 1);
    double R[P][P], id[P];
    bool ok = true;
#pragma unroll
    for (int r = 0; r < P; ++r) mu[r] = sld(tot, 2 * Q * Q + r) * inv_n;
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r <= j; ++r) R[r][j] = sld(tot, j * 2 * Q + r) - n * mu[r] * mu[j];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double s = R[k][k];
#pragma unroll
        for (int r = 0; r < k; ++r) s -= R[r][k] * R[r][k];
        ok = ok && s > 0.0;
        id[k] = fast_rsq(s);
#pragma unroll
        for (int j = k + 1; j < P; ++j) {
            double u = R[k][j];
#pragma unroll
            for (int r = 0; r < k; ++r) u -= R[r][k] * R[r][j];
            R[k][j] = u * id[k];
        }
    }
#pragma unroll
    for (int r = P; r < Q; ++r) rc[r] = 0.0;
#pragma unroll
    for (int r = P - 1; r >= 0; --r) {
        double s = r == c ? 1.0 : 0.0;
#pragma unroll
        for (int k = r + 1; k < P; ++k) s -= R[r][k] * rc[k];
        rc[r] = s * id[r];
    }
    return ok;
}

// The least (u_c, v_c) = (R^{-T} Z^T V)_cc over the columns.
template <int P>
__device__ __forceinline__ double blk_least(const double* tot, const double (&rc)[BlkSums<P>::Q]) {
    constexpr int Q = BlkSums<P>::Q;
    const int c = threadIdx.x & (Q - 1), cc = c < P ? c : P - 1;
    double uv = 0.0, ur[Q];
#pragma unroll
    for (int r = 0; r < P; ++r) uv += rc[r] * sld(tot, cc * 2 * Q + Q + r);
    blk_lanes<Q>(uv, ur);
    double least = 2.0;
#pragma unroll
    for (int r = 0; r < P; ++r) least = ur[r] < least ? ur[r] : least;
    return least;
}

// One lane's column of a row with the entries' sum t: z and v of the step,
// and their products with the row's other columns.
template <int P>
__device__ __forceinline__ double blk_row(double g, double wi, double muc, double t, const double (&rc)[BlkSums<P>::Q],
                                          bool on, double (&acc)[2 * BlkSums<P>::Q], double& cs) {
    constexpr int Q = BlkSums<P>::Q;
    const double d = wi - muc;
    const double y = g * d + t;
    double yr[Q], dr[Q], zr[Q], z = 0.0, v = 0.0;
    blk_lanes<Q>(y, yr);
    blk_lanes<Q>(d, dr);
#pragma unroll
    for (int r = 0; r < P; ++r) {
        z += yr[r] * rc[r];
        v += dr[r] * rc[r];
    }
    if (!on) z = v = 0.0;
    blk_lanes<Q>(z, zr);
    cs += z;
#pragma unroll
    for (int r = 0; r < P; ++r) {
        acc[r] += zr[r] * z;
        acc[Q + r] += zr[r] * v;
    }
    return z;
}

// One lane's column of a prolongated row (the coarse row cw through the
// coarse level's mean cmu and column crc of R^{-1}), and its products.
template <int P>
__device__ __forceinline__ double blk_prolong_row(const double* cw, bool on, double cmu,
                                                  const double (&crc)[BlkSums<P>::Q],
                                                  double (&acc)[2 * BlkSums<P>::Q], double& cs) {
    constexpr int Q = BlkSums<P>::Q;
    const int c = threadIdx.x & (Q - 1), cc = c < P ? c : P - 1;
    double d = 0.0;
    if (on) d = gld(cw, cc) - cmu;
    double dr[Q], zr[Q], z = 0.0;
    blk_lanes<Q>(d, dr);
#pragma unroll
    for (int r = 0; r < P; ++r) z += dr[r] * crc[r];
    blk_lanes<Q>(z, zr);
    cs += z;
#pragma unroll
    for (int r = 0; r < P; ++r) acc[r] += zr[r] * z;
    return z;
}

// This lane's column of a level's R^{-1} and mean.
template <int P>
__device__ __forceinline__ double blk_column(const BlkCtl* ct, double (&rc)[BlkSums<P>::Q]) {
    constexpr int Q = BlkSums<P>::Q;
    const int c = threadIdx.x & (Q - 1), cc = c < P ? c : P - 1;
#pragma unroll
    for (int r = 0; r < Q; ++r) rc[r] = r < P && c < P ? ct->rinv[(r < P ? r : 0) * P + cc] : 0.0;
    return ct->mu[cc];
}

// ---------------------------------------- larger levels, a launch per step

// Sums of one workgroup to its slot of the level's partial sums.
template <int P>
__device__ __forceinline__ void blk_post_group(double (&v)[2 * BlkSums<P>::Q], double cs, double* slots, double* part) {
    using B = BlkSums<P>;
    blk_post_wave<P>(v, cs, slots + (threadIdx.x >> 6) * B::kSlot);
    __syncthreads();
    const int q = (int)threadIdx.x;
    if (q < B::kSums) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kBlkThreads / 64; ++w) t += sld(slots, w * B::kSlot + q);
        part[(size_t)blockIdx.x * B::kSlot + q] = t;
    }
}

// prolongation of the coarser level's block and the sums of the result
template <int P>
__global__ void __launch_bounds__(kBlkThreads) k_blk_prolong(const BlkJob* __restrict__ jp) {
    using B = BlkSums<P>;
    constexpr int Q = B::Q;
    __shared__ double slots[kBlkThreads / 64 * B::kSlot];
    const BlkJob J = *jp;
    const double* cw = J.cctl->cur ? J.cW1 : J.cW0;
    const int c = (int)threadIdx.x & (Q - 1);
    double crc[Q], acc[2 * Q], cs = 0.0;
    const double cmu = blk_column<P>(J.cctl, crc);
#pragma unroll
    for (int q = 0; q < 2 * Q; ++q) acc[q] = 0.0;
    const int r0 = J.rpart[blockIdx.x], r1 = J.rpart[blockIdx.x + 1];
    for (int i0 = r0; i0 < r1; i0 += kBlkThreads / Q) {
        const int i = i0 + (int)threadIdx.x / Q;
        const bool on = i < r1;
        const double z = blk_prolong_row<P>(cw + (on ? (int64_t)gld(J.agg, i) * P : 0), on, cmu, crc, acc, cs);
        if (on && c < P) gst(J.W0, (int64_t)i * P + c, z);
    }
    blk_post_group<P>(acc, cs, slots, J.part);
}

// One step of orthogonal iteration: W[cur] -> W[cur ^ 1], Q lanes per row.
// Bounded by latency up to some 100000 rows (a row's chain: offsets,
// columns, the block's rows); a whole row per thread with 34 sums took 15.5
// us, this 8.9 on average over levels of 2527 to 200000 vertices and four columns.
template <int P>
__global__ void __launch_bounds__(kBlkThreads) k_blk_step(const BlkJob* __restrict__ jp) {
    using B = BlkSums<P>;
    constexpr int Q = B::Q;
    __shared__ double slots[kBlkThreads / 64 * B::kSlot];
    const BlkJob J = *jp;
    if (J.ctl->done) return;
    const int cur = J.ctl->cur;
    const double* win = cur ? J.W1 : J.W0;
    double* wout = cur ? J.W0 : J.W1;
    const int c = (int)threadIdx.x & (Q - 1), cc = c < P ? c : P - 1;
    double rc[Q], acc[2 * Q], cs = 0.0;
    const double muc = blk_column<P>(J.ctl, rc);
#pragma unroll
    for (int q = 0; q < 2 * Q; ++q) acc[q] = 0.0;
    const int r0 = J.rpart[blockIdx.x], r1 = J.rpart[blockIdx.x + 1];
    for (int i0 = r0; i0 < r1; i0 += kBlkThreads / Q) {
        const int i = i0 + (int)threadIdx.x / Q;
        const bool on = i < r1;
        double wi = 0.0, t = 0.0;
        if (on) {
            wi = gld(win, (int64_t)i * P + cc);
            const int a = gld(J.rp, i), b = gld(J.rp, i + 1);
#pragma unroll 4
            for (int e = a; e < b; ++e) t += gld(J.w, e) * (gld(win, (int64_t)gld(J.col, e) * P + cc) - wi);
        }
        const double z = blk_row<P>(J.g, wi, muc, t, rc, on, acc, cs);
        if (on && c < P) gst(wout, (int64_t)i * P + c, z);
    }
    blk_post_group<P>(acc, cs, slots, J.part);
}

// Sums of a prolongation (FIRST) or a step over all workgroups, the new
// (mu, R^{-1}), the stopping test of every column.  One sum per lane and a
// 16th of the workgroups per wavefront, then one wavefront: a whole set of
// sums per thread and the factorisation on one thread took 11.4 us, this 3.5.
template <int P, bool FIRST>
__global__ void __launch_bounds__(kBlkCheck) k_blk_check(const BlkJob* __restrict__ jp) {
    using B = BlkSums<P>;
    constexpr int Q = B::Q, W = kBlkCheck / 64;
    __shared__ double slots[(W + 1) * B::kSlot];
    const BlkJob J = *jp;
    if (!FIRST && J.ctl->done) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane < B::kSums) {
        double t = 0.0;
#pragma unroll 8
        for (int b = wv; b < J.nb; b += W) t += gld(J.part, (int64_t)b * B::kSlot + lane);
        sst(slots, wv * B::kSlot + lane, t);
    }
    __syncthreads();
    if (wv > 0) return;
    double* tot = slots + W * B::kSlot;
    if (lane < B::kSums) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) t += sld(slots, w * B::kSlot + lane);
        sst(tot, lane, t);
    }
    blk_wave_sync();
    double mu[P], rc[Q];
    const bool ok = blk_chol<P>(tot, (double)J.n, 1.0 / (double)J.n, mu, rc);
    const double minu = FIRST ? 0.0 : blk_least<P>(tot, rc);
    BlkCtl* s = J.ctl;
    const int k = FIRST ? 0 : s->k + 1, cur = FIRST ? 0 : s->cur ^ 1;
    int done = 0, hit = 0;
    if (!ok) {
        done = 1;
        hit = 2;
    } else if (FIRST) {
    } else if (J.kfix > 0) {
        done = k >= J.kfix;
    } else if (!(minu < 1.0 - J.tol)) {
        done = 1;
    } else if (k >= J.maxit) {
        done = 1;
        hit = 1;
    }
    if (lane < P) {
        s->mu[lane] = sld(tot, 2 * Q * Q + lane) * (1.0 / (double)J.n);
#pragma unroll
        for (int r = 0; r < P; ++r) s->rinv[r * P + lane] = rc[r];
    }
    if (lane == 0) {
        s->minutv = minu;
        s->k = k;
        s->cur = cur;
        s->done = done;
        s->hit = hit;
    }
}

// ------------------------------------------------- small levels, one workgroup
//
// A step of a small level is a few microseconds of work between two
// launches.  Levels of at most kBlkSmallN vertices therefore run all their
// steps, level after level, inside one workgroup, with both blocks in LDS
// and one barrier a step (none while one wavefront holds the level).  What
// bounds a step there is the chain of its instructions; every wavefront adds
// the posts of all and factors the Gram matrix itself, and 512 threads, as
// more would only repeat that on the same SIMDs.  Steps of 42, 115, 310 and
// 891 vertices with four columns take 1.3, 1.7, 2.9 and 7.9 us (23 us with
// two launches per step).  Past 1024 vertices the launches' share falls, and
// those levels take few steps, so they keep them.
constexpr int kBlkSmallThreads = 512;
constexpr int kBlkRegRows = 4, kBlkRegSlots = 8;  // rows per lane and entries per row kept in registers

// Totals over the workgroup's nw wavefronts: the address of the kSums
// totals.  part: 2 x 8 slots by parity, then a slot per wavefront.
template <int P>
__device__ __forceinline__ const double* blk_small_sums(double (&v)[2 * BlkSums<P>::Q], double cs, double* part,
                                                        int& parity, int nw) {
    using B = BlkSums<P>;
    constexpr int S = B::kSlot, W = kBlkSmallThreads / 64;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double* slot = part + parity * W * S;
    parity ^= 1;
    if (wv < nw) blk_post_wave<P>(v, cs, slot + wv * S);
    if (nw == 1) {
        blk_wave_sync();
        return slot;
    }
    __syncthreads();
    double* own = part + (2 * W + wv) * S;
    if (lane < B::kSums) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const double x = sld(slot, w * S + lane);
            t += w < nw ? x : 0.0;
        }
        sst(own, lane, t);
    }
    blk_wave_sync();
    return own;
}

// LDS: both blocks, then weights, and columns if they fit
constexpr size_t blk_small_fixed(int p, int n) { return 16 * (size_t)p * (size_t)n; }
__device__ inline size_t blk_small_csr(int nnz) { return 8 * (size_t)nnz + 2 * (((size_t)nnz + 3) & ~(size_t)3); }

// Levels jhi down to jlo of a hierarchy (jobs[j], each of at most kBlkSmallN
// vertices).  The last block of a level is left in its W0.
template <int P>
__global__ void __launch_bounds__(kBlkSmallThreads) k_blk_small(const BlkJob* __restrict__ jobs, int jhi, int jlo,
                                                                int lds_bytes) {
    using B = BlkSums<P>;
    constexpr int Q = B::Q, E = kBlkRegSlots;
    extern __shared__ double lds[];
    __shared__ double part[3 * (kBlkSmallThreads / 64) * B::kSlot];
    const int tid = (int)threadIdx.x, wv = tid >> 6;
    const int c = tid & (Q - 1), cc = c < P ? c : P - 1;
    const int nrow = kBlkSmallThreads / Q, row0 = tid / Q;  // rows per pass, this lane's first
    for (int j = jhi; j >= jlo; --j) {
        const BlkJob J = jobs[j];
        int parity = 0;  // (a level of one wavefront flips it there alone)
        const int n = J.n;
        const int passes = (n + nrow - 1) / nrow;
        const int nw = min(kBlkSmallThreads / 64, (n * Q + 63) / 64);
        const double dn = (double)n, inv_n = 1.0 / dn, g = J.g;
        const int nnz = gld(J.rp, n);
        double* w0 = lds;
        double* w1 = lds + (size_t)P * n;
        double* sw = w1 + (size_t)P * n;
        uint16_t* sc = (uint16_t*)(sw + nnz);
        const bool staged = blk_small_fixed(P, n) + blk_small_csr(nnz) <= (size_t)lds_bytes;
        const bool regs = passes <= kBlkRegRows;
        __syncthreads();  // the level before has been written out
        if (staged)
            for (int e = tid; e < nnz; e += kBlkSmallThreads) {
                sst(sw, e, gld(J.w, e));
                sst(sc, e, (uint16_t)gld(J.col, e));
            }
        // the first entries of a lane's rows; past the row's end its own
        // vertex with weight 0 (an exact zero)
        int ra[kBlkRegRows], rb[kBlkRegRows], rm[kBlkRegRows];
        uint32_t rcol[kBlkRegRows][E / 2];
        double rw[kBlkRegRows][E];
#pragma unroll
        for (int t = 0; t < kBlkRegRows; ++t) {
            const int i = row0 + t * nrow;
            const bool on = regs && i < n;
            ra[t] = on ? gld(J.rp, i) : 0;
            rb[t] = on ? gld(J.rp, i + 1) : 0;
            int most = min(rb[t] - ra[t], E);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, kWave));
            rm[t] = __builtin_amdgcn_readfirstlane(most);
#pragma unroll
            for (int m = 0; m < E; ++m) {
                uint32_t cv = on ? (uint32_t)i : 0u;
                double wt = 0.0;
                if (ra[t] + m < rb[t]) {
                    cv = (uint32_t)gld(J.col, ra[t] + m);
                    wt = gld(J.w, ra[t] + m);
                }
                if (m & 1) rcol[t][m >> 1] |= cv << 16;
                else rcol[t][m >> 1] = cv;
                rw[t][m] = wt;
            }
        }
        // prolongation
        double acc[2 * Q], cs = 0.0;
#pragma unroll
        for (int q = 0; q < 2 * Q; ++q) acc[q] = 0.0;
        {
            const BlkCtl* ct = J.cctl;
            const double* cw = ct->cur ? J.cW1 : J.cW0;
            double crc[Q];
            const double cmu = blk_column<P>(ct, crc);
            for (int t = 0; t < passes; ++t) {
                const int i = row0 + t * nrow;
                const bool on = i < n;
                const double z =
                    blk_prolong_row<P>(cw + (on ? (int64_t)gld(J.agg, i) * P : 0), on, cmu, crc, acc, cs);
                if (on && c < P) sst(w0, i * P + c, z);
            }
        }
        __syncthreads();
        if (nw > 1 || wv == 0) {
            const double* tot = blk_small_sums<P>(acc, cs, part, parity, nw);
            double mu[P], rc[Q];
            int k = 0, hit = blk_chol<P>(tot, dn, inv_n, mu, rc) ? 0 : 2, cur = 0;
            double minu = 0.0;
            while (hit == 0) {
                const double* win = cur ? w1 : w0;
                double* wout = cur ? w0 : w1;
                cs = 0.0;
#pragma unroll
                for (int q = 0; q < 2 * Q; ++q) acc[q] = 0.0;
                double muc = mu[0];
#pragma unroll
                for (int r = 1; r < P; ++r) muc = r == cc ? mu[r] : muc;
                auto finish = [&](int i, double wi, double t) {
                    const bool on = i < n;
                    const double z = blk_row<P>(g, wi, muc, t, rc, on, acc, cs);
                    if (on && c < P) sst(wout, i * P + c, z);
                };
                auto rest = [&](int a, int b, double wi, double t) {
                    if (staged) {
#pragma unroll 4
                        for (int e = a; e < b; ++e) t += sld(sw, e) * (sld(win, (int)sld(sc, e) * P + cc) - wi);
                    } else {
#pragma unroll 4
                        for (int e = a; e < b; ++e) t += gld(J.w, e) * (sld(win, gld(J.col, e) * P + cc) - wi);
                    }
                    return t;
                };
                if (wv < nw) {
                    if (regs) {
#pragma unroll
                        for (int r = 0; r < kBlkRegRows; ++r) {
                            if (r < passes) {
                                const int i = row0 + r * nrow;
                                // decode the columns every step: hoisted out
                                // of the step loop they would not fit
#pragma unroll
                                for (int m = 0; m < E / 2; ++m) asm volatile("" : "+v"(rcol[r][m]));
                                const double wi = sld(win, (i < n ? i : 0) * P + cc);
                                double x[E], t = 0.0;
                                auto at = [&](int m) {
                                    return (int)((m & 1) ? (rcol[r][m >> 1] >> 16) : (rcol[r][m >> 1] & 0xffffu)) * P + cc;
                                };
#pragma unroll
                                for (int m = 0; m < E / 2; ++m) x[m] = sld(win, at(m));
                                if (rm[r] > E / 2) {
#pragma unroll
                                    for (int m = E / 2; m < E; ++m) x[m] = sld(win, at(m));
#pragma unroll
                                    for (int m = 0; m < E; ++m) t += rw[r][m] * (x[m] - wi);
                                } else {
#pragma unroll
                                    for (int m = 0; m < E / 2; ++m) t += rw[r][m] * (x[m] - wi);
                                }
                                finish(i, wi, rest(ra[r] + E, rb[r], wi, t));
                            }
                        }
                    } else {
                        for (int r = 0; r < passes; ++r) {
                            const int i = row0 + r * nrow;
                            int a = 0, b = 0;
                            if (i < n) {
                                a = gld(J.rp, i);
                                b = gld(J.rp, i + 1);
                            }
                            const double wi = sld(win, (i < n ? i : 0) * P + cc);
                            finish(i, wi, rest(a, b, wi, 0.0));
                        }
                    }
                }
                tot = blk_small_sums<P>(acc, cs, part, parity, nw);
                const bool ok = blk_chol<P>(tot, dn, inv_n, mu, rc);
                minu = blk_least<P>(tot, rc);
                ++k;
                cur ^= 1;
                if (!ok) hit = 2;
                else if (J.kfix > 0) {
                    if (k >= J.kfix) break;
                } else if (!(minu < 1.0 - J.tol)) break;
                else if (k >= J.maxit) hit = 1;
            }
            const double* w = cur ? w1 : w0;
            const int step = nw > 1 ? kBlkSmallThreads : 64;
            for (int q = tid; q < n * P; q += step) gst(J.W0, q, sld(w, q));
            BlkCtl* out = J.ctl;
            if (tid < P) {
                out->mu[c] = sld(tot, 2 * Q * Q + c) * inv_n;
#pragma unroll
                for (int r = 0; r < P; ++r) out->rinv[r * P + c] = rc[r];
            }
            if (tid == 0) {
                out->minutv = minu;
                out->k = k;
                out->cur = 0;
                out->done = 1;
                out->hit = hit;
            }
        }
        __syncthreads();
    }
}

// ---- level 0: the output block (column-major) and the edge-form Rayleigh
// quotient numerators and norms of every column
template <int P>
__global__ void __launch_bounds__(kBlkThreads) k_blk_out(const BlkJob* __restrict__ jp, double* __restrict__ X) {
    __shared__ double red[16 * 2 * P + 2 * P + 8];
    const BlkJob J = *jp;
    const BlkCtl c = *J.ctl;
    const double* W = c.cur ? J.W1 : J.W0;
    const int r0 = J.rpart[blockIdx.x], r1 = J.rpart[blockIdx.x + 1];
    double acc[2 * P];
#pragma unroll
    for (int q = 0; q < 2 * P; ++q) acc[q] = 0.0;
    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
        double vi[P];
        to_v<P>(W + (size_t)i * P, c.mu, c.rinv, vi);
        for (int e = J.rp[i]; e < J.rp[i + 1]; ++e) {
            double vk[P];
            to_v<P>(W + (size_t)J.col[e] * P, c.mu, c.rinv, vk);
#pragma unroll
            for (int r = 0; r < P; ++r) {
                const double d = vi[r] - vk[r];
                acc[r] += 0.5 * J.w[e] * d * d;
            }
        }
#pragma unroll
        for (int r = 0; r < P; ++r) {
            X[(size_t)r * J.n + i] = vi[r];
            acc[P + r] += vi[r] * vi[r];
        }
    }
    blk_post<2 * P>(acc, red, J.part);
}

template <int P>
__global__ void __launch_bounds__(kBlkCheck) k_blk_rq(const BlkJob* __restrict__ jp) {
    __shared__ double red[16 * 2 * P + 2 * P + 8];
    const BlkJob J = *jp;
    double v[2 * P];
    blk_totals<2 * P>(J.part, J.nb, v, red);
    if (threadIdx.x == 0)
        for (int r = 0; r < P; ++r) {
            J.out->lambda[r] = v[r] / v[P + r];
            J.out->norm2[r] = v[P + r];
        }
}

// residual terms ((L x)_i - lambda x_i)^2 of every column
template <int P>
__global__ void __launch_bounds__(kBlkThreads) k_blk_res(const BlkJob* __restrict__ jp, const double* __restrict__ X) {
    __shared__ double red[16 * P + P + 8];
    const BlkJob J = *jp;
    double lam[P];
#pragma unroll
    for (int r = 0; r < P; ++r) lam[r] = J.out->lambda[r];
    const int r0 = J.rpart[blockIdx.x], r1 = J.rpart[blockIdx.x + 1];
    double acc[P];
#pragma unroll
    for (int r = 0; r < P; ++r) acc[r] = 0.0;
    for (int i = r0 + threadIdx.x; i < r1; i += blockDim.x) {
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const double* x = X + (size_t)r * J.n;
            const double xi = x[i];
            double t = 0.0;
            for (int e = J.rp[i]; e < J.rp[i + 1]; ++e) t += J.w[e] * (xi - x[J.col[e]]);
            const double d = t - lam[r] * xi;
            acc[r] += d * d;
        }
    }
    blk_post<P>(acc, red, J.part);
}

template <int P>
__global__ void __launch_bounds__(kBlkCheck) k_blk_fin(const BlkJob* __restrict__ jp) {
    __shared__ double red[16 * P + P + 8];
    const BlkJob J = *jp;
    double v[P];
    blk_totals<P>(J.part, J.nb, v, red);
    if (threadIdx.x == 0)
        for (int r = 0; r < P; ++r) J.out->residual[r] = sqrt(v[r] / J.out->norm2[r]);
}

template <int P>
hipError_t blk_launch(int what, const BlkJob* dj, const BlkJob& hj, double* X, const double* V, const double* ev,
                      const int32_t* idx, hipStream_t s) {
    const dim3 g(hj.nb), b(kBlkThreads), one(1), chk(kBlkCheck);
    switch (what) {
        case kBlkCoarse: hipLaunchKernelGGL(k_blk_coarse<P>, one, b, 0, s, hj, V, ev, idx); break;
        case kBlkProlong:
            hipLaunchKernelGGL(k_blk_prolong<P>, g, b, 0, s, dj);
            hipLaunchKernelGGL((k_blk_check<P, true>), one, chk, 0, s, dj);
            break;
        case kBlkStep:
            hipLaunchKernelGGL(k_blk_step<P>, g, b, 0, s, dj);
            hipLaunchKernelGGL((k_blk_check<P, false>), one, chk, 0, s, dj);
            break;
        case kBlkOut:
            hipLaunchKernelGGL(k_blk_out<P>, g, b, 0, s, dj, X);
            hipLaunchKernelGGL(k_blk_rq<P>, one, chk, 0, s, dj);
            hipLaunchKernelGGL(k_blk_res<P>, g, b, 0, s, dj, (const double*)X);
            hipLaunchKernelGGL(k_blk_fin<P>, one, chk, 0, s, dj);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int P>
int blk_small_lds() {
    static const int bytes = [] {
        int dev = 0, maxsh = 65536;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&maxsh, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, (const void*)k_blk_small<P>) != hipSuccess) return 0;
        const int b = (maxsh - (int)fa.sharedSizeBytes - 256) & ~255;
        if (hipFuncSetAttribute((const void*)k_blk_small<P>, hipFuncAttributeMaxDynamicSharedMemorySize, b) !=
            hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        return b;
    }();
    return bytes;
}

template <int P>
hipError_t blk_small_launch(const BlkJob* dj, int jhi, int jlo, hipStream_t s) {
    const int b = blk_small_lds<P>();
    hipLaunchKernelGGL(k_blk_small<P>, dim3(1), dim3(kBlkSmallThreads), b, s, dj, jhi, jlo, b);
    return hipGetLastError();
}

}  // namespace

bool blk_small_level(int p, int n) {
    const int b = p == 1 ? blk_small_lds<1>() : p == 2 ? blk_small_lds<2>() : p == 3 ? blk_small_lds<3>() : blk_small_lds<4>();
    return n <= kBlkSmallN && blk_small_fixed(p, n) <= (size_t)b;
}

hipError_t launch_blk_small(int p, const BlkJob* dj, int jhi, int jlo, hipStream_t s) {
    switch (p) {
        case 1: return blk_small_launch<1>(dj, jhi, jlo, s);
        case 2: return blk_small_launch<2>(dj, jhi, jlo, s);
        case 3: return blk_small_launch<3>(dj, jhi, jlo, s);
        case 4: return blk_small_launch<4>(dj, jhi, jlo, s);
        default: return hipErrorInvalidValue;
    }
}

int blk_parts(int p) {
    return p == 1 ? BlkSums<1>::kSlot : p == 2 ? BlkSums<2>::kSlot : BlkSums<4>::kSlot;
}

hipError_t launch_blk(int what, int p, const BlkJob* dj, const BlkJob& hj, double* X, const double* V,
                      const double* ev, const int32_t* idx, hipStream_t s) {
    switch (p) {
        case 1: return blk_launch<1>(what, dj, hj, X, V, ev, idx, s);
        case 2: return blk_launch<2>(what, dj, hj, X, V, ev, idx, s);
        case 3: return blk_launch<3>(what, dj, hj, X, V, ev, idx, s);
        case 4: return blk_launch<4>(what, dj, hj, X, V, ev, idx, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cmg
