// Device bodies of the Davidson kernels, shared by the single-space launches
// and the batched launches (davidson.hip).  Grid bodies take their block index
// and block count within their space (bid, nblk); finishing bodies run in one
// block per space.
#pragma once

#include <cmath>
#include <type_traits>

#include "small_eig.h"
#include "sqd_internal.h"

namespace dav {


constexpr int MM = SQD_MMAX;
constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxBlocks = 512;   // measured on MI355X: 512 beats 1024 and 2048 by 1-3% (fewer partials to reduce)
constexpr int kPstride = MM + 4;   // partial sums per block
constexpr int kStallWindow = 12;   // FP32 phase: iterations without a 10% better residual
constexpr double kStallFrom = 1e-4;  // ... counted once the residual is below this times |theta|
constexpr double kFloor32 = 2e-6;    // 30 FP32 unit roundoffs: FP32 products carry no more digits

enum { DONE_RUNNING = 0, DONE_CONVERGED = 1, DONE_STALLED = 2, DONE_CAP = 3, DONE_SWITCH = 4 };

// Calls f(std::integral_constant<int, NR>) with NR the smallest multiple of 4
// (at most MT) not below cnt.  Loops over the rows of the basis then run to a
// compile-time bound with every load issued before the first use; rows past
// cnt are read from row cnt - 1 (always valid) and weighted by zero.  A
// per-row branch instead makes each load wait for the one before it.
template <int MT, int NR = 4, typename F>
__device__ __forceinline__ void with_rows(int cnt, F&& f) {
    if constexpr (NR >= MT) {
        f(std::integral_constant<int, MT>{});
    } else {
        if (cnt <= NR) f(std::integral_constant<int, NR>{});
        else with_rows<MT, NR + 4>(cnt, f);
    }
}

// Row k of a block of vectors of length n, clamped to the last valid row
// (row 0 when the block is empty).  The vector kernels read basis rows with
// non-temporal loads: the basis (m rows of n) is larger than the caches, and
// what the next kernels reuse (the correction, c, the product's tables) then
// stays cached (4.0e6-determinant workload, same box: FP64 solve 0.227 ->
// 0.216 s, mixed 0.157 -> 0.150 s).
template <typename VT>
__device__ __forceinline__ const VT* row_ptr(const VT* B, int k, int cnt, int64_t n) {
    const int r = k < cnt ? k : cnt - 1;
    return B + (int64_t)(r > 0 ? r : 0) * n;
}

struct dav_state {
    int m;
    int done;
    int iter;
    int collapse;         // number of vectors kept by a pending collapse (0 = none)
    int phase;            // 0: FP32 sigma (mixed mode), 1: FP64 sigma
    int phase_start;      // iteration at which the current phase began
    int kmin;
    int nhist;
    int reortho;          // second Gram-Schmidt projection needed
    int best_it;          // iteration of the smallest residual of the current phase
    int counter[8];       // last-block tickets, one per kernel kind
    double theta;
    double rnorm;
    double tt0;           // |t|^2 before orthogonalisation
    double tinv;          // 1 / |v| of the new basis vector
    double G[MM * MM];
    double y[MM];
    double y_prev[MM];    // previous Ritz vector in the current basis
    double h[MM];
    double qc[2][MM];     // collapse coefficients (columns kept)
    double Gc[4];         // projected matrix after a collapse
    double hc[2];         // Gram-Schmidt coefficients after a collapse
    double hist_r[SQD_HIST];
    double hist_e[SQD_HIST];
    int xredo;            // locked-vector projection needs a second pass
    double best_r;        // smallest residual of the current phase
    double xc[SQD_MAXLOCK];   // X^T v of the vector being projected
    double xscale;        // scale applied after the projection (1 / |v - X xc|, or 1)
};

struct dav_params {
    double tol;
    double switch_tol;
    int max_iter;
    int m_max;
    int mixed;
};

// Sums of v[0..N) over the 64 lanes of a wavefront, by recursive halving: at
// each step a lane hands the half of its columns that its partner keeps to the
// partner and adds the other half's, so N - 1 + 6 - log2 N exchanges instead of 6 N
// (26 columns: 31 instead of 156).  The lane ends with the sum of column `col`
// (when there are fewer columns than lanes some end with none: col = -1).
template <int N, int MASK>
__device__ __forceinline__ double halve_sum(const double (&v)[N], int base, int size, int lane, int& col) {
    if constexpr (MASK == 0) {
        static_assert(N == 1, "more columns than lanes");
        col = size > 0 ? base : -1;
        return v[0];
    } else {
        constexpr int H = (N + 1) / 2;
        const bool up = (lane & MASK) != 0;
        double k[H];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const double lo = v[j], hi = j + H < N ? v[j + H] : 0.0;
            k[j] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, MASK);
        }
        // of `size` columns in use the lower lane keeps H, the upper the rest
        const int low = size < H ? size : H;
        return halve_sum<H, MASK / 2>(k, up ? base + H : base, up ? size - low : low, lane, col);
    }
}

// Block-wide sums of acc[0..NV) in wred (a slot per wave).
template <int NV>
__device__ __forceinline__ void wave_sums(const double (&acc)[NV], double (*wred)[NV]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int col;
    const double v = halve_sum<NV, 32>(acc, 0, NV, lane, col);
    if (col >= 0) wred[w][col] = v;   // lanes that share a column hold the same sum
}

// Block-wide sums of acc[0..NV); written to partial row `row`.
template <int NV>
__device__ void block_to_partial(const double (&acc)[NV], double* __restrict__ partial, int64_t row, int64_t nrows) {
    __shared__ double wred[kWaves][NV];
    wave_sums<NV>(acc, wred);
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int q = 0; q < kWaves; ++q) s += wred[q][threadIdx.x];
        partial[(size_t)threadIdx.x * nrows + row] = s;   // value-major: the reduction reads coalesced
    }
}

// One block of kThreads: out[j] = sum over rows b < nrows of partial[b][j],
// j < NV (thread t takes rows t, t + kThreads, ...; then a fixed tree), so the
// result is deterministic.  The partials come from an earlier launch.
template <int NV>
__device__ void reduce_rows(const double* __restrict__ partial, int nrows, double* out) {
    double acc[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = 0.0;
    for (int b = threadIdx.x; b < nrows; b += kThreads) {
#pragma unroll
        for (int j = 0; j < NV; ++j) acc[j] += partial[(size_t)j * nrows + b];
    }
    __shared__ double wred[kWaves][NV];
    wave_sums<NV>(acc, wred);
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int q = 0; q < kWaves; ++q) s += wred[q][threadIdx.x];
        out[threadIdx.x] = s;
    }
    __syncthreads();
}

// ---------------------------------------------------------------- kernels

// per-block (min value, first index) of the diagonal
__device__ __forceinline__ void d_argmin(const double* __restrict__ d, int64_t n,
                                                     double* __restrict__ partial, int64_t bid, int64_t nblk) {
    __shared__ double sv[kThreads];
    __shared__ long long si[kThreads];
    double best = INFINITY;
    long long bi = -1;
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
        const double v = d[i];
        if (v < best) { best = v; bi = i; }   // ascending i: first minimum kept
    }
    sv[threadIdx.x] = best;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double v = sv[threadIdx.x + s];
            const long long j = si[threadIdx.x + s];
            if (j >= 0 && (si[threadIdx.x] < 0 || v < sv[threadIdx.x] || (v == sv[threadIdx.x] && j < si[threadIdx.x]))) {
                sv[threadIdx.x] = v;
                si[threadIdx.x] = j;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[(size_t)bid * kPstride + 0] = sv[0];
        partial[(size_t)bid * kPstride + 1] = (double)si[0];
    }
}

// largest |x| (MODE 1, lowest index on ties) or smallest value (MODE 0) over
// the per-block partials -> st->kmin; MODE 1 also sums column 2 -> st->tinv = 1/sqrt.
template <int MODE>
__device__ __forceinline__ void f_pick_fin(const double* __restrict__ partial, int nrows, dav_state* st) {
    __shared__ double sv[kThreads], sn[kThreads];
    __shared__ long long si[kThreads];
    double b = MODE ? -1.0 : INFINITY, ss = 0.0;
    long long k = -1;
    for (int q = threadIdx.x; q < nrows; q += kThreads) {
        const double v = partial[(size_t)q * kPstride];
        const long long j = (long long)partial[(size_t)q * kPstride + 1];
        if (MODE) ss += partial[(size_t)q * kPstride + 2];
        const bool better = MODE ? (v > b) : (v < b);
        if (j >= 0 && (k < 0 || better || (v == b && j < k))) { b = v; k = j; }
    }
    sv[threadIdx.x] = b; si[threadIdx.x] = k; sn[threadIdx.x] = ss;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double v = sv[threadIdx.x + s];
            const long long j = si[threadIdx.x + s];
            const bool better = MODE ? (v > sv[threadIdx.x]) : (v < sv[threadIdx.x]);
            if (j >= 0 && (si[threadIdx.x] < 0 || better || (v == sv[threadIdx.x] && j < si[threadIdx.x]))) {
                sv[threadIdx.x] = v;
                si[threadIdx.x] = j;
            }
            sn[threadIdx.x] += sn[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        st->kmin = (int)(si[0] < 0 ? 0 : si[0]);
        if (MODE) st->tinv = 1.0 / sqrt(sn[0]);
    }
}

// V[0] = start vector (explicit guess, or e_kmin + noise), and |V[0]|^2 partials.
// SplitMix64 (Steele, Lea and Flood, OOPSLA 2014): a counter-based 64-bit mix.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// Entry i of the library's start noise for counter stream `stream`: uniform of
// zero mean and variance 1e-6 / n, so the noise has norm about 1e-3.  It lets a
// start on e_kmin, which has the spin-flip symmetry of an S_a = S_b space, reach
// a lowest state of the other symmetry.
__device__ __forceinline__ double start_noise(uint64_t stream, int64_t i, int64_t n) {
    const uint64_t r = splitmix64((stream << 40) ^ (uint64_t)i);
    const double uni = (double)(r >> 11) * (1.0 / 9007199254740992.0);   // [0, 1)
    return 1e-3 * sqrt(3.0 / (double)n) * (2.0 * uni - 1.0);
}

// V0 = guess, or e_kmin + noise (the caller's, else start_noise stream 0);
// |V0|^2 partials.
template <typename VT = double>
__device__ __forceinline__ void d_start(const double* __restrict__ guess, const double* __restrict__ noise,
                                                    int64_t n, const dav_state* st, VT* __restrict__ V0,
                                                    double* __restrict__ partial, int64_t bid, int64_t nblk) {
    double acc[1] = {0.0};
    const int64_t kmin = st->kmin;
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
        double v;
        if (guess) v = guess[i];
        else v = (i == kmin ? 1.0 : 0.0) + (noise ? noise[i] : start_noise(0, i, n));
        V0[i] = (VT)v;
        acc[0] += v * v;
    }
    block_to_partial<1>(acc, partial, bid, nblk);
}

__device__ __forceinline__ void f_norm_fin(const double* __restrict__ partial, int nrows, dav_state* st) {
    __shared__ double out[1];
    reduce_rows<1>(partial, nrows, out);
    if (threadIdx.x == 0) st->tinv = 1.0 / sqrt(out[0]);
}

// V0 *= tinv; copies into the product input (and its FP32 copy)
template <typename VT = double>
__device__ __forceinline__ void d_scale_copy(VT* __restrict__ V0, int64_t n, const dav_state* st,
                                                         double* __restrict__ cin, float* __restrict__ c32, int64_t bid, int64_t nblk) {
    const double sc = st->tinv;
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
        const double v = (double)V0[i] * sc;
        V0[i] = (VT)v;
        cin[i] = v;
        if (c32) c32[i] = (float)v;
    }
}

// Residual, preconditioned correction and the first Gram-Schmidt projection:
// partial columns 0..MT-1: V^T t; MT: |r|^2; MT+1: |t|^2.
template <int MT, typename VT = double>
__device__ __forceinline__ void d_residual(const VT* __restrict__ V, const VT* __restrict__ AV, const double* __restrict__ diag, int64_t n,
           const dav_state* st, double* __restrict__ T, double* __restrict__ partial, int64_t bid, int64_t nblk) {
    if (st->done) return;
    const int m = st->m;
    const double theta = st->theta;
    double acc[MT + 2];
#pragma unroll
    for (int k = 0; k < MT + 2; ++k) acc[k] = 0.0;
    with_rows<MT>(m, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        double y[NR];
        const VT* vr[NR];
        const VT* ar[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            y[k] = (k < m) ? st->y[k] : 0.0;
            vr[k] = row_ptr(V, k, m, n);
            ar[k] = row_ptr(AV, k, m, n);
        }
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double v[NR], a[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                v[k] = __builtin_nontemporal_load(vr[k] + i);
                a[k] = __builtin_nontemporal_load(ar[k] + i);
            }
            const double d = diag[i];
            double x = 0.0, ax = 0.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                x += y[k] * v[k];
                ax += y[k] * a[k];
            }
            const double r = ax - theta * x;
            double den = theta - d;
            if (fabs(den) < 1e-8) den = (den < 0.0) ? -1e-8 : 1e-8;
            const double tv = r / den;
            T[i] = tv;
            acc[MT] += r * r;
            acc[MT + 1] += tv * tv;
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[k] += (k < m) ? v[k] * tv : 0.0;
        }
    });
    block_to_partial<MT + 2>(acc, partial, bid, nblk);
}

// Convergence / cap / phase-switch decisions and the collapse plan.
template <int MT>
__device__ __forceinline__ void f_res_fin(const double* __restrict__ partial, int nrows, dav_state* st, dav_params prm) {
    // (the state's loads go out with the partials': one after another behind the
    // sums they took half of the kernel's time)
    const int over = st->done, m = st->m, it = st->iter, phase = st->phase, phase_start = st->phase_start;
    const int lane = threadIdx.x;
    const double theta = st->theta;
    double best_r = st->best_r;
    int best_it = st->best_it;
    const double yk = lane < MM ? st->y[lane] : 0.0, yp = lane < MM ? st->y_prev[lane] : 0.0;
    __shared__ double out[MT + 2];
    reduce_rows<MT + 2>(partial, nrows, out);
    if (over || lane >= 64) return;   // one wavefront
    if (lane < m) st->h[lane] = out[lane];
    const double rn = sqrt(out[MT]);
    int done = DONE_RUNNING;
    // smallest residual of this phase (a new best must improve by 10%)
    const bool best = it == phase_start || rn < 0.9 * best_r;
    if (best) {
        best_r = rn;
        best_it = it;
    }
    if (phase == 0) {
        // FP32 phase: hand over to FP64 refinement below switch_tol, on
        // reaching tol, below the FP32 floor (kFloor32 |theta|), or once the
        // residual has not improved for kStallWindow iterations after falling
        // below kStallFrom |theta| (a Davidson residual is not monotone: early
        // plateaus and bumps are not the FP32 floor)
        const double at = fabs(theta);
        const bool stall = best_r < kStallFrom * at && it - best_it >= kStallWindow;
        if (rn < prm.switch_tol || rn <= prm.tol || rn < kFloor32 * at || stall) done = DONE_SWITCH;
    } else if (rn <= prm.tol) {
        done = DONE_CONVERGED;
    }
    if (done == DONE_RUNNING && it + 1 >= prm.max_iter) done = DONE_CAP;
    int keep = 0;
    if (done == DONE_RUNNING && m >= prm.m_max) {
        // keep the Ritz vector and the previous Ritz vector, orthonormalised in
        // the small space: q1 = y, q2 ~ y_prev - (y . y_prev) y; a row of G and an
        // element of each vector per lane (one thread alone walked G four times)
        __shared__ double qs[2][MM];
        double q[2] = {lane < m ? yk : 0.0, lane < m ? yp : 0.0};
        q[1] -= sum32(q[0] * q[1]) * q[0];
        keep = 1;
        if (sum32(q[1] * q[1]) > 1e-20 && prm.m_max >= 3) {
            q[1] -= sum32(q[0] * q[1]) * q[0];
            q[1] *= 1.0 / sqrt(sum32(q[1] * q[1]));
            keep = 2;
        }
        double g[2] = {0.0, 0.0};
        if (lane < MM) {
            qs[0][lane] = st->qc[0][lane] = q[0];
            qs[1][lane] = st->qc[1][lane] = q[1];
        }
        __threadfence_block();
        for (int l = 0; l < m; ++l) {
            const double x = lane < m ? st->G[lane * MM + l] : 0.0;
            g[0] += x * qs[0][l];
            g[1] += x * qs[1][l];
        }
        const double o = lane < m ? out[lane] : 0.0;
        const double h0 = sum32(q[0] * o), h1 = sum32(q[1] * o);
        const double g00 = sum32(q[0] * g[0]), g11 = sum32(q[1] * g[1]);
        const double g01 = 0.5 * (sum32(q[0] * g[1]) + sum32(q[1] * g[0]));
        if (lane == 0) {
            st->hc[0] = h0;
            st->Gc[0] = g00;
            if (keep == 2) {
                st->hc[1] = h1;
                st->Gc[1] = st->Gc[2] = g01;
                st->Gc[3] = g11;
            }
        }
    }
    if (lane != 0) return;
    st->rnorm = rn;
    st->tt0 = out[MT + 1];
    if (it < SQD_HIST) {
        st->hist_r[it] = rn;
        st->hist_e[it] = theta;
        st->nhist = it + 1;
    }
    st->iter = it + 1;
    if (best) {
        st->best_r = best_r;
        st->best_it = best_it;
    }
    st->done = done;
    st->collapse = keep;
}

// x = V y into cin and, from an FP64 basis, V[0] (the FP64 refinement's first
// vector; an FP32 basis leaves V[0] to the caller, which it overlaps).
template <int MT, typename VT = double>
__device__ __forceinline__ void d_collapse(VT* __restrict__ V, int64_t n, const dav_state* st,
                                           double* __restrict__ cin, int64_t bid, int64_t nblk) {
    const int m = st->m;
    with_rows<MT>(m, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        double y[NR];
        const VT* vr[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            y[k] = (k < m) ? st->y[k] : 0.0;
            vr[k] = row_ptr(V, k, m, n);
        }
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double v[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(vr[k] + i);
            double x = 0.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) x += y[k] * v[k];
            if (sizeof(VT) == sizeof(double)) V[i] = (VT)x;
            cin[i] = x;
        }
    });
}

// State after it: m = 0, the next dots pass rebuilds G[0][0].
__device__ __forceinline__ void f_collapse_fin(dav_state* st) {
    if (threadIdx.x != 0) return;
    st->m = 0;
    st->collapse = 0;
}

// t1 = t - V h; partial columns 0..MT-1: V^T t1; MT: |t1|^2.  With a restart
// pending the basis is collapsed in place on the way: V[a] = V qc[a], AV[a] =
// AV qc[a] for the kept columns a (every row of an element is read before its
// row 0 or 1 is written, and elements are independent), and h is hc over those
// columns.
template <int MT, typename VT = double>
__device__ __forceinline__ void d_orth1(VT* __restrict__ V, VT* __restrict__ AV, int64_t n, const dav_state* st,
        double* __restrict__ T, double* __restrict__ partial, int64_t bid, int64_t nblk) {
    if (st->done) return;
    const int m = st->m;
    double acc[MT + 1];
#pragma unroll
    for (int k = 0; k < MT + 1; ++k) acc[k] = 0.0;
    if (st->collapse) {
        const bool two = st->collapse == 2;
        const double h0 = st->hc[0], h1 = two ? st->hc[1] : 0.0;
        with_rows<MT>(m, [&](auto nr_) {
            constexpr int NR = decltype(nr_)::value;
            double q1[NR], q2[NR];
            const VT* vr[NR];
            const VT* ar[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) {
                q1[k] = (k < m) ? st->qc[0][k] : 0.0;
                q2[k] = (k < m) ? st->qc[1][k] : 0.0;
                vr[k] = row_ptr(V, k, m, n);
                ar[k] = row_ptr(AV, k, m, n);
            }
            for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
                double v[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(vr[k] + i);
                double x1 = 0.0, x2 = 0.0;
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    x1 += q1[k] * v[k];
                    x2 += q2[k] * v[k];
                }
#pragma unroll
                for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(ar[k] + i);
                double a1 = 0.0, a2 = 0.0;
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    a1 += q1[k] * v[k];
                    a2 += q2[k] * v[k];
                }
                AV[i] = (VT)a1;
                V[i] = (VT)x1;
                if (two) {
                    AV[n + i] = (VT)a2;
                    V[n + i] = (VT)x2;
                }
                // the projection uses the rows as stored
                const double w1 = (double)(VT)x1, w2 = (double)(VT)x2;
                const double t = T[i] - h0 * w1 - h1 * w2;
                T[i] = t;
                acc[MT] += t * t;
                acc[0] += w1 * t;
                if (two) acc[1] += w2 * t;
            }
        });
        block_to_partial<MT + 1>(acc, partial, bid, nblk);
        return;
    }
    with_rows<MT>(m, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        double h[NR];
        const VT* vr[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            h[k] = (k < m) ? st->h[k] : 0.0;
            vr[k] = row_ptr((const VT*)V, k, m, n);
        }
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double v[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(vr[k] + i);
            double t = T[i];
#pragma unroll
            for (int k = 0; k < NR; ++k) t -= h[k] * v[k];
            T[i] = t;
            acc[MT] += t * t;
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[k] += (k < m) ? v[k] * t : 0.0;
        }
    });
    block_to_partial<MT + 1>(acc, partial, bid, nblk);
}

template <int MT, typename VT = double>
__device__ __forceinline__ void f_orth1_fin(const double* __restrict__ partial, int nrows, dav_state* st) {
    const int over = st->done, keep = st->collapse, m = keep ? keep : st->m;
    const double tt0 = st->tt0, rnorm = st->rnorm;
    __shared__ double out[MT + 1];
    reduce_rows<MT + 1>(partial, nrows, out);
    if (over) return;
    __syncthreads();   // every thread has read the state that changes below
    if (keep) {        // the basis was collapsed by the pass
        for (int k = threadIdx.x; k < MM * MM; k += kThreads) {
            const int i = k / MM, j = k % MM;
            st->G[k] = (i < keep && j < keep) ? st->Gc[i * 2 + j] : 0.0;
        }
        if (threadIdx.x < MM) {
            st->y[threadIdx.x] = threadIdx.x == 0 ? 1.0 : 0.0;
            st->y_prev[threadIdx.x] = threadIdx.x == 0 ? 1.0 : 0.0;
        }
    }
    if (threadIdx.x < MM) st->h[threadIdx.x] = threadIdx.x < m ? out[threadIdx.x] : 0.0;
    if (threadIdx.x >= 64) return;
    const double o = threadIdx.x < m ? out[threadIdx.x] : 0.0, hh = sum32(o * o);
    if (threadIdx.x != 0) return;
    if (keep) {
        st->m = keep;
        st->collapse = 0;
    }
    const double t1 = out[MT];
    const double nrm2 = t1 - hh;
    // a second projection only when the first left an overlap above what
    // the basis rows hold: an FP32 basis is orthonormal to its rounding
    // (6e-8), so a second pass there cannot improve the stored vector unless
    // the first left more than 1e-6 of it
    constexpr double kVisible = sizeof(VT) < sizeof(double) ? 1e-12 : 1e-26;
    const bool again = hh > kVisible * t1;
    st->reortho = again ? 1 : 0;
    if (!(nrm2 > 1e-28 * tt0) || !(nrm2 > 0.0)) {
        st->done = (rnorm <= 0.0) ? DONE_CONVERGED : DONE_STALLED;
    } else {
        st->tinv = 1.0 / sqrt(again ? nrm2 : t1);
    }
}

template <int MT, typename VT = double>
__device__ __forceinline__ void d_orth2(VT* __restrict__ V, int64_t n, const dav_state* st, const double* __restrict__ T, double* __restrict__ cin,
        float* __restrict__ c32, int64_t bid, int64_t nblk) {
    if (st->done) return;
    const int m = st->m;
    const double sc = st->tinv;
    const bool re = st->reortho != 0;
    VT* vm = V + (int64_t)m * n;
    const bool lo = (st->phase == 0) && c32;
    if (!re) {
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            const double t = T[i] * sc;
            vm[i] = (VT)t;
            cin[i] = t;
            if (lo) c32[i] = (float)t;
        }
        return;
    }
    with_rows<MT>(m, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        double h[NR];
        const VT* vr[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            h[k] = (k < m) ? st->h[k] : 0.0;
            vr[k] = row_ptr(V, k, m, n);
        }
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double v[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(vr[k] + i);
            double t = T[i];
#pragma unroll
            for (int k = 0; k < NR; ++k) t -= h[k] * v[k];
            t *= sc;
            vm[i] = (VT)t;
            cin[i] = t;
            if (lo) c32[i] = (float)t;
        }
    });
}

// AV[m] = S; partial columns 0..m: V[k] . S.
template <int MT, typename VT = double>
__device__ __forceinline__ void d_dots(const VT* __restrict__ V, VT* __restrict__ AV, const double* __restrict__ S, int64_t n,
       const dav_state* st, double* __restrict__ partial, int64_t bid, int64_t nblk) {
    if (st->done) return;
    const int m = st->m;
    double acc[MT + 1];
#pragma unroll
    for (int k = 0; k <= MT; ++k) acc[k] = 0.0;
    VT* avm = AV + (int64_t)m * n;
    const int cnt = m + 1;   // rows 0..m, the new vector included (cnt <= MT)
    with_rows<MT>(cnt, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        const VT* vr[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) vr[k] = row_ptr(V, k, cnt, n);
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double v[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) v[k] = __builtin_nontemporal_load(vr[k] + i);
            const double s = S[i];
            avm[i] = (VT)s;
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[k] += (k < cnt) ? v[k] * s : 0.0;
        }
    });
    block_to_partial<MT + 1>(acc, partial, bid, nblk);
}

// G[:, m] from the partials, m += 1, then the lowest eigenpair of G: theta, y
// (y_prev keeps the old y).
template <int MT>
__device__ __forceinline__ void f_dots_fin(const double* __restrict__ partial, int nrows, dav_state* st) {
    const int over = st->done, m0 = st->m, m = m0 + 1;
    __shared__ double out[MT + 1];
    __shared__ eig_work<MT, 1> work;
    const int lane = threadIdx.x;
    double a[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) a[j] = st->G[(lane & (MM - 1)) * MM + j];
    const double yp = lane < MM ? st->y[lane] : 0.0;
    reduce_rows<MT + 1>(partial, nrows, out);
    if (over || lane >= 64) return;   // one wavefront
#pragma unroll
    for (int j = 0; j < MT; ++j)      // row and column m0 are new
        a[j] = (lane < m && j < m) ? (lane == m0 ? out[j] : j == m0 ? out[lane] : a[j]) : 0.0;
    if (lane < m) {
        st->G[lane * MM + m0] = out[lane];
        st->G[m0 * MM + lane] = out[lane];
    }
    double theta[1], y[1];
    lowest_pairs<MT, 1>(a, m, 1, work, theta, y);
    // sign: keep continuity with the previous Ritz vector
    const double dp = sum32(lane < m ? y[0] * yp : 0.0);
    if (lane < MM) {
        st->y_prev[lane] = yp;
        st->y[lane] = lane < m ? (dp < 0.0 ? -y[0] : y[0]) : 0.0;
    }
    if (lane == 0) {
        st->m = m;
        st->theta = theta[0];
    }
}

// Final vector x = V y; per-block largest |x| (lowest index on ties) and |x|^2.
template <int MT, typename VT = double>
__device__ __forceinline__ void d_final(const VT* __restrict__ V, int64_t n, const dav_state* st, double* __restrict__ out,
        double* __restrict__ partial, int64_t bid, int64_t nblk) {
    const int m = st->m;
    __shared__ double sv[kThreads], sn[kThreads];
    __shared__ long long si[kThreads];
    double best = -1.0, nrm = 0.0;
    long long bi = -1;
    with_rows<MT>(m, [&](auto nr_) {
        constexpr int NR = decltype(nr_)::value;
        double y[NR];
        const VT* vr[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            y[k] = (k < m) ? st->y[k] : 0.0;
            vr[k] = row_ptr(V, k, m, n);
        }
        for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
            double x = 0.0;
#pragma unroll
            for (int k = 0; k < NR; ++k) x += y[k] * __builtin_nontemporal_load(vr[k] + i);
            out[i] = x;
            nrm += x * x;
            const double a = fabs(x);
            if (a > best) { best = a; bi = i; }
        }
    });
    sv[threadIdx.x] = best; si[threadIdx.x] = bi; sn[threadIdx.x] = nrm;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double v = sv[threadIdx.x + s];
            const long long j = si[threadIdx.x + s];
            if (j >= 0 && (si[threadIdx.x] < 0 || v > sv[threadIdx.x] || (v == sv[threadIdx.x] && j < si[threadIdx.x]))) {
                sv[threadIdx.x] = v;
                si[threadIdx.x] = j;
            }
            sn[threadIdx.x] += sn[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[(size_t)bid * kPstride + 0] = sv[0];
        partial[(size_t)bid * kPstride + 1] = (double)si[0];
        partial[(size_t)bid * kPstride + 2] = sn[0];
    }
}

// sign of the largest entry, read before any rescaling
__device__ __forceinline__ void f_final_sign(const double* __restrict__ out, dav_state* st) {
    if (threadIdx.x == 0) {
        const int64_t k = st->kmin;
        if (out[k] < 0.0) st->tinv = -st->tinv;
    }
}

__device__ __forceinline__ void d_final_scale(double* __restrict__ out, int64_t n, const dav_state* st, int64_t bid, int64_t nblk) {
    const double sc = st->tinv;
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads)
        out[i] *= sc;
}

// ---------------------------------------------------------------- locked roots
// Projection of a vector v against nx locked, orthonormal vectors X (the
// roots already found), so that the solve for the next root stays in their
// orthogonal complement.  One classical Gram-Schmidt pass, normalised with
// the norm it predicts; a second pass only when the first removed more than
// half of the squared norm (then the predicted norm is not trusted).

// partial column 0: |v|^2; columns 1..SQD_MAXLOCK: X_k . v (zero past nx)
// v is V itself (vrow = 0) or row st->m of V (the vector just appended).
__device__ __forceinline__ void d_xdots(const double* __restrict__ X, int nx, const double* __restrict__ V,
                                        int vrow, int64_t n, const dav_state* st, int round,
                                        double* __restrict__ partial, int64_t bid, int64_t nblk) {
    if (st->done || (round == 1 && !st->xredo)) return;
    const double* v = vrow ? V + (int64_t)st->m * n : V;
    double acc[1 + SQD_MAXLOCK];
#pragma unroll
    for (int k = 0; k <= SQD_MAXLOCK; ++k) acc[k] = 0.0;
    const double* xr[SQD_MAXLOCK];
#pragma unroll
    for (int k = 0; k < SQD_MAXLOCK; ++k) xr[k] = row_ptr(X, k, nx, n);
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
        const double vi = v[i];
        double x[SQD_MAXLOCK];
#pragma unroll
        for (int k = 0; k < SQD_MAXLOCK; ++k) x[k] = xr[k][i];
        acc[0] += vi * vi;
#pragma unroll
        for (int k = 0; k < SQD_MAXLOCK; ++k) acc[1 + k] += (k < nx) ? x[k] * vi : 0.0;
    }
    block_to_partial<1 + SQD_MAXLOCK>(acc, partial, bid, nblk);
}

__device__ __forceinline__ void f_xfin(const double* __restrict__ partial, int nrows, int nx, dav_state* st, int round) {
    if (st->done || (round == 1 && !st->xredo)) return;
    __shared__ double out[1 + SQD_MAXLOCK];
    reduce_rows<1 + SQD_MAXLOCK>(partial, nrows, out);
    if (threadIdx.x != 0) return;
    double cc = 0.0;
    for (int k = 0; k < SQD_MAXLOCK; ++k) {
        st->xc[k] = (k < nx) ? out[1 + k] : 0.0;
        cc += st->xc[k] * st->xc[k];
    }
    const double a2 = out[0], b2 = a2 - cc;
    if (round == 0 && b2 < 0.5 * a2) {
        st->xredo = 1;
        st->xscale = 1.0;
        return;
    }
    if (round == 0) st->xredo = 0;
    if (!(b2 > 1e-28 * a2) || !(b2 > 0.0)) {   // nothing left outside the locked space
        st->done = DONE_STALLED;
        return;
    }
    st->xscale = 1.0 / sqrt(b2);
}

// v = (v - X xc) * xscale; after the last pass also cin (and c32) = v
__device__ __forceinline__ void d_xapply(const double* __restrict__ X, int nx, double* __restrict__ V, int vrow,
                                         int64_t n, const dav_state* st, int round, double* __restrict__ cin,
                                         float* __restrict__ c32, int64_t bid, int64_t nblk) {
    if (st->done || (round == 1 && !st->xredo)) return;
    double* v = vrow ? V + (int64_t)st->m * n : V;
    const bool last = (round == 1) || !st->xredo;
    const double sc = st->xscale;
    double c[SQD_MAXLOCK];
    const double* xr[SQD_MAXLOCK];
#pragma unroll
    for (int k = 0; k < SQD_MAXLOCK; ++k) {
        c[k] = (k < nx) ? st->xc[k] : 0.0;
        xr[k] = row_ptr(X, k, nx, n);
    }
    const bool lo = (st->phase == 0) && c32;
    for (int64_t i = (int64_t)bid * kThreads + threadIdx.x; i < n; i += (int64_t)nblk * kThreads) {
        double x[SQD_MAXLOCK];
#pragma unroll
        for (int k = 0; k < SQD_MAXLOCK; ++k) x[k] = xr[k][i];
        double t = v[i];
#pragma unroll
        for (int k = 0; k < SQD_MAXLOCK; ++k) t -= c[k] * x[k];
        t *= sc;
        v[i] = t;
        if (last) {
            cin[i] = t;
            if (lo) c32[i] = (float)t;
        }
    }
}

__device__ __forceinline__ void f_set_phase(dav_state* st, int phase, int done) {
    if (threadIdx.x == 0) {
        st->phase = phase;
        st->phase_start = st->iter;
        st->done = done;
    }
}


}  // namespace dav
