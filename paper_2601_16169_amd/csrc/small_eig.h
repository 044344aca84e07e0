// The lowest eigenpairs of the small projected matrices (m <= 32), by one
// wavefront: Householder reduction to tridiagonal form with a row of the
// matrix per lane, multisection on Sturm counts, inverse iteration on the
// tridiagonal matrix and the reflections applied to its vectors (Golub and
// Van Loan, Matrix Computations, 8.3 and 8.4).  What bounds it is a chain of
// dependent steps; keeping the matrix in registers and the sums within a
// wavefront leaves some 22 short steps for m = 24, where cyclic Jacobi takes
// two or three sweeps of 23 rotations with two workgroup barriers each
// (finishing kernel of a Davidson iteration, m up to 24: 60 us then, 27 now;
// the block solver's k_beigh for four pairs of 24 rows: 81 and 38).  Rows
// are exchanged through the LDS: read from lanes, the values pass through the
// scalar registers one by one (33 us).
#pragma once

#include "sqd_internal.h"

namespace dav {

// 1/x and 1/sqrt(x) from the hardware estimates refined by two Newton steps
// (each squares the relative error, so two reach FP64 rounding); a dependent
// chain far shorter than IEEE division and square root.
__device__ __forceinline__ double rcp_refined(double x) {
    double r = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int k = 0; k < 2; ++k) r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

__device__ __forceinline__ double rsqrt_refined(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
#pragma unroll
    for (int k = 0; k < 2; ++k) y = fma(y, fma(-h * y, y, 0.5), y);
    return y;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v) {
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
__device__ __forceinline__ double lane_of(double v, int lane) {   // lane uniform
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
// sum over lanes 0..31 (row shifts by 1, 2, 4, 8, then row 0's total into row
// 1), the same value in every lane
__device__ __forceinline__ double sum32(double v) {
    v += dpp_or_zero<0x111, 0xf>(v);
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    return lane_of(v, 31);
}

// Workspace (LDS) of lowest_pairs.
template <int MT, int KR>
struct eig_work {
    double2 de[MT];                   // diagonal and next off-diagonal element
    double tau[MT];
    double2 v[MT][MT / 2];            // reflection k, by row
    double2 q[MT / 2], row[MT / 2], q2[MT];
    double z[MT][KR];
    double u0[MT][KR], u1[MT][KR], u2[MT][KR], mu[MT][KR];   // u0: reciprocals of the pivots
    int sw[MT][KR];
};

// The k <= KR lowest eigenpairs of the symmetric m x m matrix (1 <= m <= MT <=
// 32) whose row `lane` each lane of one wavefront holds in a (zeros past m):
// theta ascending and y, the lane's component of every vector, normalised.
template <int MT, int KR>
__device__ __forceinline__ void lowest_pairs(double (&a)[MT], int m, int k, eig_work<MT, KR>& w, double (&theta)[KR],
                                             double (&y)[KR]) {
    const int lane = threadIdx.x & 63;
    // ---- tridiagonal form.  Vectors are handed round through LDS (each lane
    // reads all of them, two elements at a time, at addresses that do not
    // depend on the lane).
    double* row = reinterpret_cast<double*>(w.row);
    double* qv = reinterpret_cast<double*>(w.q);
    for (int c = 0; c < m; ++c) {
        if (lane == c) {   // row c, by symmetry column c
#pragma unroll
            for (int j = 0; j < MT / 2; ++j) w.row[j] = make_double2(a[2 * j], a[2 * j + 1]);
        }
        double* vc = reinterpret_cast<double*>(w.v[c]);
        __threadfence_block();
        const double x = (lane > c && lane < m) ? row[lane] : 0.0;
        const double dc = row[c];
        double tau = 0.0, v = 0.0, e = c + 1 < m ? row[c + 1] : 0.0;
        if (c + 2 < m) {
            const double s2 = sum32(lane > c + 1 ? x * x : 0.0);
            if (s2 > 1e-290) {   // (a column this small is zero to rounding, and below the estimates' range)
                const double x1 = e, n2 = x1 * x1 + s2, nr = n2 * rsqrt_refined(n2);
                e = x1 > 0.0 ? -nr : nr;
                v = lane == c + 1 ? x1 - e : x;
                tau = rcp_refined(nr * (nr + fabs(x1)));   // 2 / |v|^2
            }
        }
        if (lane == 0) {
            w.de[c] = make_double2(dc, e);
            w.tau[c] = tau;
        }
        if (lane < MT) vc[lane] = v;
        if (tau == 0.0) continue;
        __threadfence_block();
        double p0 = 0.0, p1 = 0.0;
#pragma unroll
        for (int j = 0; j < MT / 2; ++j) {
            const double2 t = w.v[c][j];
            p0 += a[2 * j] * t.x;
            p1 += a[2 * j + 1] * t.y;
        }
        const double p = (lane > c && lane < m) ? (p0 + p1) * tau : 0.0;
        const double q = p - 0.5 * tau * sum32(p * v) * v;
        if (lane < MT) qv[lane] = q;
        __threadfence_block();
#pragma unroll
        for (int j = 0; j < MT / 2; ++j) {
            const double2 t = w.v[c][j], u = w.q[j];
            a[2 * j] -= v * u.x + q * t.x;
            a[2 * j + 1] -= v * u.y + q * t.y;
        }
    }
    __threadfence_block();
    // ---- eigenvalues: scaled to norm one, a group of 64 / KR lanes per root
    double di = 0.0, ei = 0.0, ep = 0.0, es = 0.0;
    if (lane < m) {
        di = w.de[lane].x;
        es = lane + 1 < m ? w.de[lane].y : 0.0;
        ei = fabs(es);
        ep = lane > 0 ? fabs(w.de[lane - 1].y) : 0.0;
    }
    double glo = lane < m ? di - ei - ep : INFINITY, ghi = lane < m ? di + ei + ep : -INFINITY;
    for (int o = 16; o > 0; o >>= 1) {
        glo = fmin(glo, __shfl_xor(glo, o));
        ghi = fmax(ghi, __shfl_xor(ghi, o));
    }
    glo = lane_of(glo, 0);
    ghi = lane_of(ghi, 0);
    const double norm = fmax(fabs(glo), fabs(ghi));
    const double inv = norm > 0.0 ? 1.0 / norm : 1.0;
    // scaled; de[i] = (d_i, e_i), and beside it (d_i, e_{i-1}^2) for the counts
    double2* dq = w.q2;
    if (lane < MT) {
        w.de[lane] = make_double2(di * inv, es * inv);
        dq[lane] = make_double2(di * inv, (ep * inv) * (ep * inv));
    }
    __threadfence_block();
    constexpr int L = 64 / KR;
    const int r = lane / L, sub = lane - r * L;   // this lane's root and section
    double lo = glo * inv - 4e-16, hi = ghi * inv + 4e-16;
    constexpr int kRounds = KR == 1 ? 9 : KR == 2 ? 11 : KR == 4 ? 13 : 17;   // (L + 1)^rounds > 2^53
    for (int it = 0; it < kRounds; ++it) {
        const double width = hi - lo;
        const double x = lo + width * ((double)(sub + 1) * (1.0 / (L + 1)));
        // eigenvalues below x: sign changes of the leading minors (a zero
        // counts as positive: its neighbours differ in sign)
        double p0 = 1.0, p1 = dq[0].x - x;
        int sign = __double2hiint(p1) < 0 ? 1 : 0, cnt = sign;
#pragma unroll 4
        for (int i = 1; i < m; ++i) {
            const double2 t = dq[i];
            const double p2 = (t.x - x) * p1 - t.y * p0;
            const int now = (int)((unsigned)__double2hiint(p2) >> 31);
            cnt += now ^ sign;
            sign = now;
            p0 = p1;
            p1 = p2;
        }
        const uint64_t hit = __ballot(cnt > r) >> (r * L);
        const uint64_t grp = L == 64 ? hit : hit & ((1ull << (L & 63)) - 1);
        const int first = grp ? __ffsll((unsigned long long)grp) - 1 : L;   // first section above the root
        const double nlo = first > 0 ? lo + width * ((double)first * (1.0 / (L + 1))) : lo;
        if (first < L) hi = lo + width * ((double)(first + 1) * (1.0 / (L + 1)));
        lo = nlo;
    }
    const double lam = 0.5 * (lo + hi);
    // ---- vectors: inverse iteration, lane q < k its own root, LU with row exchanges
    const double lam_q = __shfl(lam, min(lane, KR - 1) * L);
    if (lane < k && lane < KR) {
        const int q = lane;
        // right-hand sides of positive entries, different for every root (the
        // vectors of roots that agree to rounding must not)
        auto rhs = [&](int i) { return 1.0 + 0.125 * (double)((5 * i + 3 * q * (i + 1)) & 7); };
        double2 t0 = w.de[0];
        double c0 = t0.x - lam_q, c1 = t0.y, f = rhs(0);
        double2 t1 = w.de[m > 1 ? 1 : 0];
        for (int i = 0; i + 1 < m; ++i) {
            const double2 t2 = w.de[i + 2 < m ? i + 2 : m - 1];   // (loads before this step's stores)
            const double sub_ = t0.y, nd = t1.x - lam_q, ne = i + 2 < m ? t1.y : 0.0, g = rhs(i + 1);
            t0 = t1;
            t1 = t2;
            // the pivot row: this one, or after an exchange the next (sub, nd, ne)
            const bool sw = fabs(sub_) > fabs(c0);
            double piv = sw ? sub_ : c0;
            if (fabs(piv) < 2e-16) piv = 2e-16;
            const double ip = rcp_refined(piv), mu = (sw ? c0 : sub_) * ip;
            const double a1 = sw ? nd : c1, a2 = sw ? ne : 0.0, fr = sw ? g : f;
            w.u0[i][q] = ip;
            w.u1[i][q] = a1;
            w.u2[i][q] = a2;
            w.mu[i][q] = mu;
            w.sw[i][q] = sw;
            w.z[i][q] = fr;
            f = (sw ? f : g) - mu * fr;
            c0 = (sw ? c1 : nd) - mu * a1;
            c1 = (sw ? 0.0 : ne) - mu * a2;
        }
        if (fabs(c0) < 2e-16) c0 = 2e-16;
        w.u0[m - 1][q] = rcp_refined(c0);
        w.u1[m - 1][q] = 0.0;
        w.u2[m - 1][q] = 0.0;
        w.z[m - 1][q] = f;
        for (int pass = 0; pass < 2; ++pass) {
            if (pass) {   // right-hand side: the first vector, scaled, through the eliminations
                double big = 0.0;
                for (int i = 0; i < m; ++i) big = fmax(big, fabs(w.z[i][q]));
                const double sc = 1.0 / big;
                double x0 = w.z[0][q] * sc;
                for (int i = 0; i + 1 < m; ++i) {
                    const double x1 = w.z[i + 1][q] * sc, mu = w.mu[i][q];
                    if (w.sw[i][q]) {
                        w.z[i][q] = x1;
                        x0 = x0 - mu * x1;
                    } else {
                        w.z[i][q] = x0;
                        x0 = x1 - mu * x0;
                    }
                }
                w.z[m - 1][q] = x0;
            }
            double z1 = 0.0, z2 = 0.0;
            for (int i = m - 1; i >= 0; --i) {
                const double z0 = (w.z[i][q] - w.u1[i][q] * z1 - w.u2[i][q] * z2) * w.u0[i][q];
                w.z[i][q] = z0;
                z2 = z1;
                z1 = z0;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
#pragma unroll
    for (int q = 0; q < KR; ++q) {
        theta[q] = __shfl(lam, q * L) * norm;
        y[q] = (q < k && lane < m) ? w.z[lane][q] : 0.0;
        if (q >= k) continue;
        // scaled first: the entries reach the reciprocal of the rounding unit
        double big = fabs(y[q]);
        for (int o = 16; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o));
        y[q] *= 1.0 / lane_of(big, 0);
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int s = 0; s < q; ++s) y[q] -= sum32(y[q] * y[s]) * y[s];
            y[q] *= rsqrt_refined(sum32(y[q] * y[q]));
        }
    }
    // ---- back to the matrix's own basis
    for (int c = m - 3; c >= 0; --c) {
        const double tau = w.tau[c];
        if (tau == 0.0) continue;
        const double v = lane < m ? reinterpret_cast<const double*>(w.v[c])[lane] : 0.0;
#pragma unroll
        for (int q = 0; q < KR; ++q) y[q] -= tau * sum32(v * y[q]) * v;
    }
}

}  // namespace dav
