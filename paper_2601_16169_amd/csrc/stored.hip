// Stored-H mode: H restricted to S evaluated once into CSR on the device and
// applied by a sparse matrix-vector product in every Davidson iteration (the
// second of the two methods of Sec. II: compute the matrix elements one time,
// keep them, and reuse them, trading memory for the recomputation the
// matrix-free product does).
//
// Row d = (ia, ib) lists, in this order: the diagonal, the alpha singles and
// alpha doubles of ia (columns ia' * nb + ib), the beta singles and beta
// doubles of ib (columns ia * nb + ib'), and the alpha x beta singles pairs
// (columns ia' * nb + ib').  Each in-set connection appears exactly once (a
// string pair at Hamming distance 2 is a single, at 4 a double), so the row
// length is 1 + A(ia) + B(ib) + sa(ia) sb(ib), with A = singles + doubles and
// s = singles of each spin, and the row pointer has a closed form in per-spin
// prefix sums.  Values come from the same per-string tables as the
// matrix-free kernels: same-spin singles add the cross-spin term
// sum_{k in other string} (pq|kk), alpha-beta pairs are s_a s_b (ai|bj).
//
// The product y = H x streams the values from HBM with the parts of x that a
// block of rows reads staged in the LDS (k_spmv_staged), or, for few, short or
// very long rows, values and columns with a wavefront per row (k_spmv).
#include <algorithm>

#include "sqd_internal.h"

namespace {

constexpr int kRowsPerBlock = 4;   // wavefronts (rows) per 256-thread workgroup

struct store_args {
    int64_t na, nb;
    const int* as_off; const uint32_t* as_pk; const double* as_val;
    const int* ad_off; const int* ad_nbr; const double* ad_val;
    const int* bs_off; const uint32_t* bs_pk; const double* bs_val;
    const int* bd_off; const int* bd_nbr; const double* bd_val;
    const uint64_t* astr; const uint64_t* bstr;
    int nw;                    // words per string
    const double* jk;          // jk[k * norb2 + pq] = (pq|kk)
    const double* V;           // (pq|rs) as a norb2 x norb2 matrix
    int norb;
    const double* diag;
    const int64_t* rp;
    int* col;
    double* val;
};

// sum over occupied k of the string (nw words), in increasing k, of (pq|kk)
__device__ __forceinline__ double cross_spin(const double* __restrict__ jk, int norb2, const uint64_t* s, int nw,
                                             int pair) {
    double w = 0.0;
    str_for_each(s, nw, [&](int k) { w += jk[(int64_t)k * norb2 + pair]; });
    return w;
}

// row pointer: rp[d] = RA[ia] + ib (1 + A(ia)) + PB[ib] + sa(ia) PSB[ib]
__global__ void k_store_rowptr(const int64_t* __restrict__ RA, const int64_t* __restrict__ PB,
                               const int64_t* __restrict__ PSB, const int* __restrict__ as_off,
                               const int* __restrict__ ad_off, int64_t na, int64_t nb, int64_t* __restrict__ rp) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t dim = na * nb;
    if (d > dim) return;
    if (d == dim) { rp[d] = RA[na]; return; }
    const int64_t ia = d / nb, ib = d - ia * nb;
    const int64_t sa = as_off[ia + 1] - as_off[ia];
    const int64_t A1 = 1 + sa + (ad_off[ia + 1] - ad_off[ia]);
    rp[d] = RA[ia] + ib * A1 + PB[ib] + sa * PSB[ib];
}

__global__ void __launch_bounds__(256) k_store_fill(store_args a) {
    const int lane = threadIdx.x & 63;
    const int norb2 = a.norb * a.norb;
    const int64_t dim = a.na * a.nb;
    for (int64_t d = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6); d < dim;
         d += (int64_t)gridDim.x * kRowsPerBlock) {
        const int64_t ia = d / a.nb, ib = d - ia * a.nb;
        const int sa0 = a.as_off[ia], nsa = a.as_off[ia + 1] - sa0;
        const int da0 = a.ad_off[ia], nda = a.ad_off[ia + 1] - da0;
        const int sb0 = a.bs_off[ib], nsb = a.bs_off[ib + 1] - sb0;
        const int db0 = a.bd_off[ib], ndb = a.bd_off[ib + 1] - db0;
        const int64_t e1 = 1 + nsa, e2 = e1 + nda, e3 = e2 + nsb, e4 = e3 + ndb;
        const int64_t e5 = e4 + (int64_t)nsa * nsb;
        const int64_t base = a.rp[d];
        const uint64_t* sa_str = a.astr + ia * a.nw;
        const uint64_t* sb_str = a.bstr + ib * a.nw;
        for (int64_t e = lane; e < e5; e += 64) {
            int64_t c;
            double v;
            if (e == 0) {
                c = d;
                v = a.diag[d];
            } else if (e < e1) {            // alpha single: ia' <- ia, beta string fixed
                const int p = sa0 + (int)(e - 1);
                const uint32_t pk = a.as_pk[p];
                const int pair = (int)((pk >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
                const double w = cross_spin(a.jk, norb2, sb_str, a.nw, pair);
                v = a.as_val[p] + ((pk >> 31) ? -w : w);
                c = (int64_t)(pk & SQD_NBR_MASK) * a.nb + ib;
            } else if (e < e2) {            // alpha double
                const int p = da0 + (int)(e - e1);
                v = a.ad_val[p];
                c = (int64_t)a.ad_nbr[p] * a.nb + ib;
            } else if (e < e3) {            // beta single: ib' <- ib, alpha string fixed
                const int p = sb0 + (int)(e - e2);
                const uint32_t pk = a.bs_pk[p];
                const int pair = (int)((pk >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
                const double w = cross_spin(a.jk, norb2, sa_str, a.nw, pair);
                v = a.bs_val[p] + ((pk >> 31) ? -w : w);
                c = ia * a.nb + (int64_t)(pk & SQD_NBR_MASK);
            } else if (e < e4) {            // beta double
                const int p = db0 + (int)(e - e3);
                v = a.bd_val[p];
                c = ia * a.nb + a.bd_nbr[p];
            } else {                        // one alpha and one beta single
                const int k = (int)(e - e4);
                const int ka = k / nsb, kb = k - ka * nsb;
                const uint32_t pa = a.as_pk[sa0 + ka], pb = a.bs_pk[sb0 + kb];
                const int qa = (int)((pa >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
                const int qb = (int)((pb >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
                v = a.V[(int64_t)qa * norb2 + qb];
                if ((pa ^ pb) >> 31) v = -v;
                c = (int64_t)(pa & SQD_NBR_MASK) * a.nb + (int64_t)(pb & SQD_NBR_MASK);
            }
            a.col[base + e] = (int)c;
            a.val[base + e] = v;
        }
    }
}

struct xcd_rows {
    int64_t r[9];
};

// y[r] = sum_k val[k] x[col[k]]: one wavefront per row, four 64-entry blocks
// of the row in flight per lane; the matrix stream is read non-temporally so
// that the cached lines of x stay resident.  The rows are cut into eight
// ranges of equal element counts, one per XCD (workgroup k runs on XCD k mod
// 8 and walks range k mod 8), so that the rows in flight on one XCD share
// their alpha string and the rows of x they gather from stay in that XCD's
// L2.
__global__ void __launch_bounds__(256) k_spmv(const int64_t* __restrict__ rp, const int* __restrict__ col,
                                              const double* __restrict__ val, const double* __restrict__ x,
                                              double* __restrict__ y, xcd_rows xr, const int* __restrict__ skip) {
    if (skip && *skip) return;
    const int lane = threadIdx.x & 63;
    const int xcd = (int)(blockIdx.x & 7);
    const int64_t j = blockIdx.x >> 3, nj = gridDim.x >> 3;
    const int64_t r0 = xr.r[xcd], r1 = xr.r[xcd + 1];
    for (int64_t r = r0 + j * kRowsPerBlock + (threadIdx.x >> 6); r < r1; r += nj * kRowsPerBlock) {
        const int64_t k1 = rp[r + 1];
        int64_t k = rp[r] + lane;
        double acc = 0.0;
        for (; k + 192 < k1; k += 256) {
            int c[4];
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = __builtin_nontemporal_load(col + k + 64 * u);
                v[u] = __builtin_nontemporal_load(val + k + 64 * u);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += v[u] * x[c[u]];
        }
        for (; k < k1; k += 64) acc += __builtin_nontemporal_load(val + k) * x[__builtin_nontemporal_load(col + k)];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (lane == 0) y[r] = acc;
    }
}

// The same product with the parts of x that a block of rows reads staged in the
// LDS.  What bounds k_spmv is the gathers from x: 64-byte requests to the L2 for
// eight bytes each (1001 x 903 strings, 3.1e8 elements: 1.61 ms; keeping twice the
// matrix stream in flight changed it by 2%).  The columns of a row follow from
// the lists of its two strings, in the order in which the row was filled, so a
// workgroup takes kSpmvRows rows (ia, ib0 ..), stages for the alpha part the kSpmvRows
// values of each neighbour of ia, for the beta part the row ia of x and for the
// alpha-beta part the rows of the alpha singles, as many at a time as fit, and
// streams the values alone (8 bytes an element): 0.87 ms.  A wavefront holds the
// sums of its eight rows, a lane taking every 64th element.
constexpr int kSpmvWaves = 16, kSpmvPer = 8;
constexpr int kSpmvRows = kSpmvWaves * kSpmvPer;
constexpr int kSpmvCap = 64 * (kSpmvRows + 1);   // values of x staged at a time

struct staged_args {
    int64_t nb;
    const int *as_off, *ad_off, *ad_nbr, *bs_off, *bd_off, *bd_nbr;
    const uint32_t *as_pk, *bs_pk;
    const int64_t* rp;
    const double* val;
    const double* x;
    double* y;
    const int2* units;   // (ia, ib0); ia < 0: none
    int cap, step;       // values staged at a time; rows of a unit
};

// v[0..N) summed over the lanes: lane l returns the sum of value l >> (6 - log2 N)
// (the exchanges halve the values)
template <int N, int MASK>
__device__ __forceinline__ double lane_sums(const double (&v)[N], int lane) {
    if constexpr (N > 1) {
        double h[N / 2];
        const bool up = (lane & MASK) != 0;
#pragma unroll
        for (int j = 0; j < N / 2; ++j) h[j] = (up ? v[j + N / 2] : v[j]) + __shfl_xor(up ? v[j] : v[j + N / 2], MASK);
        return lane_sums<N / 2, MASK / 2>(h, lane);
    } else {
        double s = v[0];
#pragma unroll
        for (int m = MASK; m > 0; m >>= 1) s += __shfl_xor(s, m);
        return s;
    }
}

__global__ void __launch_bounds__(64 * kSpmvWaves, 8) k_spmv_staged(staged_args a, const int* __restrict__ skip) {
    if (skip && *skip) return;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int2 unit = a.units[blockIdx.x];
    if (unit.x < 0) return;
    double* xs = reinterpret_cast<double*>(lds_raw);
    int* list = reinterpret_cast<int*>(xs + a.cap);   // beta singles of the rows, as neighbours
    const int64_t nb = a.nb, ia = unit.x;
    const int ib0 = unit.y, rows = (int)min((int64_t)a.step, nb - ib0);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sa0 = a.as_off[ia], nsa = a.as_off[ia + 1] - sa0;
    const int da0 = a.ad_off[ia], nA = nsa + a.ad_off[ia + 1] - da0;
    const int list0 = a.bs_off[ib0], nlist = a.bs_off[ib0 + rows] - list0;
    for (int q = threadIdx.x; q < nlist; q += 64 * kSpmvWaves) list[q] = (int)(a.bs_pk[list0 + q] & SQD_NBR_MASK);
    // the wavefront's rows (those past the end repeat the last and are not stored)
    const int each = (rows + kSpmvWaves - 1) / kSpmvWaves;
    const int r0 = wave * each, mine = max(0, min(each, rows - r0));
    double acc[kSpmvPer];
    // lane j holds what the walks need of row j (read from lanes: scalars for every
    // row would not stay in registers): its next value, from val; the first of its
    // beta singles in list, and their number; its number of beta entries, and the
    // first double less the singles
    const int64_t first = ia * nb + ib0 + min(r0, rows - 1);
    const double* val = a.val + a.rp[first];
    const int mr = min(r0 + (lane & (kSpmvPer - 1)), rows - 1);
    const int at_v = (int)(a.rp[ia * nb + ib0 + mr] - a.rp[first]);
    const int sb_v = a.bs_off[ib0 + mr] - list0, nsb_v = a.bs_off[ib0 + mr + 1] - list0 - sb_v;
    const int db_v = a.bd_off[ib0 + mr] - nsb_v, nB_v = a.bd_off[ib0 + mr + 1] - db_v;
    auto of = [](int v, int j) { return __builtin_amdgcn_readlane(v, j); };
    {
        const double t = lane < mine ? val[at_v] * a.x[ia * nb + ib0 + mr] : 0.0;   // the diagonal
#pragma unroll
        for (int j = 0; j < kSpmvPer; ++j) acc[j] = lane == j ? t : 0.0;
    }
    // alpha part: 64 neighbours at a time, neighbour e of row q at e * (kSpmvRows + 1) + q
    for (int e0 = 0; e0 < nA; e0 += 64) {
        const int ne = min(64, nA - e0);
        double v[kSpmvPer];
#pragma unroll
        for (int j = 0; j < kSpmvPer; ++j)
            v[j] = (lane < ne && j < mine) ? __builtin_nontemporal_load(val + of(at_v, j) + 1 + e0 + lane) : 0.0;
        __syncthreads();
        for (int e = wave; e < ne; e += kSpmvWaves) {
            const int p = e0 + e;
            const int64_t src = p < nsa ? (int64_t)(a.as_pk[sa0 + p] & SQD_NBR_MASK) : (int64_t)a.ad_nbr[da0 + p - nsa];
            const double* xr = a.x + src * nb + ib0;
#pragma unroll
            for (int u = 0; u < kSpmvRows / 64; ++u)
                if (lane + 64 * u < rows) xs[e * (kSpmvRows + 1) + lane + 64 * u] = xr[lane + 64 * u];
        }
        __syncthreads();
        if (lane < ne) {
#pragma unroll
            for (int j = 0; j < kSpmvPer; ++j)
                if (j < mine) acc[j] += v[j] * xs[lane * (kSpmvRows + 1) + r0 + j];
        }
    }
    // beta part: row ia of x; then alpha-beta part: the rows of the alpha singles.
    // The first values of four rows at a time load ahead of their use.
    constexpr int kH = kSpmvPer / 2;
    __syncthreads();
    for (int64_t q = threadIdx.x; q < nb; q += 64 * kSpmvWaves) xs[q] = a.x[ia * nb + q];
    __syncthreads();
    const double* bval = val + 1 + nA;
#pragma unroll
    for (int h = 0; h < kSpmvPer; h += kH) {
        int most = 0;
#pragma unroll
        for (int j = 0; j < kH; ++j)
            if (h + j < mine) most = max(most, of(nB_v, h + j));
        for (int k = lane; k < most; k += 64) {
            double v[kH];
            int c[kH];
#pragma unroll
            for (int j = 0; j < kH; ++j) {
                const bool in = k < of(nB_v, h + j) && h + j < mine;
                v[j] = in ? __builtin_nontemporal_load(bval + of(at_v, h + j) + k) : 0.0;
                c[j] = (in && k >= of(nsb_v, h + j)) ? a.bd_nbr[of(db_v, h + j) + k] : -1;
            }
#pragma unroll
            for (int j = 0; j < kH; ++j)
                if (k < of(nB_v, h + j) && h + j < mine) acc[h + j] += v[j] * xs[c[j] < 0 ? list[of(sb_v, h + j) + k] : c[j]];
        }
    }
    const int ab_v = at_v + nB_v;
    const int per = (int)(a.cap / nb);
    for (int ka0 = 0; ka0 < nsa; ka0 += per) {
        const int nka = min(per, nsa - ka0);
        __syncthreads();
        for (int e = 0; e < nka; ++e) {
            const double* xr = a.x + (int64_t)(a.as_pk[sa0 + ka0 + e] & SQD_NBR_MASK) * nb;
            for (int q = threadIdx.x; q < (int)nb; q += 64 * kSpmvWaves) xs[e * (int)nb + q] = xr[q];
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kSpmvPer; h += kH) {
            // the first 128 values of four rows in flight, then the rest of long rows
            // 256 at a time
            double v[kH][2];
#pragma unroll
            for (int j = 0; j < kH; ++j)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int k = 64 * u + lane, n = of(nsb_v, h + j);
                    v[j][u] = (k < nka * n && h + j < mine)
                                  ? __builtin_nontemporal_load(bval + of(ab_v, h + j) + (ka0 * n + k)) : 0.0;
                }
#pragma unroll
            for (int j = 0; j < kH; ++j) {
                const int n = of(nsb_v, h + j), len = h + j < mine ? nka * n : 0;
                const int* l = list + of(sb_v, h + j);
                const float inv = 1.0f / (float)max(n, 1);
                auto use = [&](double y, int k) {   // (k below 2^22: exact)
                    const int ka = (int)(((float)k + 0.5f) * inv), kb = k - ka * n;
                    if (k < len) acc[h + j] += y * xs[ka * (int)nb + l[kb]];
                };
#pragma unroll
                for (int u = 0; u < 2; ++u) use(v[j][u], 64 * u + lane);
                const double* row = bval + of(ab_v, h + j) + ka0 * n;
                for (int k0 = 128 + lane; k0 < len; k0 += 256) {
                    double w[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) w[u] = k0 + 64 * u < len ? __builtin_nontemporal_load(row + k0 + 64 * u) : 0.0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) use(w[u], k0 + 64 * u);
                }
            }
        }
    }
    const double s = lane_sums<kSpmvPer, 32>(acc, lane);
    const int j = lane >> 3;
    if ((lane & 7) == 0 && j < mine) a.y[ia * nb + ib0 + r0 + j] = s;
}

unsigned fill_grid(int64_t rows) {
    const int64_t b = (rows + kRowsPerBlock - 1) / kRowsPerBlock;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 1 << 16));
}

}  // namespace

void sqd_release_stored_h(sqd_space* sp) {
    void* ptrs[] = {sp->h_rowptr, sp->h_col, sp->h_val, sp->h_units};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    sp->bytes -= sp->h_bytes;
    sp->h_rowptr = nullptr;
    sp->h_col = nullptr;
    sp->h_val = nullptr;
    sp->h_units = nullptr;
    sp->h_nunits = sp->h_list = 0;
    sp->h_nnz = 0;
    sp->h_bytes = 0;
    sp->h_version = -1;
}

// Units of the staged product, or none where it is not taken: a row of x and the
// lists have to fit the LDS, two units are wanted for every compute unit, a unit
// of few rows leaves most of its lanes without work, and each staged value has to
// serve at least one element.  Measured on MI355X, us, rows from the L2 / staged:
// 252 x 252 strings 212 / 93, 400 x 300: 226 / 119, 2000 x 64: 156 / 105, 2000 x
// 130: 276 / 195, 20 x 5000: 124 / 86, 1500 x 700: 1752 / 879, 1500 x 1500: 3640 /
// 1940; not taken: 128 x 128 (128 units) 8 / 15, 3 x 12000 (282 units) 101 / 136,
// 5000 x 20 (20 rows) 208 / 296, 300 x 3000 (1.4 staged for an element) 1308 / 1392.
static int plan_staged(sqd_ctx* ctx, sqd_space* sp, const std::vector<int>& as, const std::vector<int>& ad,
                       const std::vector<int>& bs, const std::vector<int64_t>& PB, int64_t nnz) {
    const int64_t na = sp->sp[0].n, nb = sp->sp[1].n, nblk = (nb + kSpmvRows - 1) / kSpmvRows, step = (nb + nblk - 1) / nblk;
    int most = 0;
    for (int64_t b = 0; b < nb; b += step) most = std::max(most, bs[std::min(nb, b + step)] - bs[b]);
    const size_t cap = (size_t)std::max<int64_t>(kSpmvCap, nb);
    if (cap * 8 + (size_t)most * 4 > (size_t)ctx->max_lds) return SQD_OK;
    const int64_t per_string = (nb + step - 1) / step;   // units of an alpha string
    const int64_t staged = per_string * nb * (as[na] + na) + nb * (as[na] + ad[na]);
    if (na * per_string < 2 * ctx->num_cu || step < 32 || staged > nnz) return SQD_OK;
    // units of one alpha string on one XCD (they stage the same rows of x), the
    // strings dealt by their elements, heaviest first
    std::vector<std::pair<int64_t, int>> order(na);
    for (int64_t i = 0; i < na; ++i) {
        const int64_t sa = as[i + 1] - as[i], nA = sa + ad[i + 1] - ad[i];
        order[i] = {-(nb * (1 + nA) + PB[nb] + sa * bs[nb]), (int)i};
    }
    std::sort(order.begin(), order.end());
    std::vector<int2> per[8];
    int64_t load[8] = {};
    for (const auto& o : order) {
        const int q = (int)(std::min_element(load, load + 8) - load);
        load[q] -= o.first;
        for (int64_t b = 0; b < nb; b += step) per[q].push_back(make_int2(o.second, (int)b));
    }
    size_t longest = 0;
    for (const auto& p : per) longest = std::max(longest, p.size());
    std::vector<int2> units(longest * 8, make_int2(-1, 0));
    for (int q = 0; q < 8; ++q)
        for (size_t k = 0; k < per[q].size(); ++k) units[8 * k + q] = per[q][k];
    int rc;
    if ((rc = sqd_alloc(ctx, (void**)&sp->h_units, sizeof(int2) * (units.size() + 1), nullptr))) return rc;
    sp->h_bytes += (int64_t)(sizeof(int2) * (units.size() + 1));
    sp->bytes += (int64_t)(sizeof(int2) * (units.size() + 1));
    SQD_HIP(ctx, hipMemcpy(sp->h_units, units.data(), sizeof(int2) * units.size(), hipMemcpyHostToDevice));
    SQD_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(k_spmv_staged),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, ctx->max_lds));
    sp->h_nunits = (int)units.size();
    sp->h_list = most;
    sp->h_cap = (int)cap;
    sp->h_step = (int)step;
    return SQD_OK;
}

int sqd_store_h_impl(sqd_ctx* ctx, sqd_space* sp, int64_t* nnz_out) {
    int rc = sqd_ensure_diag(ctx, sp);
    if (rc) return rc;
    const spin_tables& A = sp->sp[0];
    const spin_tables& B = sp->sp[1];
    const int64_t na = A.n, nb = B.n, dim = sp->dim;
    if (dim >= 2147483647LL) return sqd_fail(ctx, SQD_E_LIMIT, "stored H needs dim < 2^31 (int32 columns)");
    // per-spin counts -> prefix sums of the closed-form row lengths
    std::vector<int> as(na + 1), ad(na + 1), bs(nb + 1), bd(nb + 1);
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    SQD_HIP(ctx, hipMemcpy(as.data(), A.s_off, sizeof(int) * (na + 1), hipMemcpyDeviceToHost));
    SQD_HIP(ctx, hipMemcpy(ad.data(), A.d_off, sizeof(int) * (na + 1), hipMemcpyDeviceToHost));
    SQD_HIP(ctx, hipMemcpy(bs.data(), B.s_off, sizeof(int) * (nb + 1), hipMemcpyDeviceToHost));
    SQD_HIP(ctx, hipMemcpy(bd.data(), B.d_off, sizeof(int) * (nb + 1), hipMemcpyDeviceToHost));
    std::vector<int64_t> PB(nb + 1), PSB(nb + 1), RA(na + 1);
    PB[0] = PSB[0] = 0;
    for (int64_t j = 0; j < nb; ++j) {
        PB[j + 1] = PB[j] + (bs[j + 1] - bs[j]) + (bd[j + 1] - bd[j]);
        PSB[j + 1] = PSB[j] + (bs[j + 1] - bs[j]);
    }
    RA[0] = 0;
    for (int64_t i = 0; i < na; ++i) {
        const int64_t sa = as[i + 1] - as[i], A1 = 1 + sa + (ad[i + 1] - ad[i]);
        RA[i + 1] = RA[i] + nb * A1 + PB[nb] + sa * PSB[nb];
    }
    const int64_t nnz = RA[na];
    // (re)allocate
    sqd_release_stored_h(sp);
    const size_t bytes = sizeof(int64_t) * (dim + 1) + (sizeof(int) + sizeof(double)) * (size_t)nnz;
    if ((rc = sqd_alloc(ctx, (void**)&sp->h_rowptr, sizeof(int64_t) * (dim + 1), nullptr)) ||
        (rc = sqd_alloc(ctx, (void**)&sp->h_col, sizeof(int) * (size_t)nnz, nullptr)) ||
        (rc = sqd_alloc(ctx, (void**)&sp->h_val, sizeof(double) * (size_t)nnz, nullptr))) {
        sqd_release_stored_h(sp);
        return sqd_fail(ctx, SQD_E_OOM, "stored H of " + std::to_string(nnz) + " elements (" +
                                            std::to_string(bytes) + " bytes) does not fit");
    }
    sp->h_bytes = (int64_t)bytes;
    sp->bytes += sp->h_bytes;
    int64_t *dRA = nullptr, *dPB = nullptr, *dPSB = nullptr;
    if ((rc = sqd_alloc(ctx, (void**)&dRA, sizeof(int64_t) * (na + 1), nullptr)) ||
        (rc = sqd_alloc(ctx, (void**)&dPB, sizeof(int64_t) * (nb + 1), nullptr)) ||
        (rc = sqd_alloc(ctx, (void**)&dPSB, sizeof(int64_t) * (nb + 1), nullptr))) {
        if (dRA) (void)hipFree(dRA);
        if (dPB) (void)hipFree(dPB);
        sqd_release_stored_h(sp);
        return rc;
    }
    hipError_t e = hipMemcpy(dRA, RA.data(), sizeof(int64_t) * (na + 1), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(dPB, PB.data(), sizeof(int64_t) * (nb + 1), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(dPSB, PSB.data(), sizeof(int64_t) * (nb + 1), hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_store_rowptr, dim3((unsigned)((dim + 256) / 256)), dim3(256), 0, ctx->stream, dRA, dPB,
                           dPSB, A.s_off, A.d_off, na, nb, sp->h_rowptr);
        store_args a{na, nb, A.s_off, A.s_pk, A.s_val64, A.d_off, A.d_nbr, A.d_val64,
                     B.s_off, B.s_pk, B.s_val64, B.d_off, B.d_nbr, B.d_val64,
                     A.str, B.str, sp->nw, ctx->jk64, ctx->eri, sp->norb, sp->diag, sp->h_rowptr, sp->h_col,
                     sp->h_val};
        hipLaunchKernelGGL(k_store_fill, dim3(fill_grid(dim)), dim3(256), 0, ctx->stream, a);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    }
    (void)hipFree(dRA);
    (void)hipFree(dPB);
    (void)hipFree(dPSB);
    if (e != hipSuccess) {
        sqd_release_stored_h(sp);
        return sqd_hip_fail(ctx, e, "stored H build");
    }
    sp->h_nnz = nnz;
    // row ranges of equal element counts for the eight XCDs (binary search
    // on the row pointer)
    sp->h_xcd_rows[0] = 0;
    sp->h_xcd_rows[8] = dim;
    for (int q = 1; q < 8; ++q) {
        const int64_t target = nnz * q / 8;
        int64_t lo = sp->h_xcd_rows[q - 1], hi = dim;   // first row whose start is >= target
        while (lo < hi) {
            const int64_t mid = lo + (hi - lo) / 2;
            int64_t v = 0;
            e = hipMemcpy(&v, sp->h_rowptr + mid, sizeof(int64_t), hipMemcpyDeviceToHost);
            if (e != hipSuccess) {
                sqd_release_stored_h(sp);
                return sqd_hip_fail(ctx, e, "stored H row ranges");
            }
            if (v < target) lo = mid + 1; else hi = mid;
        }
        sp->h_xcd_rows[q] = lo;
    }
    if ((rc = plan_staged(ctx, sp, as, ad, bs, PB, nnz))) {
        sqd_release_stored_h(sp);
        return rc;
    }
    sp->h_version = ctx->ham_version;
    if (nnz_out) *nnz_out = nnz;
    return SQD_OK;
}

int sqd_spmv_impl(sqd_ctx* ctx, sqd_space* sp, const double* x, double* y, const int* skip) {
    if (!sp->h_val || sp->h_version != ctx->ham_version)
        return sqd_fail(ctx, SQD_E_STATE, "no current stored H on this space (call sqd_store_hamiltonian)");
    prof_scope ps(ctx, "k_spmv");
    if (sp->h_nunits) {
        const spin_tables& A = sp->sp[0];
        const spin_tables& B = sp->sp[1];
        const size_t lds = (size_t)sp->h_cap * sizeof(double) + (size_t)sp->h_list * sizeof(int);
        staged_args a{B.n, A.s_off, A.d_off, A.d_nbr, B.s_off, B.d_off, B.d_nbr, A.s_pk, B.s_pk,
                      sp->h_rowptr, sp->h_val, x, y, sp->h_units, sp->h_cap, sp->h_step};
        hipLaunchKernelGGL(k_spmv_staged, dim3(sp->h_nunits), dim3(64 * kSpmvWaves), lds, ctx->stream, a, skip);
        SQD_HIP(ctx, hipGetLastError());
        return SQD_OK;
    }
    // eight workgroups of four rows per CU, a multiple of the 8 XCDs
    const int64_t want = std::max<int64_t>(1, (sp->dim + kRowsPerBlock - 1) / kRowsPerBlock);
    const unsigned grid = (unsigned)(8 * std::max<int64_t>(1, std::min<int64_t>(ctx->num_cu, (want + 7) / 8)));
    xcd_rows xr;
    for (int q = 0; q < 9; ++q) xr.r[q] = sp->h_xcd_rows[q];
    hipLaunchKernelGGL(k_spmv, dim3(grid), dim3(256), 0, ctx->stream, sp->h_rowptr, sp->h_col, sp->h_val, x, y, xr,
                       skip);
    SQD_HIP(ctx, hipGetLastError());
    return SQD_OK;
}

extern "C" {

int sqd_store_hamiltonian(sqd_ctx* ctx, const sqd_space* spc, int64_t* nnz_out) {
    if (!ctx || !spc) return SQD_E_INVALID_ARG;
    sqd_space* sp = const_cast<sqd_space*>(spc);
    if (sp->ctx != ctx) return sqd_fail(ctx, SQD_E_INVALID_ARG, "space belongs to another context");
    if (ctx->norb != sp->norb) return sqd_fail(ctx, SQD_E_STATE, "integrals changed norb since the space was built");
    SQD_HIP(ctx, hipSetDevice(ctx->device));
    return sqd_store_h_impl(ctx, sp, nnz_out);
}

int sqd_release_hamiltonian(sqd_ctx* ctx, const sqd_space* spc) {
    if (!ctx || !spc) return SQD_E_INVALID_ARG;
    sqd_space* sp = const_cast<sqd_space*>(spc);
    if (sp->ctx != ctx) return sqd_fail(ctx, SQD_E_INVALID_ARG, "space belongs to another context");
    SQD_HIP(ctx, hipSetDevice(ctx->device));
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    sqd_release_stored_h(sp);
    return SQD_OK;
}

int sqd_spmv(sqd_ctx* ctx, const sqd_space* spc, const double* c, double* sigma) {
    if (!ctx || !spc || !c || !sigma) return SQD_E_INVALID_ARG;
    sqd_space* sp = const_cast<sqd_space*>(spc);
    if (sp->ctx != ctx) return sqd_fail(ctx, SQD_E_INVALID_ARG, "space belongs to another context");
    if (ctx->norb != sp->norb) return sqd_fail(ctx, SQD_E_STATE, "integrals changed norb since the space was built");
    if (c == sigma) return sqd_fail(ctx, SQD_E_INVALID_ARG, "c and sigma must be distinct buffers");
    SQD_HIP(ctx, hipSetDevice(ctx->device));
    return sqd_spmv_impl(ctx, sp, c, sigma, nullptr);
}

int sqd_get_stored_hamiltonian(const sqd_space* spc, int64_t* rowptr, int32_t* cols, double* vals) {
    if (!spc || !rowptr) return SQD_E_INVALID_ARG;
    sqd_space* sp = const_cast<sqd_space*>(spc);
    sqd_ctx* ctx = sp->ctx;
    if (!ctx) return SQD_E_STATE;
    if (!sp->h_val || sp->h_version != ctx->ham_version)
        return sqd_fail(ctx, SQD_E_STATE, "no current stored H on this space");
    SQD_HIP(ctx, hipSetDevice(ctx->device));
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    SQD_HIP(ctx, hipMemcpy(rowptr, sp->h_rowptr, sizeof(int64_t) * (sp->dim + 1), hipMemcpyDeviceToHost));
    if (sp->h_nnz > 0) {
        if (!cols || !vals) return sqd_fail(ctx, SQD_E_INVALID_ARG, "null column or value pointer");
        SQD_HIP(ctx, hipMemcpy(cols, sp->h_col, sizeof(int) * (size_t)sp->h_nnz, hipMemcpyDeviceToHost));
        SQD_HIP(ctx, hipMemcpy(vals, sp->h_val, sizeof(double) * (size_t)sp->h_nnz, hipMemcpyDeviceToHost));
    }
    return SQD_OK;
}

}  // extern "C"
