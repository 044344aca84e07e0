// Excitation tables on the device (Sec. IV-A persistent configuration data and
// Sec. V-A flattened per-string excitation lists, offset + entries).
//
// For each string of a sorted set, the in-set single (i -> a) and double
// (i < j -> a < b) excitations are enumerated one wavefront per string, lanes
// over candidates; each candidate target is looked up by binary search in the
// sorted strings; the found entries are compacted into CSR rows, sorted inside
// each row by target index (canonical order) and packed.  The integral-
// dependent same-spin values are computed per entry afterwards, so that a new
// Hamiltonian does not rebuild the structure.
#include <algorithm>

#include <rocprim/device/device_radix_sort.hpp>

#include "slices.h"
#include "sqd_internal.h"

namespace {

// A string of NW 64-bit words (word q: orbitals 64q .. 64q+63) held in registers.
template <int NW>
struct wstr {
    uint64_t w[NW];
    __device__ __forceinline__ void flip(int k) { w[k >> 6] ^= 1ull << (k & 63); }
};

template <int NW>
__device__ __forceinline__ wstr<NW> load_str(const uint64_t* __restrict__ s, int64_t r) {
    wstr<NW> x;
#pragma unroll
    for (int q = 0; q < NW; ++q) x.w[q] = s[r * NW + q];
    return x;
}

// Binary search of the ascending strings (as NW-word integers, word NW-1 most
// significant) for key.
template <int NW>
__device__ __forceinline__ int64_t find_string(const uint64_t* __restrict__ s, int64_t n, const wstr<NW>& key) {
    int64_t lo = 0, hi = n - 1;
    while (lo <= hi) {
        const int64_t mid = (lo + hi) >> 1;
        int c = 0;
#pragma unroll
        for (int q = NW - 1; q >= 0; --q) {
            const uint64_t v = s[mid * NW + q];
            if (c == 0 && v != key.w[q]) c = v < key.w[q] ? -1 : 1;
        }
        if (c == 0) return mid;
        if (c < 0) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// Occupied / virtual orbital lists of string s, built by one wavefront (lane =
// orbital within a word) into LDS, each ascending.
template <int NW>
__device__ __forceinline__ void orbital_lists(const wstr<NW>& s, int norb, uint8_t* occ, uint8_t* vir) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    int no = 0, nv = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const int orb = 64 * q + lane;
        const bool in = orb < norb;
        const bool o = in && ((s.w[q] >> lane) & 1ull);
        const uint64_t bo = __ballot(o);
        const uint64_t bv = __ballot(in && !o);
        if (o) occ[no + __popcll(bo & below)] = (uint8_t)orb;
        if (in && !o) vir[nv + __popcll(bv & below)] = (uint8_t)orb;
        no += __popcll(bo);
        nv += __popcll(bv);
    }
}

// (-1)^(occupied orbitals below k) as 0 / 1
template <int NW>
__device__ __forceinline__ int parity_below(const wstr<NW>& s, int k) {
    int c = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const int lo = 64 * q;
        if (k >= lo + 64) c += __popcll(s.w[q]);
        else if (k > lo) c += __popcll(s.w[q] & ((~0ull) >> (64 - (k - lo))));
    }
    return c & 1;
}

// Sign of a+_a a_i applied to s (a_i first).
template <int NW>
__device__ __forceinline__ int single_sign(wstr<NW> s, int i, int a) {
    int p = parity_below(s, i);
    s.flip(i);
    p ^= parity_below(s, a);
    return p;  // 1 = negative
}

// Sign of a+_a a+_b a_j a_i applied to s (a_i, a_j, a+_b, a+_a in that order).
template <int NW>
__device__ __forceinline__ int double_sign(wstr<NW> s, int i, int j, int a, int b) {
    int p = parity_below(s, i);
    s.flip(i);
    p ^= parity_below(s, j);
    s.flip(j);
    p ^= parity_below(s, b);
    s.flip(b);
    p ^= parity_below(s, a);
    return p;
}

// Waves per block and LDS slots for the (x < y) orbital pairs of one string:
// C(64, 2) for one-word strings, C(128, 2) (one wave per block) for two.
template <int NW> struct enum_shape;
template <> struct enum_shape<1> { static constexpr int kWaves = 4, kPairs = 2016; };
template <> struct enum_shape<2> { static constexpr int kWaves = 1, kPairs = 8128; };

// KIND 0: singles, 1: doubles.  MODE 0: count, 1: fill.
template <int KIND, int MODE, int NW>
__global__ void __launch_bounds__(64 * enum_shape<NW>::kWaves)
k_enum(const uint64_t* __restrict__ str, int64_t n, int norb, int nel,
       int* __restrict__ counts, const int* __restrict__ off,
       uint64_t* __restrict__ keys, uint32_t* __restrict__ payload) {
    constexpr int WPB = enum_shape<NW>::kWaves, NP = enum_shape<NW>::kPairs;
    __shared__ uint8_t s_occ[WPB][64 * NW];
    __shared__ uint8_t s_vir[WPB][64 * NW];
    __shared__ uint16_t s_op[WPB][KIND == 1 ? NP : 1];
    __shared__ uint16_t s_vp[WPB][KIND == 1 ? NP : 1];
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * WPB + w;
    // every wave reaches both barriers; waves past the end do no work
    const bool valid = row < n;
    wstr<NW> s;
#pragma unroll
    for (int q = 0; q < NW; ++q) s.w[q] = 0ull;
    if (valid) s = load_str<NW>(str, row);
    const int nvir = norb - nel;
    uint8_t* occ = s_occ[w];
    uint8_t* vir = s_vir[w];
    if (valid) orbital_lists<NW>(s, norb, occ, vir);
    int npo = 0, npv = 0;
    if (KIND == 1) {
        npo = nel * (nel - 1) / 2;
        npv = nvir * (nvir - 1) / 2;
    }
    __syncthreads();
    if (KIND == 1 && valid) {
        for (int k = lane; k < npo; k += 64) {
            // decode k -> (x < y) in row-major upper-triangle order
            int x = 0, rem = k;
            while (rem >= nel - 1 - x) { rem -= nel - 1 - x; ++x; }
            s_op[w][k] = (uint16_t)(occ[x] | (occ[x + 1 + rem] << 8));
        }
        for (int k = lane; k < npv; k += 64) {
            int x = 0, rem = k;
            while (rem >= nvir - 1 - x) { rem -= nvir - 1 - x; ++x; }
            s_vp[w][k] = (uint16_t)(vir[x] | (vir[x + 1 + rem] << 8));
        }
    }
    __syncthreads();
    if (!valid) return;
    const int64_t ncand = (KIND == 0) ? (int64_t)nel * nvir : (int64_t)npo * npv;
    int found = 0;
    const int base = (MODE == 1) ? off[row] : 0;
    for (int64_t c0 = 0; c0 < ncand; c0 += 64) {
        const int64_t c = c0 + lane;
        int64_t tgt = -1;
        int i = 0, j = 0, a = 0, b = 0;
        if (c < ncand) {
            wstr<NW> t = s;
            if (KIND == 0) {
                i = occ[c / nvir];
                a = vir[c % nvir];
                t.flip(i);
                t.flip(a);
            } else {
                const uint16_t op = s_op[w][c / npv];
                const uint16_t vp = s_vp[w][c % npv];
                i = op & 0xFF; j = op >> 8; a = vp & 0xFF; b = vp >> 8;
                t.flip(i);
                t.flip(j);
                t.flip(a);
                t.flip(b);
            }
            tgt = find_string<NW>(str, n, t);
        }
        const bool hit = tgt >= 0;
        const uint64_t m = __ballot(hit);
        if (MODE == 1 && hit) {
            const uint64_t below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
            const int pos = base + found + __popcll(m & below);
            keys[pos] = ((uint64_t)row << 17) | (uint64_t)tgt;
            uint32_t neg = (KIND == 0) ? (uint32_t)single_sign<NW>(s, i, a)
                                       : (uint32_t)double_sign<NW>(s, i, j, a, b);
            payload[pos] = (uint32_t)i | ((uint32_t)j << 7) | ((uint32_t)a << 14) |
                           ((uint32_t)b << 21) | (neg << 31);
        }
        found += __popcll(m);
    }
    if (MODE == 0 && lane == 0) counts[row] = found;
}

// Exclusive scan of n ints into off[0..n] with off[n] = total (one block).
__global__ void __launch_bounds__(1024) k_scan(const int* __restrict__ in, int64_t n, int* __restrict__ out,
                                               long long* __restrict__ total) {
    __shared__ long long part[1024];
    const int t = threadIdx.x;
    const int64_t chunk = (n + 1023) / 1024;
    const int64_t b = t * chunk, e = (b + chunk < n) ? b + chunk : n;
    long long s = 0;
    for (int64_t k = b; k < e; ++k) s += in[k];
    part[t] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        long long v = (t >= o) ? part[t - o] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    long long run = part[t] - s;
    for (int64_t k = b; k < e; ++k) {
        out[k] = (int)run;
        run += in[k];
    }
    if (t == 1023) {
        out[n] = (int)part[1023];
        *total = part[1023];
    }
}

template <int KIND>
__global__ void k_pack(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ payload,
                       int64_t nnz, int norb, uint64_t* __restrict__ ent, uint32_t* __restrict__ pk,
                       int* __restrict__ nbr) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const uint64_t tgt = keys[e] & SQD_NBR_MASK;
    const uint32_t p = payload[e];
    const uint64_t i = p & 127, j = (p >> 7) & 127, a = (p >> 14) & 127, b = (p >> 21) & 127;
    const uint64_t neg = p >> 31;
    if (KIND == 0) {
        ent[e] = tgt | (i << 32) | (a << 39) | (neg << 63);
        const uint32_t pair = (uint32_t)(a * norb + i);
        pk[e] = (uint32_t)tgt | (pair << SQD_PAIR_SHIFT) | ((uint32_t)neg << 31);
    } else {
        ent[e] = tgt | (i << 32) | (j << 39) | (a << 46) | (b << 53) | (neg << 63);
        nbr[e] = (int)tgt;
    }
}

// Fill a sliced same-spin table (layout: sell_table): column c of a lane that
// is the i-th of g = 2^split lanes of its row takes CSR entry c * g + i, the
// columns of the singles' blocks from the singles, the others from the doubles.
template <typename T>
__global__ void __launch_bounds__(256) k_sell_fill(sell_table<T> L, int64_t n, const int* __restrict__ s_off,
                                                   const uint32_t* __restrict__ s_pk, const int* __restrict__ d_off,
                                                   const int* __restrict__ d_nbr) {
    const int sl = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int k = L.split ? L.split[sl] : 0;
    const int sub = lane & ((1 << k) - 1);
    const int r = L.perm[sl * 64 + lane - sub];
    const int b0 = L.blk[sl], nb = L.blk[sl + 1] - b0, sb = L.s_blk[sl];
    const int s0 = r < n ? s_off[r] : 0, s1 = r < n ? s_off[r + 1] : 0;
    const int d0 = r < n ? d_off[r] : 0, d1 = r < n ? d_off[r + 1] : 0;
    for (int b = threadIdx.x >> 6; b < nb; b += blockDim.x >> 6) {
        const bool single = b < sb;
        const int from = single ? s0 : d0, to = single ? s1 : d1;
        const int64_t pos = (int64_t)(b0 + b) * 256 + lane * 4;
        for (int q = 0; q < 4; ++q) {
            const int e = from + (((single ? b : b - sb) * 4 + q) << k) + sub;
            const bool in = e < to;
            L.ent[pos + q] = !in ? (uint32_t)n : single ? s_pk[e] : (uint32_t)d_nbr[e];
            L.csr[pos + q] = !in ? -1 : single ? e : -2 - e;
        }
    }
}

// Fill the alpha-beta table (layout: ab_table), one workgroup per slice.  An
// entry's place in its row is the number of the row's singles with a smaller
// pair (the pairs of one row are distinct); the place p of a row over g lanes
// is column p / g of its lane p % g.
__global__ void __launch_bounds__(256) k_ab_fill(ab_table L, int64_t n, const int* __restrict__ off,
                                                 const uint32_t* __restrict__ pk) {
    const int sl = blockIdx.x;
    const int b0 = L.blk[sl], nb = L.blk[sl + 1] - b0;
    uint32_t* out = L.ent + (int64_t)b0 * 256;
    for (int q = threadIdx.x; q < nb * 256; q += 256) out[q] = (uint32_t)n;   // padding: zero column, pair 0
    __syncthreads();
    auto pair = [](uint32_t x) { return (x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK; };
    const int k = L.split ? L.split[sl] : 0;
    const int wave = threadIdx.x >> 6;
    for (int row = wave; row < (64 >> k); row += 4) {
        const int r = L.perm[L.slot[sl] + row];
        if (r >= n) continue;
        for (int e = off[r] + (threadIdx.x & 63); e < off[r + 1]; e += 64) {
            const uint32_t x = pk[e];
            int place = 0;
            for (int f = off[r]; f < off[r + 1]; ++f) place += pair(pk[f]) < pair(x);
            const int col = place >> k, lane = (row << k) + (place & ((1 << k) - 1));
            out[(col >> 2) * 256 + lane * 4 + (col & 3)] = x;
        }
    }
}

// ---- integral-dependent values ----

// e_same[r] = sum_{i in s} h_ii + 1/2 sum_{i,j in s} [(ii|jj) - (ij|ji)]
__global__ void k_same_energy(const uint64_t* __restrict__ str, int nw, int64_t n, int norb,
                              const double* __restrict__ h, const double* __restrict__ eri,
                              double* __restrict__ e) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const uint64_t* s = str + r * nw;
    const int64_t n2 = (int64_t)norb * norb;
    double acc = 0.0;
    str_for_each(s, nw, [&](int i) {
        acc += h[i * norb + i];
        str_for_each(s, nw, [&](int j) {
            acc += 0.5 * (eri[(int64_t)(i * norb + i) * n2 + j * norb + j] -
                          eri[(int64_t)(i * norb + j) * n2 + j * norb + i]);
        });
    });
    e[r] = acc;
}

// single (row string s, i -> a in the neighbour): sign * [h_ai + sum_{k in s}((ai|kk) - (ak|ki))]
__global__ void k_single_values(const uint64_t* __restrict__ str, int nw, const int* __restrict__ off, int64_t n,
                                const uint64_t* __restrict__ ent, int norb,
                                const double* __restrict__ h, const double* __restrict__ eri,
                                double* __restrict__ v64, float* __restrict__ v32) {
    const int64_t r = (int64_t)blockIdx.x;
    if (r >= n) return;
    const uint64_t* s = str + r * nw;
    const int64_t n2 = (int64_t)norb * norb;
    for (int e = off[r] + threadIdx.x; e < off[r + 1]; e += blockDim.x) {
        const uint64_t x = ent[e];
        const int i = SQD_ENT_ORB(x, 0), a = SQD_ENT_ORB(x, 1);
        double acc = h[a * norb + i];
        str_for_each(s, nw, [&](int k) {
            acc += eri[(int64_t)(a * norb + i) * n2 + k * norb + k] -
                   eri[(int64_t)(a * norb + k) * n2 + k * norb + i];
        });
        if (x >> 63) acc = -acc;
        v64[e] = acc;
        v32[e] = (float)acc;
    }
}

// double (i < j -> a < b): sign * [(ai|bj) - (aj|bi)]
__global__ void k_double_values(const uint64_t* __restrict__ ent, int64_t nnz, int norb,
                                const double* __restrict__ eri, double* __restrict__ v64,
                                float* __restrict__ v32) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const uint64_t x = ent[e];
    const int i = SQD_ENT_ORB(x, 0), j = SQD_ENT_ORB(x, 1);
    const int a = SQD_ENT_ORB(x, 2), b = SQD_ENT_ORB(x, 3);
    const int64_t n2 = (int64_t)norb * norb;
    double v = eri[(int64_t)(a * norb + i) * n2 + b * norb + j] - eri[(int64_t)(a * norb + j) * n2 + b * norb + i];
    if (x >> 63) v = -v;
    v64[e] = v;
    v32[e] = (float)v;
}

template <typename T>
__global__ void k_sell_values(const int* __restrict__ csr, int64_t m, const T* __restrict__ s_val,
                              const T* __restrict__ d_val, T* __restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m) return;
    const int e = csr[k];
    const T v = e >= 0 ? s_val[e] : e == -1 ? (T)0 : d_val[-2 - e];
    // FP64: the four values of a lane as two planes of 16-byte pieces
    const int64_t q = k & 3, lane = (k >> 2) & 63;
    out[sizeof(T) == 8 ? (k & ~(int64_t)255) + 128 * (q >> 1) + 2 * lane + (q & 1) : k] = v;
}

// ws[s * norb2 + pq] = sum over occupied k of s (ascending) of jk[k * norb2 + pq]
template <typename T>
__global__ void k_cross_table(const uint64_t* __restrict__ str, int nw, int64_t n, int norb,
                              const T* __restrict__ jk, T* __restrict__ ws) {
    const int norb2 = norb * norb;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * norb2) return;
    const int64_t s = idx / norb2;
    const int pq = (int)(idx - s * norb2);
    T acc = (T)0;
    str_for_each(str + s * nw, nw, [&](int k) { acc += jk[(int64_t)k * norb2 + pq]; });
    ws[idx] = acc;
}

inline unsigned nblocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// Sort (key, value) pairs with rocPRIM's device radix sort; end_bit bits of key used.
template <typename K, typename V>
int radix_sort(sqd_ctx* ctx, K* keys, V* vals, int64_t n, int end_bit) {
    if (n <= 1) return SQD_OK;
    K* k2 = nullptr; V* v2 = nullptr; void* tmp = nullptr; size_t tmpb = 0;
    SQD_HIP(ctx, hipMalloc(&k2, sizeof(K) * n));
    SQD_HIP(ctx, hipMalloc(&v2, sizeof(V) * n));
    SQD_HIP(ctx, rocprim::radix_sort_pairs(nullptr, tmpb, keys, k2, vals, v2, (size_t)n, 0u, (unsigned)end_bit,
                                           ctx->stream));
    SQD_HIP(ctx, hipMalloc(&tmp, tmpb > 0 ? tmpb : 1));
    SQD_HIP(ctx, rocprim::radix_sort_pairs(tmp, tmpb, keys, k2, vals, v2, (size_t)n, 0u, (unsigned)end_bit, ctx->stream));
    SQD_HIP(ctx, hipMemcpyAsync(keys, k2, sizeof(K) * n, hipMemcpyDeviceToDevice, ctx->stream));
    SQD_HIP(ctx, hipMemcpyAsync(vals, v2, sizeof(V) * n, hipMemcpyDeviceToDevice, ctx->stream));
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    hipFree(k2); hipFree(v2); hipFree(tmp);
    return SQD_OK;
}

// Build one kind (singles or doubles) of canonical CSR table.
template <int KIND>
int build_kind(sqd_ctx* ctx, sqd_space* sp, spin_tables& t, int** off_out, uint64_t** ent_out,
               uint32_t** pk_out, int** nbr_out, int64_t* nnz_out) {
    const int norb = sp->norb;
    int* counts = nullptr;
    long long* dtot = nullptr;
    SQD_HIP(ctx, hipMalloc(&counts, sizeof(int) * (t.n + 1)));
    SQD_HIP(ctx, hipMalloc(&dtot, sizeof(long long)));
    int* off = nullptr;
    int rc = sqd_alloc(ctx, (void**)&off, sizeof(int) * (t.n + 1), &sp->bytes);
    if (rc) return rc;
    uint64_t* keys_ = nullptr;
    uint32_t* pay_ = nullptr;
    auto launch_enum = [&](int mode) {
        const int wpb = t.nw == 1 ? enum_shape<1>::kWaves : enum_shape<2>::kWaves;
        const dim3 grid(nblocks(t.n, wpb)), block(64 * wpb);
        int* cnt = mode == 0 ? counts : nullptr;
        const int* of = mode == 0 ? nullptr : off;
        uint64_t* ky = mode == 0 ? nullptr : keys_;
        uint32_t* py = mode == 0 ? nullptr : pay_;
        if (t.nw == 1) {
            if (mode == 0) hipLaunchKernelGGL((k_enum<KIND, 0, 1>), grid, block, 0, ctx->stream, t.str, t.n, norb, t.nel, cnt, of, ky, py);
            else hipLaunchKernelGGL((k_enum<KIND, 1, 1>), grid, block, 0, ctx->stream, t.str, t.n, norb, t.nel, cnt, of, ky, py);
        } else {
            if (mode == 0) hipLaunchKernelGGL((k_enum<KIND, 0, 2>), grid, block, 0, ctx->stream, t.str, t.n, norb, t.nel, cnt, of, ky, py);
            else hipLaunchKernelGGL((k_enum<KIND, 1, 2>), grid, block, 0, ctx->stream, t.str, t.n, norb, t.nel, cnt, of, ky, py);
        }
    };
    launch_enum(0);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, ctx->stream, counts, t.n, off, dtot);
    long long total = 0;
    SQD_HIP(ctx, hipMemcpyAsync(&total, dtot, sizeof(long long), hipMemcpyDeviceToHost, ctx->stream));
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    SQD_HIP(ctx, hipGetLastError());
    if (total >= (1LL << 31) - 64LL * 1024) {
        hipFree(counts); hipFree(dtot);
        return sqd_fail(ctx, SQD_E_LIMIT, "excitation table exceeds 2^31 entries");
    }
    const int64_t nnz = total;
    uint64_t* keys = nullptr; uint32_t* pay = nullptr;
    SQD_HIP(ctx, hipMalloc(&keys, sizeof(uint64_t) * (nnz + 1)));
    SQD_HIP(ctx, hipMalloc(&pay, sizeof(uint32_t) * (nnz + 1)));
    keys_ = keys;
    pay_ = pay;
    launch_enum(1);
    SQD_HIP(ctx, hipGetLastError());
    rc = radix_sort(ctx, keys, pay, nnz, 34);   // (row << 17 | target): rows, then targets
    if (rc) return rc;
    uint64_t* ent = nullptr; uint32_t* pk = nullptr; int* nbr = nullptr;
    if ((rc = sqd_alloc(ctx, (void**)&ent, sizeof(uint64_t) * (nnz + 1), &sp->bytes))) return rc;
    if (KIND == 0) {
        if ((rc = sqd_alloc(ctx, (void**)&pk, sizeof(uint32_t) * (nnz + 1), &sp->bytes))) return rc;
    } else {
        if ((rc = sqd_alloc(ctx, (void**)&nbr, sizeof(int) * (nnz + 1), &sp->bytes))) return rc;
    }
    if (nnz > 0)
        hipLaunchKernelGGL((k_pack<KIND>), dim3(nblocks(nnz, 256)), dim3(256), 0, ctx->stream,
                           keys, pay, nnz, norb, ent, pk, nbr);
    SQD_HIP(ctx, hipGetLastError());
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    hipFree(keys); hipFree(pay); hipFree(counts); hipFree(dtot);
    *off_out = off; *ent_out = ent; *pk_out = pk; *nbr_out = nbr; *nnz_out = nnz;
    return SQD_OK;
}

// Slices of a sliced table over rows sorted by length, the longest remaining
// row setting the lanes per row of the next slice; then dealt into bins.
struct sell_plan {
    std::vector<int> perm, split, blk{0}, s_blk, bin;
};
sell_plan plan_slices(const std::vector<int>& rows, const int* s_off, const int* d_off, int cap) {
    struct slice { int split, s_blk, nblk; std::vector<int> perm; };
    std::vector<slice> sl;
    const int n = (int)rows.size();
    auto cols = [](const int* off, int r, int k) { return (off[r + 1] - off[r] + (1 << k) - 1) >> k; };
    for (int at = 0; at < n;) {
        slice x;
        x.split = split_of(cols(s_off, rows[at], 0) + cols(d_off, rows[at], 0), cap);
        int ms = 0, md = 0;
        for (int lane = 0; lane < 64; ++lane) {
            const bool first = (lane & ((1 << x.split) - 1)) == 0;
            const int r = first && at < n ? rows[at++] : n;
            x.perm.push_back(r);
            if (r == n) continue;
            ms = std::max(ms, cols(s_off, r, x.split));
            md = std::max(md, cols(d_off, r, x.split));
        }
        x.s_blk = (ms + 3) / 4;
        x.nblk = (x.s_blk + (md + 3) / 4 + 1) & ~1;
        sl.push_back(std::move(x));
    }
    // a single costs about two doubles (two LDS columns), a slice about one block
    std::vector<int> cost;
    for (const slice& x : sl) cost.push_back(x.nblk + x.s_blk + 1);
    const auto in = deal_bins(cost);
    sell_plan p;
    for (int q = 0; q < kBins; ++q) {
        p.bin.push_back((int)p.split.size());
        for (int k : in[q]) {
            p.perm.insert(p.perm.end(), sl[k].perm.begin(), sl[k].perm.end());
            p.split.push_back(sl[k].split);
            p.s_blk.push_back(sl[k].s_blk);
            p.blk.push_back(p.blk.back() + sl[k].nblk);
        }
    }
    p.bin.push_back((int)p.split.size());
    for (int q = 0; q <= kBins; ++q) p.bin.push_back(p.blk[p.bin[q]]);
    return p;
}

// Sizes of a sliced table from its plan, and its arrays among those to be allocated.
constexpr int64_t kMaxSlots = (1LL << 31) - 1;
template <typename T>
bool size_sell(const sell_plan& p, sell_table<T>& L, array_list& arrays) {
    L.nslices = (int)p.split.size();
    L.slots = (int64_t)p.blk.back() * 256;
    arrays.insert(arrays.end(), {{(void**)&L.ent, sizeof(uint32_t) * (L.slots + 256)},
                                 {(void**)&L.csr, sizeof(int) * (L.slots + 256)},
                                 {(void**)&L.val, sizeof(T) * (L.slots + 256)}});
    return L.slots <= kMaxSlots;
}
bool size_ab(const ab_plan& p, ab_table& L, array_list& arrays) {
    L.nslices = (int)p.split.size();
    L.nslots = (int64_t)p.perm.size();
    L.nblk = p.blk.back();
    arrays.push_back({(void**)&L.ent, sizeof(uint32_t) * (L.nblk + 2) * 256});
    return L.nblk * 256 <= kMaxSlots;
}

template <typename T>
void sell_values(sqd_ctx* ctx, const sell_table<T>& L, const T* s_val, const T* d_val) {
    if (L.slots > 0)
        hipLaunchKernelGGL(k_sell_values<T>, dim3(nblocks(L.slots, 256)), dim3(256), 0, ctx->stream, L.csr, L.slots,
                           s_val, d_val, L.val);
}

}  // namespace

int sqd_build_spin_tables(sqd_ctx* ctx, sqd_space* sp, int spin, const uint64_t* host_str, int64_t n, int nel) {
    spin_tables& t = sp->sp[spin];
    t.n = n;
    t.nel = nel;
    t.nw = sp->nw;
    int rc = sqd_alloc(ctx, (void**)&t.str, sizeof(uint64_t) * (n > 0 ? n : 1) * t.nw, &sp->bytes);
    if (rc) return rc;
    SQD_HIP(ctx, hipMemcpyAsync(t.str, host_str, sizeof(uint64_t) * n * t.nw, hipMemcpyHostToDevice, ctx->stream));
    int* dummy_nbr = nullptr; uint32_t* dummy_pk = nullptr;
    if ((rc = build_kind<0>(ctx, sp, t, &t.s_off, &t.s_ent, &t.s_pk, &dummy_nbr, &t.nnz_s))) return rc;
    if ((rc = build_kind<1>(ctx, sp, t, &t.d_off, &t.d_ent, &dummy_pk, &t.d_nbr, &t.nnz_d))) return rc;

    // sliced layouts, planned on the host from the row lengths: same-spin rows
    // by singles + doubles, alpha-beta rows by singles
    t.str_host.assign(host_str, host_str + n * t.nw);
    std::vector<int>& so = t.s_off_host;
    so.resize(n + 1);
    std::vector<int> dof(n + 1), len(n);
    SQD_HIP(ctx, hipMemcpy(so.data(), t.s_off, sizeof(int) * (n + 1), hipMemcpyDeviceToHost));
    SQD_HIP(ctx, hipMemcpy(dof.data(), t.d_off, sizeof(int) * (n + 1), hipMemcpyDeviceToHost));
    t.max_singles = t.max_doubles = 0;
    for (int64_t r = 0; r < n; ++r) {
        len[r] = so[r + 1] - so[r];
        t.max_singles = std::max(t.max_singles, len[r]);
        t.max_doubles = std::max(t.max_doubles, dof[r + 1] - dof[r]);
    }
    constexpr int kWhole = 1 << 30;
    const std::vector<int> rows_s = rows_longest_first(len);
    const ab_plan a32 = plan_ab(rows_s, so.data(), kWhole);
    const ab_plan a64 = plan_ab(rows_s, so.data(), split_cap(t.nnz_s, 8));
    for (int64_t r = 0; r < n; ++r) len[r] += dof[r + 1] - dof[r];
    const std::vector<int> rows = rows_longest_first(len);
    const sell_plan p32 = plan_slices(rows, so.data(), dof.data(), kWhole);
    const sell_plan p64 = plan_slices(rows, so.data(), dof.data(), split_cap(t.nnz_s + t.nnz_d, 12));
    {
        const std::pair<const std::vector<int>*, const int**> parts[] = {
            {&p32.perm, &t.ss32.perm}, {&p32.blk, &t.ss32.blk},   {&p32.s_blk, &t.ss32.s_blk}, {&p32.bin, &t.ss32.bin},
            {&p64.perm, &t.ss64.perm}, {&p64.blk, &t.ss64.blk},   {&p64.s_blk, &t.ss64.s_blk}, {&p64.bin, &t.ss64.bin},
            {&p64.split, &t.ss64.split}, {&a32.perm, &t.ab32.perm}, {&a32.blk, &t.ab32.blk},   {&a32.cols, &t.ab32.cols},
            {&a32.slot, &t.ab32.slot}, {&a32.bin, &t.ab32.bin},   {&a32.order, &t.ab32.order}, {&a64.perm, &t.ab64.perm},
            {&a64.blk, &t.ab64.blk},   {&a64.cols, &t.ab64.cols}, {&a64.slot, &t.ab64.slot},   {&a64.bin, &t.ab64.bin},
            {&a64.split, &t.ab64.split}, {&rows_s, &t.by_singles}};
        std::vector<int> all;
        for (const auto& q : parts) all.insert(all.end(), q.first->begin(), q.first->end());
        // the sliced tables, their plans and the values (CSR order)
        int* index = nullptr;
        array_list arrays = {{(void**)&index, sizeof(int) * (all.size() + 1)},
                             {(void**)&t.s_val64, sizeof(double) * (t.nnz_s + 1)},
                             {(void**)&t.s_val32, sizeof(float) * (t.nnz_s + 1)},
                             {(void**)&t.d_val64, sizeof(double) * (t.nnz_d + 1)},
                             {(void**)&t.d_val32, sizeof(float) * (t.nnz_d + 1)},
                             {(void**)&t.e_same, sizeof(double) * (n + 1)}};
        const bool fits[] = {size_sell(p32, t.ss32, arrays), size_sell(p64, t.ss64, arrays),
                             size_ab(a32, t.ab32, arrays), size_ab(a64, t.ab64, arrays)};
        for (bool f : fits)
            if (!f) return sqd_fail(ctx, SQD_E_LIMIT, "sliced table exceeds 2^31 slots");
        if ((rc = alloc_tables(ctx, arrays, t.table_mem, &sp->bytes))) return rc;
        SQD_HIP(ctx, hipMemcpy(index, all.data(), sizeof(int) * all.size(), hipMemcpyHostToDevice));
        const int* at = index;
        for (const auto& q : parts) {
            *q.second = at;
            at += q.first->size();
        }
    }
    hipLaunchKernelGGL(k_sell_fill<float>, dim3(t.ss32.nslices), dim3(256), 0, ctx->stream, t.ss32, n, t.s_off, t.s_pk,
                       t.d_off, t.d_nbr);
    hipLaunchKernelGGL(k_sell_fill<double>, dim3(t.ss64.nslices), dim3(256), 0, ctx->stream, t.ss64, n, t.s_off, t.s_pk,
                       t.d_off, t.d_nbr);
    hipLaunchKernelGGL(k_ab_fill, dim3(t.ab32.nslices), dim3(256), 0, ctx->stream, t.ab32, n, t.s_off, t.s_pk);
    hipLaunchKernelGGL(k_ab_fill, dim3(t.ab64.nslices), dim3(256), 0, ctx->stream, t.ab64, n, t.s_off, t.s_pk);
    SQD_HIP(ctx, hipGetLastError());
    return SQD_OK;
}

int sqd_ensure_split32(sqd_ctx* ctx, sqd_space* sp) {
    int rc = sqd_build_values(ctx, sp);
    if (rc) return rc;
    for (int spin = 0; spin < 2; ++spin) {
        spin_tables& t = sp->sp[spin];
        if (t.alias) {
            t.split32 = sp->sp[0].split32;
            continue;
        }
        if (t.split32_version == ctx->ham_version) continue;
        sell_table<float>& L = t.split32;
        const sell_table<double>& D = t.ss64;
        if (!L.val && (rc = sqd_alloc(ctx, (void**)&L.val, sizeof(float) * (D.slots + 256), &sp->bytes))) return rc;
        L.nslices = D.nslices;
        L.perm = D.perm, L.split = D.split, L.blk = D.blk, L.s_blk = D.s_blk, L.bin = D.bin;
        L.slots = D.slots;
        L.ent = D.ent, L.csr = D.csr;
        sell_values(ctx, L, t.s_val32, t.d_val32);
        SQD_HIP(ctx, hipGetLastError());
        t.split32_version = ctx->ham_version;
    }
    return SQD_OK;
}

int sqd_host_singles(sqd_ctx* ctx, spin_tables& t) {
    if ((int64_t)t.s_pk_host.size() == t.nnz_s) return SQD_OK;
    std::vector<uint32_t> pk(t.nnz_s);
    SQD_HIP(ctx, sqd_copy_now(ctx, pk.data(), t.s_pk, sizeof(uint32_t) * t.nnz_s, hipMemcpyDeviceToHost));
    t.s_pk_host.swap(pk);
    return SQD_OK;
}

int sqd_build_values(sqd_ctx* ctx, sqd_space* sp) {
    if (sp->values_version == ctx->ham_version) return SQD_OK;
    const int norb = sp->norb;
    for (int spin = 0; spin < 2; ++spin) {
        spin_tables& t = sp->sp[spin];
        if (t.alias) continue;
        if (t.n > 0) {
            hipLaunchKernelGGL(k_same_energy, dim3(nblocks(t.n, 128)), dim3(128), 0, ctx->stream, t.str, t.nw, t.n,
                               norb, ctx->h, ctx->eri, t.e_same);
            hipLaunchKernelGGL(k_single_values, dim3((unsigned)t.n), dim3(64), 0, ctx->stream, t.str, t.nw, t.s_off,
                               t.n, t.s_ent, norb, ctx->h, ctx->eri, t.s_val64, t.s_val32);
        }
        if (t.nnz_d > 0)
            hipLaunchKernelGGL(k_double_values, dim3(nblocks(t.nnz_d, 256)), dim3(256), 0, ctx->stream, t.d_ent,
                               t.nnz_d, norb, ctx->eri, t.d_val64, t.d_val32);
        sell_values(ctx, t.ss64, t.s_val64, t.d_val64);
        sell_values(ctx, t.ss32, t.s_val32, t.d_val32);
        const int64_t m = t.n * (int64_t)norb * norb;
        if (t.ws64)
            hipLaunchKernelGGL(k_cross_table<double>, dim3(nblocks(m, 256)), dim3(256), 0, ctx->stream, t.str, t.nw,
                               t.n, norb, ctx->jk64, t.ws64);
        if (t.ws32)
            hipLaunchKernelGGL(k_cross_table<float>, dim3(nblocks(m, 256)), dim3(256), 0, ctx->stream, t.str, t.nw,
                               t.n, norb, ctx->jk32, t.ws32);
        SQD_HIP(ctx, hipGetLastError());
    }
    SQD_HIP(ctx, hipStreamSynchronize(ctx->stream));
    sp->values_version = ctx->ham_version;
    return SQD_OK;
}

void sqd_free_spin_tables(spin_tables* t) {
    if (t->alias) { *t = spin_tables(); return; }
    sqd_free_window_tables(t);
    for (void* p : t->table_mem) (void)hipFree(p);
    void* ptrs[] = {t->split32.val, t->str, t->s_off, t->s_ent, t->d_off, t->d_ent, t->s_pk, t->d_nbr};
    for (void* p : ptrs)
        if (p) hipFree(p);
    *t = spin_tables();
}
