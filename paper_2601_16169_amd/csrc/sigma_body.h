// Device bodies of the sigma kernels, shared by the single-space launches
// (sigma.hip) and the launches over many spaces (batched.hip).  Each body
// processes one work unit (a block index of its own launch shape) of one
// space described by an argument struct.
#pragma once

#include <type_traits>

#include "sqd_internal.h"

// LDS layout of R values per column c (staged rows of C, or rows of the
// cross-spin table): column c owns R * sizeof(T) bytes at c * R.  Lanes read
// whole columns at random c in 16-byte pieces; when a column is two or four
// 16-byte pieces, the pieces are stored XOR-permuted by bits of c above those
// that already select the bank group, so that for any piece index the 64
// lanes spread over all LDS banks instead of a quarter or half of them.
template <typename T, int R>
struct lds_cols {
    static constexpr int kE = 16 / (int)sizeof(T);                 // elements per 16-byte piece
    static constexpr int kU = (R * (int)sizeof(T)) / 16;           // pieces per column (0: under 16 bytes)
    static constexpr bool kSwz = (kU == 2 || kU == 4);
    __device__ static __forceinline__ int swz(int64_t c) {
        return kU == 4 ? (int)((c >> 2) & 3) : (int)((c >> 3) & 1);
    }
    __device__ static __forceinline__ int64_t idx(int64_t c, int r) {
        if constexpr (kSwz) return c * R + (((r / kE) ^ swz(c)) * kE) + (r % kE);
        else return c * R + r;
    }
    __device__ static __forceinline__ void load(const T* __restrict__ xs, int64_t c, T (&v)[R]) {
        if constexpr (kSwz) {
            const int f = swz(c);
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const T* src = xs + c * R + ((u ^ f) * kE);
#pragma unroll
                for (int w = 0; w < kE; ++w) v[u * kE + w] = src[w];
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = xs[c * R + r];
        }
    }
};

// Stage R rows of length ncols (row r starts at rows[r], or zeros when null;
// rows[0] is never null) into LDS in the lds_cols<T, R> layout; column ncols
// is zero.  Each thread takes four columns per pass and issues all 4R loads
// before any store: null rows read row 0 and are zeroed by a select, columns
// past the end read the last column and are not stored, so no load sits
// behind a branch.
template <typename T, int R>
__device__ __forceinline__ void stage_rows(T* __restrict__ xs, const T* const (&rows)[R], int ncols) {
    using L = lds_cols<T, R>;
    constexpr int kCols = 4;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const T* src[R];
    bool ok[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        ok[r] = rows[r] != nullptr;
        src[r] = ok[r] ? rows[r] : rows[0];
    }
    for (int col0 = tid; col0 < ncols; col0 += kCols * nthr) {
        T v[kCols][R];
#pragma unroll
        for (int u = 0; u < kCols; ++u) {
            const int c = min(col0 + u * nthr, ncols - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) v[u][r] = src[r][c];
        }
#pragma unroll
        for (int u = 0; u < kCols; ++u) {
            const int c = col0 + u * nthr;
            if (c < ncols) {
#pragma unroll
                for (int r = 0; r < R; ++r) xs[L::idx(c, r)] = ok[r] ? v[u][r] : (T)0;
            }
        }
    }
    if (tid < R) xs[(int64_t)ncols * R + tid] = (T)0;
}

// Stage rows row0 .. row0+R-1 of X held column-major (element (row, col) at
// col * nrows + row) into LDS in the lds_cols<T, R> layout; column ncols is
// zero.  A thread reads the R consecutive values of a column (one or two
// cache lines), two columns per pass with all loads before any store.
template <typename T, int R>
__device__ __forceinline__ void stage_cols(T* __restrict__ xs, const T* __restrict__ X, int64_t nrows, int64_t row0,
                                           int64_t ncols) {
    using L = lds_cols<T, R>;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const bool full = row0 + R <= nrows;   // uniform over the workgroup
    for (int64_t c0 = tid; c0 < ncols; c0 += 2 * nthr) {
        T v[2][R];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t c = c0 + u * nthr < ncols ? c0 + u * nthr : ncols - 1;
            const T* src = X + c * nrows + row0;
            if (full) {
                if constexpr (R * sizeof(T) % 16 == 0) {
                    if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {   // 16-byte pieces
                        using V4 = typename std::conditional<sizeof(T) == 8, double2, float4>::type;
                        constexpr int kP = (int)(16 / sizeof(T));
#pragma unroll
                        for (int q = 0; q < R / kP; ++q) {
                            const V4 x = reinterpret_cast<const V4*>(src)[q];
                            const T* xv = reinterpret_cast<const T*>(&x);
#pragma unroll
                            for (int i = 0; i < kP; ++i) v[u][q * kP + i] = xv[i];
                        }
                        continue;
                    }
                }
#pragma unroll
                for (int r = 0; r < R; ++r) v[u][r] = src[r];
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[u][r] = (row0 + r < nrows) ? src[r] : (T)0;
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t c = c0 + u * nthr;
            if (c < ncols) {
#pragma unroll
                for (int r = 0; r < R; ++r) xs[L::idx(c, r)] = v[u][r];
            }
        }
    }
    if (tid < R) xs[ncols * R + tid] = (T)0;
}

// ---------------------------------------------------------------- same spin
template <typename T>
struct ss_args {
    const T* X;            // nrows x ncols
    T* Y;
    int64_t nrows, ncols;
    sell_table<T> tab;     // sliced table of the column spin
    const T* ws;           // cross-spin sums of the row spin's strings, string-major (null: summed here)
    const uint64_t* row_str;   // strings of the row spin (cross-spin term), nw words each
    int nw;
    const double* diag;        // fused DIAG term (or null)
    int accumulate;
    int colmajor;              // X, Y (and diag) hold the transposes: (row, col) at col * nrows + row
};

// Rows blk*R .. blk*R+R-1: Y (=|+=) same-spin singles and doubles of the column
// spin.  LDS: xs[(ncols+1)*R] as [col][r]; ws[norb2*R] as [pq][r].
template <typename T, int R>
__device__ __forceinline__ void ss_block(const ss_args<T>& a, const T* __restrict__ jk, int norb, int64_t blk,
                                         unsigned char* lds_raw) {
    T* xs = reinterpret_cast<T*>(lds_raw);
    const int norb2 = norb * norb;
    const int64_t ncols = a.ncols, nrows = a.nrows;
    T* ws = xs + (ncols + 1) * R;
    const int64_t row0 = blk * R;
    const int nthr = blockDim.x;
    const int tid = threadIdx.x;
    // Each wave walks its bins' blocks (sell_table) as one stream, two blocks
    // (eight entries) ahead: what bounds the walk is the LDS, 64-byte pieces
    // at random columns, as long as the table's loads are in flight early
    // enough and the waves end together.  The first blocks load before the rows
    // are staged.
    const sell_table<T>& tab = a.tab;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int per = kBins / (nthr >> 6);
    int sl = tab.bin[wave * per];
    const int sl_end = tab.bin[(wave + 1) * per];
    int b = tab.bin[kBins + 1 + wave * per];
    const int b_last = max(tab.bin[kBins + 1 + (wave + 1) * per] - 1, 0);   // (the arrays hold one block past the last)
    struct block { uint32_t e[4]; T v[4]; };
    auto load = [&](int q) {
        block x;
        const int64_t at = (int64_t)min(q, b_last) * 256;
        const uint4 e = *reinterpret_cast<const uint4*>(tab.ent + at + lane * 4);
        x.e[0] = e.x, x.e[1] = e.y, x.e[2] = e.z, x.e[3] = e.w;
        if constexpr (sizeof(T) == 8) {
            const double2 v0 = *reinterpret_cast<const double2*>(tab.val + at + lane * 2);
            const double2 v1 = *reinterpret_cast<const double2*>(tab.val + at + 128 + lane * 2);
            x.v[0] = v0.x, x.v[1] = v0.y, x.v[2] = v1.x, x.v[3] = v1.y;
        } else {
            const float4 v = *reinterpret_cast<const float4*>(tab.val + at + lane * 4);
            x.v[0] = v.x, x.v[1] = v.y, x.v[2] = v.z, x.v[3] = v.w;
        }
        return x;
    };
    block x0 = load(b), x1 = load(b + 1);
    if (a.colmajor) {
        stage_cols<T, R>(xs, a.X, nrows, row0, ncols);
    } else {
        const T* rows[R];
#pragma unroll
        for (int r = 0; r < R; ++r) rows[r] = (row0 + r < nrows) ? a.X + (row0 + r) * ncols : nullptr;
        stage_rows<T, R>(xs, rows, (int)ncols);
    }
    // cross-spin term of the staged rows: ws[pq][r] = sum_{k in row string} (pq|kk),
    // from the per-string table, or summed over k in increasing order: every
    // (pq|kk) is loaded (no load behind a branch) and unoccupied k contribute
    // an exact zero
    if (a.ws) {
        for (int idx = tid; idx < R * norb2; idx += nthr) {
            const int r = idx / norb2, pq = idx - r * norb2;
            const int64_t row = row0 + r < nrows ? row0 + r : nrows - 1;
            ws[lds_cols<T, R>::idx(pq, r)] = a.ws[row * norb2 + pq];
        }
    } else {
        for (int idx = tid; idx < R * norb2; idx += nthr) {
            const int r = idx / norb2, pq = idx - r * norb2;
            const int64_t row = row0 + r;
            T acc = (T)0;
            for (int q = 0; q < a.nw; ++q) {
                const uint64_t x = (row < nrows) ? a.row_str[row * a.nw + q] : 0ull;
                const int kend = min(norb - 64 * q, 64);
                const T* jq = jk + (int64_t)(64 * q) * norb2 + pq;
                int k = 0;
                for (; k + 4 <= kend; k += 4) {
                    T v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = jq[(int64_t)(k + u) * norb2];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if ((x >> (k + u)) & 1ull) acc += v[u];
                }
                for (; k < kend; ++k)
                    if ((x >> k) & 1ull) acc += jq[(int64_t)k * norb2];
            }
            ws[lds_cols<T, R>::idx(pq, r)] = acc;
        }
    }
    __syncthreads();
    if (sl == sl_end) return;
    for (; sl < sl_end; ++sl) {
        const int b_end = tab.blk[sl + 1], s_end = b + tab.s_blk[sl];
        const int split = tab.split ? tab.split[sl] : 0;
        const int t = tab.perm[sl * 64 + lane];
        T acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = (T)0;
        auto use = [&](const block& x, bool single) {
            if (single) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int pair = (int)((x.e[u] >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
                    T xr[R], wr[R];
                    lds_cols<T, R>::load(xs, (int)(x.e[u] & SQD_NBR_MASK), xr);
                    lds_cols<T, R>::load(ws, pair, wr);
                    const bool neg = (x.e[u] >> 31) != 0;
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r] += (x.v[u] + (neg ? -wr[r] : wr[r])) * xr[r];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    T xr[R];
                    lds_cols<T, R>::load(xs, (int)x.e[u], xr);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r] += x.v[u] * xr[r];
                }
            }
        };
        for (; b < b_end; b += 2) {   // an even number of blocks
            use(x0, b < s_end);
            x0 = load(b + 2);
            use(x1, b + 1 < s_end);
            x1 = load(b + 3);
        }
        // the sums of a row held by several lanes, added across them
        for (int o = 1; o < (1 << split); o <<= 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] += __shfl_xor(acc[r], o);
        }
        if constexpr (R * sizeof(T) % 16 == 0) {
            // column-major output of a whole row block: R consecutive values
            // of the target's column in 16-byte pieces
            T* yp = a.Y + (int64_t)t * nrows + row0;
            if (a.colmajor && !a.diag && t < ncols && row0 + R <= nrows &&
                (reinterpret_cast<uintptr_t>(yp) & 15) == 0) {
                using V4 = typename std::conditional<sizeof(T) == 8, double2, float4>::type;
                constexpr int kP = (int)(16 / sizeof(T));
                V4 old[R / kP];
                if (a.accumulate) {
#pragma unroll
                    for (int q = 0; q < R / kP; ++q) old[q] = reinterpret_cast<const V4*>(yp)[q];
                }
#pragma unroll
                for (int q = 0; q < R / kP; ++q) {
                    V4 y;
                    T* yv = reinterpret_cast<T*>(&y);
                    const T* ov = reinterpret_cast<const T*>(&old[q]);
#pragma unroll
                    for (int i = 0; i < kP; ++i) yv[i] = acc[q * kP + i] + (a.accumulate ? ov[i] : (T)0);
                    reinterpret_cast<V4*>(yp)[q] = y;
                }
                continue;
            }
        }
        if (t < ncols) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t row = row0 + r;
                if (row < nrows) {
                    const int64_t o = a.colmajor ? (int64_t)t * nrows + row : row * ncols + t;
                    T val = acc[r];
                    if (a.diag) val += (T)(a.diag[o] * (double)xs[lds_cols<T, R>::idx(t, r)]);
                    if (a.accumulate) val += a.Y[o];
                    a.Y[o] = val;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- alpha-beta, grouped
// The alpha single entries e (CSR position in the target row's list; source
// row src(e), pair ai(e), sign s(e)) are grouped by pair ai and cut into chunks
// of G entries that share ai.  One unit per chunk stages the G source rows of C
// in LDS (lds_cols layout) and the row (ai|..) of the (pq|rs) matrix, then
// walks the sliced beta singles table once for all G rows:
//   Y[e][slot(jb')] = s(e) * sum_{beta singles jb' <- jb (pair bj, s_b)} s_b (ai|bj) C[src(e)][jb]
// Y is written in slot order (ab_table), so each wave stores consecutive
// values, with non-temporal stores (read once, by the gather); the gather maps
// slots back to beta strings.
template <typename T>
struct abg_args {
    const T* C;
    T* Y;                     // nnz_alpha_singles x ldy, columns in sliced (slot) order
    int64_t nb;
    const int2* grp;          // chunks x G alpha singles: CSR position (-1 = padding), gather form
    const int* chunk_pair;
    ab_table tab;             // sliced beta singles; Y has tab.nslots columns
};

// The calling wave's walk over its bins of a sliced singles table.  The first
// blocks are loaded at construction (before the rows are staged, so that the
// two waits run together), the others three blocks ahead.  run() calls begin(),
// each(entry) for every entry of the lane and end(split, slot) for each slice.
struct ab_walk {
    const ab_table& tab;
    int lane, sl, sl_end, b = 0, b_last = 0;
    uint4 x0, x1, x2;
    __device__ __forceinline__ uint4 load(int q) const {
        return *reinterpret_cast<const uint4*>(tab.ent + (int64_t)min(q, b_last) * 256 + lane * 4);
    }
    __device__ __forceinline__ explicit ab_walk(const ab_table& t) : tab(t), lane(threadIdx.x & 63) {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int per = kBins / ((int)blockDim.x >> 6);
        sl = tab.bin[wave * per];
        sl_end = tab.bin[(wave + 1) * per];
        b = tab.bin[kBins + 1 + wave * per];
        b_last = max(tab.bin[kBins + 1 + (wave + 1) * per] - 1, 0);   // (the table holds one block past the last)
        x0 = load(b);
        x1 = load(b + 1);
        x2 = load(b + 2);
    }
    template <typename B, typename F, typename E>
    __device__ __forceinline__ void run(B&& begin, F&& each, E&& end) {
        for (; sl < sl_end; ++sl) {
            int left = tab.cols[sl];
            const int split = tab.split ? tab.split[sl] : 0, slot = tab.slot[sl];
            begin();
            for (; left > 0; left -= 4) {
                const uint4 x = x0;
                x0 = x1;
                x1 = x2;
                x2 = load(b + 3);
                ++b;
                each(x.x);
                if (left > 1) each(x.y);
                if (left > 2) each(x.z);
                if (left > 3) each(x.w);
            }
            end(split, slot);
        }
    }
};

// The sums of one slice for G alpha singles (CSR positions e, -1: none): added
// across the lanes of each row, times the sign, into Y.
template <typename T, int G>
__device__ __forceinline__ void put_y(const abg_args<T>& a, const int (&e)[G], const T (&sgn)[G], T (&acc)[G], int lane,
                                      int split, int slot) {
    for (int o = 1; o < (1 << split); o <<= 1) {
#pragma unroll
        for (int r = 0; r < G; ++r) acc[r] += __shfl_xor(acc[r], o);
    }
    if (lane & ((1 << split) - 1)) return;
    // lanes without a row read only the zero column: their value is zero
    T* y = a.Y + slot + (lane >> split);
#pragma unroll
    for (int r = 0; r < G; ++r)
        if (e[r] >= 0) __builtin_nontemporal_store(sgn[r] * acc[r], y + (int64_t)e[r] * a.tab.nslots);
}

template <typename T, int G>
__device__ __forceinline__ void abg_block(const abg_args<T>& a, const T* __restrict__ V, int norb, int64_t chunk,
                                          unsigned char* lds_raw) {
    T* xs = reinterpret_cast<T*>(lds_raw);
    const int norb2 = norb * norb;
    const int64_t nb = a.nb;
    T* vrow = xs + (nb + 1) * G;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int pair = a.chunk_pair[chunk];
    ab_walk walk(a.tab);
    int e[G];
    T sgn[G];
    {
        const T* rows[G];
#pragma unroll
        for (int r = 0; r < G; ++r) {
            const int2 x = a.grp[chunk * G + r];
            e[r] = x.x;
            sgn[r] = ((uint32_t)x.y >> 31) ? (T)-1 : (T)1;
            rows[r] = e[r] >= 0 ? a.C + (int64_t)((uint32_t)x.y & SQD_NBR_MASK) * nb : nullptr;
        }
        stage_rows<T, G>(xs, rows, (int)nb);
    }
    for (int q = tid; q < norb2; q += nthr) vrow[q] = V[(int64_t)pair * norb2 + q];
    __syncthreads();
    const int lane = tid & 63;
    T acc[G];
    walk.run(
        [&] {
#pragma unroll
            for (int r = 0; r < G; ++r) acc[r] = (T)0;
        },
        [&](uint32_t b) {
            const int nbr = (int)(b & SQD_NBR_MASK);
            const int pb = (int)((b >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
            T v = vrow[pb];
            if (b >> 31) v = -v;
            T xr[G];
            lds_cols<T, G>::load(xs, nbr, xr);
#pragma unroll
            for (int r = 0; r < G; ++r) acc[r] += v * xr[r];
        },
        [&](int split, int slot) { put_y<T, G>(a, e, sgn, acc, lane, split, slot); });
}

// The same Y from blocks of G sources by one or two pairs (sqd_ensure_ab_blocks):
// where the G staged rows of C serve two pairs, an entry of the table costs 8 G
// bytes of LDS for C and 16 for the integrals for 2 G products instead of 8 G + 8
// for G, and the table is read once for both (2000 strings per spin, norb 16: 6100
// walks of the beta table in place of 8800, sigma FP64 715 -> 653 us, FP32
// 411 -> 389).  Same products and summation order as abg_block.
template <typename T>
struct abb_args {
    const T* C;
    T* Y;
    int64_t nb;
    const int2* grp;          // alpha singles: CSR position (-1 = padding), gather form
    const int2* pair;
    int n2;                   // the first n2 blocks: G singles of pair.x, G of pair.y; the others G of pair.x
    ab_table tab;
};

template <typename T, int G, int P>
__device__ __forceinline__ void abb_walk(const abb_args<T>& a, const T* __restrict__ V, int norb, int64_t chunk, int2 pair,
                                         unsigned char* lds_raw) {
    T* xs = reinterpret_cast<T*>(lds_raw);
    const int norb2 = norb * norb;
    const int64_t nb = a.nb;
    T* vrow = xs + (nb + 1) * G;             // the pairs' integrals, P side by side
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    ab_walk walk(a.tab);
    int e[P * G];
    uint32_t neg = 0;
    {
        const T* rows[G];
        const int2* grp = a.grp + (chunk + (P > 1 ? chunk : a.n2)) * G;
#pragma unroll
        for (int r = 0; r < P * G; ++r) {
            const int2 x = grp[r];
            e[r] = x.x;
            neg |= ((uint32_t)x.y >> 31) << r;
            if (r < G) rows[r] = e[r] >= 0 ? a.C + (int64_t)((uint32_t)x.y & SQD_NBR_MASK) * nb : nullptr;
        }
        stage_rows<T, G>(xs, rows, (int)nb);
    }
    for (int q = tid; q < norb2; q += nthr) {
        vrow[q * P] = V[(int64_t)pair.x * norb2 + q];
        if (P > 1) vrow[q * P + 1] = V[(int64_t)pair.y * norb2 + q];
    }
    __syncthreads();
    T acc[P * G];
    walk.run(
        [&] {
#pragma unroll
            for (int r = 0; r < P * G; ++r) acc[r] = (T)0;
        },
        [&](uint32_t b) {
            const int nbr = (int)(b & SQD_NBR_MASK);
            const int pb = (int)((b >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
            T v[P], xr[G];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                v[p] = vrow[pb * P + p];
                if (b >> 31) v[p] = -v[p];
            }
            lds_cols<T, G>::load(xs, nbr, xr);
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int r = 0; r < G; ++r) acc[p * G + r] += v[p] * xr[r];
        },
        [&](int split, int slot) {
            for (int o = 1; o < (1 << split); o <<= 1) {
#pragma unroll
                for (int r = 0; r < P * G; ++r) acc[r] += __shfl_xor(acc[r], o);
            }
            if (lane & ((1 << split) - 1)) return;
            T* y = a.Y + slot + (lane >> split);
#pragma unroll
            for (int r = 0; r < P * G; ++r)
                if (e[r] >= 0)
                    __builtin_nontemporal_store((neg >> r) & 1 ? -acc[r] : acc[r], y + (int64_t)e[r] * a.tab.nslots);
        });
}

template <typename T, int G>
__device__ __forceinline__ void abb_block(const abb_args<T>& a, const T* __restrict__ V, int norb, int64_t chunk,
                                          unsigned char* lds_raw) {
    const int2 pair = a.pair[chunk];
    if (chunk >= a.n2) abb_walk<T, G, 1>(a, V, norb, chunk, pair, lds_raw);
    else abb_walk<T, G, 2>(a, V, norb, chunk, pair, lds_raw);
}

// The same Y from chunks of up to GS alpha singles that share their source
// string (chunk_src): one staged row of C serves GS pairs, whose (ai|..) rows
// are staged beside it.  Where a row of C fills most of the LDS (long rows,
// where the pair-grouped chunks hold one single) this reads 8 bytes of LDS
// per table entry for C and 8 per single for the integral, (8 + 8 GS) / GS
// bytes per connection instead of 16, and stages each source row once per GS
// singles.  Same products and summation order as abg_block.
template <typename T, int GS>
__device__ __forceinline__ void abs_block(const abg_args<T>& a, const int* __restrict__ chunk_src,
                                          const T* __restrict__ V, int norb, int64_t chunk, unsigned char* lds_raw) {
    T* xs = reinterpret_cast<T*>(lds_raw);   // the source row, column nb zero
    const int norb2 = norb * norb;
    const int64_t nb = a.nb;
    T* vrows = xs + (nb + 1);                // GS rows of (ai|..), row g at g * norb2
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int64_t src = chunk_src[chunk];
    ab_walk walk(a.tab);
    int e[GS], pr[GS];
    T sgn[GS];
#pragma unroll
    for (int g = 0; g < GS; ++g) {
        const int2 y = a.grp[chunk * GS + g];
        e[g] = y.x;
        const uint32_t x = (uint32_t)y.y;   // 0 where none
        sgn[g] = (x >> 31) ? (T)-1 : (T)1;
        pr[g] = (int)((x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
    }
    const T* crow = a.C + src * nb;
    for (int64_t k = tid; k < nb; k += nthr) xs[k] = crow[k];
    if (tid == 0) xs[nb] = (T)0;
    for (int q = tid; q < GS * norb2; q += nthr) {
        const int g = q / norb2, r = q - g * norb2;
        vrows[q] = e[g] >= 0 ? V[(int64_t)pr[g] * norb2 + r] : (T)0;
    }
    __syncthreads();
    const int lane = tid & 63;
    T acc[GS];
    walk.run(
        [&] {
#pragma unroll
            for (int g = 0; g < GS; ++g) acc[g] = (T)0;
        },
        [&](uint32_t b) {
            const int nbr = (int)(b & SQD_NBR_MASK);
            const int pb = (int)((b >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
            T x = xs[nbr];
            if (b >> 31) x = -x;   // (-v) x = v (-x) exactly
#pragma unroll
            for (int g = 0; g < GS; ++g) acc[g] += vrows[g * norb2 + pb] * x;
        },
        [&](int split, int slot) { put_y<T, GS>(a, e, sgn, acc, lane, split, slot); });
}

// What the gather adds to a row of sigma, and where the row goes.
template <typename T>
struct gather_args {
    const T* Y;
    int64_t nb;
    int64_t nslots;           // columns of Y
    const int* perm;          // string of each slot
    const int* a_off;
    T* S;                     // rows of sigma: read and, without out64, written
    const T* S2;              // added too, or null
    const double* diag;       // diag * c added too (FP64 or into out64), or null
    const double* c;
    double* out64;            // FP32 sums: the row goes here in FP64 (S is only read)
};

// Row ia of sigma: S + S2 + sum_{e in row ia} Y[e][slot] (+ diag c), one
// workgroup per row.  A thread reads two adjacent slots with one vector load,
// eight rows of Y in flight; Y is written once and read once, so both sides
// bypass the caches' retention (non-temporal accesses): the tables and C of
// the next kernels stay cached (4.0e6-determinant workload, same box: gather
// 142 -> 103 us, the beta-beta kernel after it 192 -> 176 us).  Rows of Y
// shorter than the workgroup are read by ng groups of threads, each taking
// every ng-th single, whose sums are added in order.  With `row` (LDS, ng x nb
// values) the sums are placed by target first and sigma is updated with
// coalesced accesses; without it (rows too long for the LDS; one group) each
// sum is added in place.
template <typename T>
__device__ __forceinline__ void gather_row(const gather_args<T>& a, int64_t ia, int ng, T* row) {
    typedef T T2 __attribute__((ext_vector_type(2)));
    constexpr int kU = 8;
    const int64_t nb = a.nb, nslots = a.nslots;
    const int per = (int)blockDim.x / ng, grp = (int)threadIdx.x / per, t = (int)threadIdx.x - grp * per;
    const int e0 = a.a_off[ia] + grp, e1 = a.a_off[ia + 1];
    auto put = [&](int64_t j, T v) {                 // sum v of target j of the row
        const int64_t o = ia * nb + j;
        v += a.S2 ? a.S[o] + a.S2[o] : a.S[o];
        if constexpr (sizeof(T) == 8) {
            if (a.diag) v += a.diag[o] * a.c[o];
            a.S[o] = v;
        } else if (a.out64) {
            double d = (double)v;
            if (a.diag) d += a.diag[o] * a.c[o];
            a.out64[o] = d;
        } else {
            a.S[o] = v;
        }
    };
    T* mine = row + grp * nb;
    for (int64_t p = 2 * (int64_t)t; p < nslots; p += 2 * (int64_t)per) {
        T a0 = (T)0, a1 = (T)0;
        for (int e = e0; e < e1; e += kU * ng) {
            T2 v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u)
                v[u] = (e + u * ng < e1) ? __builtin_nontemporal_load(
                                                 reinterpret_cast<const T2*>(a.Y + (int64_t)(e + u * ng) * nslots + p))
                                           : T2{(T)0, (T)0};
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                a0 += v[u].x;
                a1 += v[u].y;
            }
        }
        const int t0 = a.perm[p], t1 = a.perm[p + 1];
        if (row) {
            if (t0 < nb) mine[t0] = a0;
            if (t1 < nb) mine[t1] = a1;
        } else {
            if (t0 < nb) put(t0, a0);
            if (t1 < nb) put(t1, a1);
        }
    }
    if (!row) return;
    __syncthreads();
    for (int64_t j = threadIdx.x; j < nb; j += blockDim.x) {
        T v = row[j];
        for (int q = 1; q < ng; ++q) v += row[q * nb + j];
        put(j, v);
    }
}

// out[c][r] (=|+=) in[r][c] for the 64 x 64 tile (ty, tx); in is rows x cols.
template <typename TI, typename TO, bool ADD>
__device__ __forceinline__ void transpose_tile(const TI* __restrict__ in, TO* __restrict__ out, int64_t rows,
                                               int64_t cols, int64_t ty, int64_t tx_, TI (*tile)[65]) {
    const int64_t r0 = ty * 64, c0 = tx_ * 64;
    const int tx = threadIdx.x & 63, tyy = threadIdx.x >> 6, ny = blockDim.x >> 6;
    for (int k = tyy; k < 64; k += ny) {
        const int64_t r = r0 + k, c = c0 + tx;
        if (r < rows && c < cols) tile[k][tx] = in[r * cols + c];
    }
    __syncthreads();
    for (int k = tyy; k < 64; k += ny) {
        const int64_t c = c0 + k, r = r0 + tx;
        if (r < rows && c < cols) {
            TO v = (TO)tile[tx][k];
            if (ADD) v += out[c * rows + r];
            out[c * rows + r] = v;
        }
    }
}
