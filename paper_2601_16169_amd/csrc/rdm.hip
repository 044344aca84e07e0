// Spin-summed reduced density matrices of a normalised vector c, the energy
// gradients by Hellmann-Feynman: dE/dh_pq = rdm1_pq, dE/d(pq|rs) = rdm2_pqrs/2
// (E = ecore + sum h.rdm1 + 1/2 sum (pq|rs) rdm2 for the Hamiltonian of
// Sec. I-II restricted to the product space of Sec. IV).
//
//   rdm1[p,q]     = sum_s <a+_ps a_qs>
//   rdm2[p,q,r,s] = sum_st <a+_ps a+_rt a_st a_qs>
//
// Same-spin parts come from pairs of strings of one spin connected by the
// excitation tables (or equal), weighted by the overlap of the matching rows
// (alpha) or columns (beta) of C: P_a = C C^T, P_b = C^T C, two symmetric FP64
// MFMA products.  The alpha-beta part is
//   X[pq][rs] = <c| E^a_pq E^b_rs |c>
//             = sum over alpha pairs (I <- J by pq) and beta pairs (K <- L by rs)
//               of their signs times c[J, K] c[I, L],
// a sum over exactly the pairs of singles (and diagonal pairs): for one alpha
// pair the rows I and J of C are staged in LDS and the beta singles, sorted by
// orbital pair into a sliced table, are walked once, a lane per orbital pair
// (or part of one).  X[qp][sr] = X[pq][rs], so alpha pairs with p > q alone
// are walked; rdm2 receives X[pq][rs] + X[rs][pq] (the beta-alpha term).
#include <algorithm>
#include <type_traits>

#include "sigma_body.h"
#include "slices.h"
#include "sqd_internal.h"

namespace {

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

typedef double double4_t __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4: A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k;
// lane l, element q of the accumulator holds D[l / 16 + 4 q][l % 16] (checked on
// gfx950; the f32 form of the same shape uses row 4 (l / 16) + q instead).
__device__ __forceinline__ int acc_row(int lane, int q) { return (lane >> 4) + 4 * q; }

// ---------------------------------------------------------------- P = A A^T
// A: M x K (row-major), P: M x M, symmetric: only the 64 x 64 tiles that reach
// the lower triangle are computed and every element is written to both places.
// Four waves of 32 x 32 (2 x 2 MFMA tiles), K steps of 16 through two LDS
// buffers, the next step's loads in flight while the matrix cores run.  Bound
// by the FP64 matrix cores: 4000 x 4000 x 4000, 6.4e10 flop of the triangle, 1.25
// ms (51 TFLOP/s; the whole product, one buffer: 4.1 ms; tiles of 128 x 64: 1.53
// ms, the last of two rounds of workgroups half empty; tiles grouped by XCD
// for the L2: 1.49 ms).
constexpr int kTM = 64, kTN = 64, kTK = 16;
__global__ void __launch_bounds__(256)
k_gram(const double* __restrict__ A, double* __restrict__ P, int64_t M, int64_t K) {
    __shared__ double As[2][kTM][kTK + 1];
    __shared__ double Bs[2][kTN][kTK + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int tm = 0, tn = blockIdx.x;   // tile row tm holds the tiles 0 .. tm
    {
        tm = (int)((sqrt(8.0 * tn + 1.0) - 1.0) * 0.5);
        while ((tm + 1) * (tm + 2) / 2 <= tn) ++tm;
        while (tm * (tm + 1) / 2 > tn) --tm;
        tn -= tm * (tm + 1) / 2;
    }
    const int64_t m0 = (int64_t)tm * kTM, n0 = (int64_t)tn * kTN;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    double4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (double4_t){0.0, 0.0, 0.0, 0.0};
    // thread tid loads column tid % 16 of rows tid / 16, + 16, ...
    const int lr = tid >> 4, lc = tid & 15;
    double ra[kTM / 16], rb[kTN / 16];
    auto fetch = [&](int64_t k0) {
        const int64_t gk = k0 + lc;
#pragma unroll
        for (int u = 0; u < kTM / 16; ++u) {
            const int64_t r = m0 + lr + 16 * u;
            ra[u] = (r < M && gk < K) ? A[r * K + gk] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kTN / 16; ++u) {
            const int64_t r = n0 + lr + 16 * u;
            rb[u] = (r < M && gk < K) ? A[r * K + gk] : 0.0;
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int u = 0; u < kTM / 16; ++u) As[buf][lr + 16 * u][lc] = ra[u];
#pragma unroll
        for (int u = 0; u < kTN / 16; ++u) Bs[buf][lr + 16 * u][lc] = rb[u];
    };
    fetch(0);
    store(0);
    __syncthreads();
    int buf = 0;
    for (int64_t k0 = 0; k0 < K; k0 += kTK) {
        const bool more = k0 + kTK < K;
        if (more) fetch(k0 + kTK);
#pragma unroll
        for (int ks = 0; ks < kTK; ks += 4) {
            double a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = As[buf][wm + i * 16 + (lane & 15)][ks + (lane >> 4)];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = Bs[buf][wn + j * 16 + (lane & 15)][ks + (lane >> 4)];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (more) store(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t r = m0 + wm + i * 16 + acc_row(lane, q);
                const int64_t c = n0 + wn + j * 16 + (lane & 15);
                if (r < M && c <= r) {
                    P[r * M + c] = acc[i][j][q];
                    P[c * M + r] = acc[i][j][q];
                }
            }
}

// ---------------------------------------------------------------- same spin
// One wavefront per string I of one spin; w(J) = P[I][J].  Pairs visited in
// both directions by the symmetric tables.  Updates (Gamma_pqrs = <a+_p a+_r a_s a_q>):
//   diagonal:   rdm1[k][k] += w;  Gamma[k][k][l][l] += w, Gamma[l][k][k][l] -= w (k != l in I)
//   single (i in I, a in J, sign s; spectators k in I, k != i):
//               rdm1[i][a] += s w; Gamma[i][a][k][k] += s w, Gamma[k][k][i][a] += s w,
//               Gamma[k][a][i][k] -= s w, Gamma[i][k][k][a] -= s w
//   double (i < j in I, a < b in J, sign s):
//               Gamma[i][a][j][b] += s w, Gamma[j][b][i][a] += s w,
//               Gamma[j][a][i][b] -= s w, Gamma[i][b][j][a] -= s w
__global__ void __launch_bounds__(256)
k_rdm_same(const uint64_t* __restrict__ str, int nw, int64_t n, const int* __restrict__ s_off,
           const uint64_t* __restrict__ s_ent, const int* __restrict__ d_off, const uint64_t* __restrict__ d_ent,
           const double* __restrict__ P, int norb, double* __restrict__ rdm1, double* __restrict__ rdm2) {
    const int64_t I = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (I >= n) return;
    const int64_t n2 = (int64_t)norb * norb;
    auto G = [&](int p, int q, int r, int s) -> double* { return rdm2 + ((int64_t)p * norb + q) * n2 + r * norb + s; };
    const uint64_t* sI = str + I * nw;
    const double wd = P[I * n + I];
    // diagonal
    for (int k = lane; k < norb; k += 64) {
        if (!str_bit(sI, k)) continue;
        atomicAdd(&rdm1[k * norb + k], wd);
        if (rdm2)
            str_for_each(sI, nw, [&](int l) {
                if (l == k) return;
                atomicAdd(G(k, k, l, l), wd);
                atomicAdd(G(l, k, k, l), -wd);
            });
    }
    for (int e = s_off[I] + lane; e < s_off[I + 1]; e += 64) {
        const uint64_t x = s_ent[e];
        const int64_t J = (int64_t)(x & 0xFFFFFFFFull);
        const int i = SQD_ENT_ORB(x, 0), a = SQD_ENT_ORB(x, 1);
        const double sw = ((x >> 63) ? -1.0 : 1.0) * P[I * n + J];
        atomicAdd(&rdm1[i * norb + a], sw);
        if (rdm2)
            str_for_each(sI, nw, [&](int k) {
                if (k == i) return;
                atomicAdd(G(i, a, k, k), sw);
                atomicAdd(G(k, k, i, a), sw);
                atomicAdd(G(k, a, i, k), -sw);
                atomicAdd(G(i, k, k, a), -sw);
            });
    }
    if (!rdm2) return;
    for (int e = d_off[I] + lane; e < d_off[I + 1]; e += 64) {
        const uint64_t x = d_ent[e];
        const int64_t J = (int64_t)(x & 0xFFFFFFFFull);
        const int i = SQD_ENT_ORB(x, 0), j = SQD_ENT_ORB(x, 1);
        const int a = SQD_ENT_ORB(x, 2), b = SQD_ENT_ORB(x, 3);
        const double sw = ((x >> 63) ? -1.0 : 1.0) * P[I * n + J];
        atomicAdd(G(i, a, j, b), sw);
        atomicAdd(G(j, b, i, a), sw);
        atomicAdd(G(j, a, i, b), -sw);
        atomicAdd(G(i, b, j, a), -sw);
    }
}

// ---------------------------------------------------------------- alpha-beta
// The beta singles by orbital pair rs (entry K -> L of a string's table, i -> a:
// r = i, s = a) and the diagonal pairs rr of every string, sliced as sell_table: a row is an orbital pair, its entries (K, L, sign), long rows
// over several lanes, four entries of a lane to a block.
struct pair_table {
    int nslices;
    const int* perm;       // nslices*64: rs at the first lane of its group, else -1
    const int* split;
    const int* blk;        // nslices+1 block offsets
    const int* bin;        // kBins+1 slice offsets
    const uint2* ent;      // entry q of lane l of block b at 256 b + 64 q + l: K | sign << 31, L; padding K = L = nb
};
// alpha pairs (I <- J by pq, p > q), sorted by pq: sign in bit 31 of j
struct alpha_unit { int i; uint32_t j; };

// One workgroup per chunk of alpha pairs that share pq: G at a time, columns of
// ws (s c[J, :]) and us (c[I, :]) side by side in LDS, or (staged = false, rows
// too long for that) read from C.  What bounds it is the LDS: 16 bytes per
// product at random columns, 2.2e9 + 1.0e9 products on 4000 + 4000 strings of
// 20 orbitals (norb^2 MFMA products over dense blocks of the same sums, most
// of them zero: 44 ms; this: 1.35 ms).  The sums of a lane stay in
// LDS across the batches of the chunk (acc; one batch: null).
template <int G, bool STAGED>
__global__ void __launch_bounds__(1024)
k_rdm_ab(const double* __restrict__ C, int64_t nb, pair_table tab, const alpha_unit* __restrict__ units,
         const int4* __restrict__ chunks, int norb, int keep, double* __restrict__ rdm2) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    using L = lds_cols<double, G>;
    double* ws = reinterpret_cast<double*>(lds_raw);
    double* us = ws + (STAGED ? (nb + 1) * G : 0);
    double* acc = us + (STAGED ? (nb + 1) * G : 0);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int per = kBins / (nthr >> 6);
    const int sl0 = tab.bin[wave * per], sl1 = tab.bin[(wave + 1) * per];
    const int4 ch = chunks[blockIdx.x];   // first unit, units, pq
    const int64_t n2 = (int64_t)norb * norb;
    const int pq = ch.z, qp = (pq % norb) * norb + pq / norb;
    auto put = [&](int sl, double v) {
        for (int o = 1; o < (1 << tab.split[sl]); o <<= 1) v += __shfl_xor(v, o);
        const int rs = tab.perm[sl * 64 + lane];
        if (rs < 0) return;
        const int sr = (rs % norb) * norb + rs / norb;
        atomicAdd(&rdm2[pq * n2 + rs], v);
        atomicAdd(&rdm2[rs * n2 + pq], v);
        atomicAdd(&rdm2[qp * n2 + sr], v);
        atomicAdd(&rdm2[sr * n2 + qp], v);
    };
    if (keep)
        for (int sl = sl0; sl < sl1; ++sl) acc[sl * 64 + lane] = 0.0;
    if (STAGED && tid < G) ws[L::idx(nb, tid)] = us[L::idx(nb, tid)] = 0.0;   // the padding's column
    for (int k0 = 0; k0 < ch.y; k0 += G) {
        const double* wr[G];
        const double* ur[G];
        double sg[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const bool in = k0 + g < ch.y;
            const alpha_unit x = units[ch.x + (in ? k0 + g : 0)];
            wr[g] = C + (int64_t)(x.j & 0x7FFFFFFFu) * nb;
            ur[g] = C + (int64_t)x.i * nb;
            sg[g] = !in ? 0.0 : (x.j >> 31) ? -1.0 : 1.0;
        }
        if constexpr (STAGED) {
            __syncthreads();   // the previous batch is done with the rows
            for (int64_t c = tid; c < nb; c += nthr) {
                double w[G], u[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    w[g] = wr[g][c];
                    u[g] = ur[g][c];
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    // a batch's missing pairs count as zero whatever their rows hold
                    ws[L::idx(c, g)] = sg[g] == 0.0 ? 0.0 : sg[g] * w[g];
                    us[L::idx(c, g)] = sg[g] == 0.0 ? 0.0 : u[g];
                }
            }
            __syncthreads();
        }
        for (int sl = sl0; sl < sl1; ++sl) {
            const int b1 = tab.blk[sl + 1];
            double v = 0.0;
            auto use = [&](uint2 e) {
                if constexpr (STAGED) {
                    double w[G], u[G];
                    L::load(ws, (int)(e.x & 0x7FFFFFFFu), w);
                    L::load(us, (int)e.y, u);
                    double t = 0.0;
#pragma unroll
                    for (int g = 0; g < G; ++g) t += w[g] * u[g];
                    v += (e.x >> 31) ? -t : t;
                } else {
                    const int64_t k = e.x & 0x7FFFFFFFu;
                    const double t = k < nb ? wr[0][k] * ur[0][e.y] : 0.0;
                    v += (e.x >> 31) ? -t : t;
                }
            };
            int b = tab.blk[sl];
            uint2 x[4], y[4];
            auto load = [&](uint2 (&z)[4], int q) {
#pragma unroll
                for (int u = 0; u < 4; ++u) z[u] = tab.ent[(int64_t)min(q, b1 - 1) * 256 + u * 64 + lane];
            };
            if (b < b1) load(x, b);
            for (; b < b1; ++b) {
                load(y, b + 1);
#pragma unroll
                for (int u = 0; u < 4; ++u) use(x[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = y[u];
            }
            if constexpr (!STAGED) v *= sg[0];
            if (keep) acc[sl * 64 + lane] += v;
            else put(sl, v);
        }
    }
    if (keep)
        for (int sl = sl0; sl < sl1; ++sl) put(sl, acc[sl * 64 + lane]);
}

// Diagonal alpha pairs: t[I][rs] = sum over beta pairs of sign c[I, K] c[I, L]
// for G rows I at a time, then X[pp][rs] = sum of t[I][rs] over the I that
// hold p (k_rdm_occ).  t: na rows of ldt, slot (slice, lane / group) order.
template <int G, bool STAGED>
__global__ void __launch_bounds__(1024)
k_rdm_diag(const double* __restrict__ C, int64_t na, int64_t nb, pair_table tab, double* __restrict__ t) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    using L = lds_cols<double, G>;
    double* us = reinterpret_cast<double*>(lds_raw);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int per = kBins / (nthr >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * G;
    const int64_t ldt = (int64_t)tab.nslices * 64;
    const double* ur[G];
#pragma unroll
    for (int g = 0; g < G; ++g) ur[g] = C + (row0 + g < na ? row0 + g : na - 1) * nb;
    if constexpr (STAGED) {
        for (int64_t c = tid; c < nb; c += nthr) {
            double u[G];
#pragma unroll
            for (int g = 0; g < G; ++g) u[g] = ur[g][c];
#pragma unroll
            for (int g = 0; g < G; ++g) us[L::idx(c, g)] = u[g];
        }
        if (tid < G) us[L::idx(nb, tid)] = 0.0;
        __syncthreads();
    }
    for (int sl = tab.bin[wave * per]; sl < tab.bin[(wave + 1) * per]; ++sl) {
        double v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) v[g] = 0.0;
        for (int b = tab.blk[sl]; b < tab.blk[sl + 1]; ++b) {
            uint2 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = tab.ent[(int64_t)b * 256 + u * 64 + lane];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = (int)(x[u].x & 0x7FFFFFFFu), l = (int)x[u].y;
                double w[G], z[G];
                if constexpr (STAGED) {
                    L::load(us, k, w);
                    L::load(us, l, z);
                } else {
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        w[g] = k < nb ? ur[g][k] : 0.0;
                        z[g] = k < nb ? ur[g][l] : 0.0;
                    }
                }
#pragma unroll
                for (int g = 0; g < G; ++g) v[g] += (x[u].x >> 31) ? -(w[g] * z[g]) : w[g] * z[g];
            }
        }
        for (int o = 1; o < (1 << tab.split[sl]); o <<= 1) {
#pragma unroll
            for (int g = 0; g < G; ++g) v[g] += __shfl_xor(v[g], o);
        }
        if (tab.perm[sl * 64 + lane] >= 0) {
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (row0 + g < na) t[(row0 + g) * ldt + sl * 64 + lane] = v[g];
        }
    }
}

// X[pp][rs] from t: a wave per slice of orbital pairs and range of strings,
// the sums per orbital p in LDS (a column per lane).
__global__ void __launch_bounds__(64)
k_rdm_occ(const double* __restrict__ t, pair_table tab, const uint64_t* __restrict__ str, int nw, int64_t na,
          int64_t per, int norb, double* __restrict__ rdm2) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double* acc = reinterpret_cast<double*>(lds_raw);   // norb x 64
    const int lane = threadIdx.x;
    const int sl = blockIdx.x;
    const int rs = tab.perm[sl * 64 + lane];
    const int64_t n2 = (int64_t)norb * norb, ldt = (int64_t)tab.nslices * 64;
    const int64_t i0 = (int64_t)blockIdx.y * per, i1 = i0 + per < na ? i0 + per : na;
    if (rs < 0) return;
    for (int p = 0; p < norb; ++p) acc[p * 64 + lane] = 0.0;
    for (int64_t i = i0; i < i1; ++i) {
        const double v = t[i * ldt + sl * 64 + lane];
        str_for_each(str + i * nw, nw, [&](int p) { acc[p * 64 + lane] += v; });
    }
    for (int p = 0; p < norb; ++p) {
        const int64_t pp = (int64_t)p * norb + p;
        const double v = acc[p * 64 + lane];
        if (v == 0.0) continue;
        atomicAdd(&rdm2[pp * n2 + rs], v);
        atomicAdd(&rdm2[rs * n2 + pp], v);
    }
}

template <typename T>
__global__ void k_zero(T* __restrict__ p, int64_t n) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = (T)0;
}

__global__ void __launch_bounds__(256) k_transpose_d(const double* __restrict__ in, double* __restrict__ out,
                                                     int64_t rows, int64_t cols) {
    __shared__ double tile[64][65];
    const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int k = ty; k < 64; k += 4) {
        const int64_t r = r0 + k, c = c0 + tx;
        if (r < rows && c < cols) tile[k][tx] = in[r * cols + c];
    }
    __syncthreads();
    for (int k = ty; k < 64; k += 4) {
        const int64_t c = c0 + k, r = r0 + tx;
        if (r < rows && c < cols) out[c * rows + r] = tile[tx][k];
    }
}

// Host-built part of the alpha-beta sums, kept with the space (it does not
// depend on the integrals): the beta pair table, the alpha pairs sorted by
// orbital pair and their chunks.
int build_rdm_plan(sqd_ctx* ctx, sqd_space* sp) {
    if (sp->rdm_mem) return SQD_OK;
    const sqd_beside_capture beside;   // a first call may be captured
    spin_tables& A = sp->sp[0];
    spin_tables& B = sp->sp[1].alias ? A : sp->sp[1];
    const int norb = sp->norb, n2 = norb * norb;
    const int64_t na = A.n, nb = B.n;
    int rc;
    if ((rc = sqd_host_singles(ctx, A)) || (rc = sqd_host_singles(ctx, B))) return rc;
    const std::vector<int>&ao = A.s_off_host, &bo = B.s_off_host;
    const std::vector<uint32_t>&ap = A.s_pk_host, &bp = B.s_pk_host;
    const std::vector<uint64_t>& bs = B.str_host;
    // beta pairs by rs (counting sort)
    auto rs_of = [&](uint32_t x) {
        const int pair = (int)((x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
        return (pair % norb) * norb + pair / norb;
    };
    std::vector<int> at(n2 + 1, 0);
    auto each_beta = [&](auto&& f) {   // f(rs, K, L with the sign in bit 31 of K)
        for (int64_t k = 0; k < nb; ++k) {
            for (int e = bo[k]; e < bo[k + 1]; ++e)
                f(rs_of(bp[e]), (uint32_t)k | (bp[e] & 0x80000000u), bp[e] & SQD_NBR_MASK);
            for (int r = 0; r < norb; ++r)
                if ((bs[(size_t)k * sp->nw + (r >> 6)] >> (r & 63)) & 1ull) f(r * norb + r, (uint32_t)k, (uint32_t)k);
        }
    };
    each_beta([&](int rs, uint32_t, uint32_t) { at[rs + 1] += 1; });
    for (int k = 0; k < n2; ++k) at[k + 1] += at[k];
    std::vector<uint2> list(at[n2] + 1);
    {
        std::vector<int> pos(at.begin(), at.end() - 1);
        each_beta([&](int rs, uint32_t k, uint32_t l) { list[pos[rs]++] = make_uint2(k, l); });
    }
    std::vector<int> used, len;
    for (int k = 0; k < n2; ++k)
        if (at[k + 1] > at[k]) {
            used.push_back(k);
            len.push_back(at[k + 1] - at[k]);
        }
    const std::vector<int> rows = rows_longest_first(len);
    const int cap = split_cap(at[n2], 8);
    struct slice { int split, first, nblk; };
    std::vector<slice> sl;
    std::vector<int> cost;
    for (size_t r = 0; r < rows.size();) {
        const int k = split_of(len[rows[r]], cap);
        const int cols = (len[rows[r]] + (1 << k) - 1) >> k;
        sl.push_back({k, (int)r, (cols + 3) / 4});
        cost.push_back(cols + 4);
        r += 64 >> k;
    }
    const auto in = deal_bins(cost);
    std::vector<int> perm, split, blk{0}, bin;
    std::vector<uint2> ent;
    for (int q = 0; q < kBins; ++q) {
        bin.push_back((int)split.size());
        for (int k : in[q]) {
            const int g = 1 << sl[k].split;
            split.push_back(sl[k].split);
            const size_t e0 = ent.size();
            ent.resize(e0 + (size_t)sl[k].nblk * 256, make_uint2((uint32_t)nb, (uint32_t)nb));
            for (int lane = 0; lane < 64; ++lane) {
                const size_t r = (size_t)sl[k].first + lane / g;
                const bool any = r < rows.size();
                perm.push_back(any && lane % g == 0 ? used[rows[r]] : -1);
                if (!any) continue;
                const int rs = used[rows[r]];
                int c = 0;
                for (int e = at[rs] + lane % g; e < at[rs + 1]; e += g, ++c)
                    ent[e0 + (size_t)(c / 4) * 256 + (c % 4) * 64 + lane] = list[e];
            }
            blk.push_back(blk.back() + sl[k].nblk);
        }
    }
    bin.push_back((int)split.size());
    const int nslices = (int)split.size();
    // shape: pairs (rows) at a time, two workgroups per compute unit where they fit
    const size_t lim = (size_t)ctx->max_lds, accb = (size_t)nslices * 64 * sizeof(double);
    auto bytes = [&](int G) { return (size_t)2 * (nb + 1) * G * sizeof(double) + accb; };
    sp->rdm_keep = accb <= lim / 4;
    const size_t extra = sp->rdm_keep ? 0 : accb;
    sp->rdm_G = 0;
    for (int G : {8, 4, 2})
        if (!sp->rdm_G && bytes(G) - extra <= lim / 2) sp->rdm_G = G;
    for (int G : {4, 2, 1})
        if (!sp->rdm_G && bytes(G) - extra <= lim) sp->rdm_G = G;
    const int G = sp->rdm_G ? sp->rdm_G : 1;
    // alpha pairs p > q by pq, and chunks of a few batches each
    std::vector<std::vector<alpha_unit>> by(n2);
    int64_t total = 0;
    for (int64_t i = 0; i < na; ++i)
        for (int e = ao[i]; e < ao[i + 1]; ++e) {
            const int pq = (int)((ap[e] >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
            if (pq / norb <= pq % norb) continue;
            by[pq].push_back({(int)i, (ap[e] & SQD_NBR_MASK) | (ap[e] & 0x80000000u)});
            ++total;
        }
    const int64_t most = sp->rdm_keep ? std::max<int64_t>(G, (total / (4 * ctx->num_cu) + G - 1) / G * G) : G;
    std::vector<alpha_unit> units;
    std::vector<int4> chunks;
    for (int pq = 0; pq < n2; ++pq)
        for (size_t k = 0; k < by[pq].size(); k += most) {
            const int cnt = (int)std::min<size_t>(most, by[pq].size() - k);
            chunks.push_back(make_int4((int)units.size(), cnt, pq, 0));
            units.insert(units.end(), by[pq].begin() + k, by[pq].begin() + k + cnt);
        }
    std::stable_sort(chunks.begin(), chunks.end(), [](const int4& x, const int4& y) { return x.y > y.y; });
    // one allocation
    const host_part parts[] = {
        {ent.data(), sizeof(uint2) * ent.size()},        {units.data(), sizeof(alpha_unit) * units.size()},
        {chunks.data(), sizeof(int4) * chunks.size()},   {perm.data(), sizeof(int) * perm.size()},
        {split.data(), sizeof(int) * split.size()},      {blk.data(), sizeof(int) * blk.size()},
        {bin.data(), sizeof(int) * bin.size()}};
    sp->rdm_nslices = nslices;
    sp->rdm_nchunks = (int)chunks.size();
    return upload_parts(ctx, parts, 7, &sp->rdm_mem, sp->rdm_off, &sp->bytes);
}

}  // namespace

int sqd_rdm_impl(sqd_ctx* ctx, sqd_space* sp, const double* c, double* rdm1, double* rdm2) {
    int rc = sqd_build_values(ctx, sp);
    if (rc) return rc;
    const spin_tables& A = sp->sp[0];
    const spin_tables& B = sp->sp[1];
    const int64_t na = A.n, nb = B.n;
    const int norb = sp->norb;
    const int64_t n2 = (int64_t)norb * norb;
    hipStream_t s = ctx->stream;
    if (rdm2 && (rc = build_rdm_plan(ctx, sp))) return rc;
    // scratch: P_a (na^2), P_b (nb^2), C^T (dim), diagonal alpha pairs' sums
    const int64_t ldt = rdm2 ? (int64_t)sp->rdm_nslices * 64 : 0;
    const size_t bytes =
        sizeof(double) * ((size_t)na * na + (size_t)nb * nb + (size_t)sp->dim + (size_t)(na * ldt) + 64);
    void* scr = sqd_ctx_scratch(ctx, bytes, &rc);
    if (!scr) return sqd_fail(ctx, SQD_E_OOM, "RDM scratch allocation failed (" + std::to_string(bytes) + " bytes)");
    double* Pa = (double*)scr;
    double* Pb = Pa + na * na;
    double* Ct = Pb + nb * nb;
    double* t = Ct + sp->dim;
    hipLaunchKernelGGL(k_zero<double>, dim3(nblk(n2, 256)), dim3(256), 0, s, rdm1, n2);
    if (rdm2) hipLaunchKernelGGL(k_zero<double>, dim3(nblk(n2 * n2, 256)), dim3(256), 0, s, rdm2, n2 * n2);
    // overlaps of alpha rows and of beta columns
    auto gram = [&](const double* X, double* P, int64_t M, int64_t K) {
        const unsigned tm = nblk(M, kTM);
        hipLaunchKernelGGL(k_gram, dim3(tm * (tm + 1) / 2), dim3(256), 0, s, X, P, M, K);
    };
    gram(c, Pa, na, nb);
    hipLaunchKernelGGL(k_transpose_d, dim3(nblk(nb, 64), nblk(na, 64)), dim3(256), 0, s, c, Ct, na, nb);
    gram(Ct, Pb, nb, na);
    hipLaunchKernelGGL(k_rdm_same, dim3(nblk(na, 4)), dim3(256), 0, s, A.str, sp->nw, na, A.s_off, A.s_ent, A.d_off,
                       A.d_ent, Pa, norb, rdm1, rdm2);
    hipLaunchKernelGGL(k_rdm_same, dim3(nblk(nb, 4)), dim3(256), 0, s, B.str, sp->nw, nb, B.s_off, B.s_ent, B.d_off,
                       B.d_ent, Pb, norb, rdm1, rdm2);
    if (rdm2 && sp->rdm_nslices > 0) {
        const char* m = (const char*)sp->rdm_mem;
        const pair_table tab{sp->rdm_nslices, (const int*)(m + sp->rdm_off[3]), (const int*)(m + sp->rdm_off[4]),
                             (const int*)(m + sp->rdm_off[5]), (const int*)(m + sp->rdm_off[6]),
                             (const uint2*)(m + sp->rdm_off[0])};
        const alpha_unit* units = (const alpha_unit*)(m + sp->rdm_off[1]);
        const int4* chunks = (const int4*)(m + sp->rdm_off[2]);
        const size_t row = (size_t)(nb + 1) * sizeof(double);
        const size_t accb = sp->rdm_keep ? (size_t)sp->rdm_nslices * 64 * sizeof(double) : 0;
        auto launch = [&](auto g, auto staged) {
            constexpr int G = decltype(g)::value;
            constexpr bool kStaged = decltype(staged)::value;
            const size_t la = (kStaged ? 2 * G * row : 0) + accb, ld = kStaged ? G * row : 0;
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_rdm_ab<G, kStaged>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)la);
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_rdm_diag<G, kStaged>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)ld);
            if (sp->rdm_nchunks > 0)
                hipLaunchKernelGGL((k_rdm_ab<G, kStaged>), dim3(sp->rdm_nchunks), dim3(64 * kBins), la, s, c, nb, tab,
                                   units, chunks, norb, sp->rdm_keep ? 1 : 0, rdm2);
            hipLaunchKernelGGL((k_rdm_diag<G, kStaged>), dim3(nblk(na, G)), dim3(64 * kBins), ld, s, c, na, nb, tab, t);
        };
        using std::integral_constant;
        switch (sp->rdm_G) {
            case 8: launch(integral_constant<int, 8>(), std::true_type()); break;
            case 4: launch(integral_constant<int, 4>(), std::true_type()); break;
            case 2: launch(integral_constant<int, 2>(), std::true_type()); break;
            case 1: launch(integral_constant<int, 1>(), std::true_type()); break;
            default: launch(integral_constant<int, 1>(), std::false_type()); break;
        }
        // ranges of alpha strings, enough waves for the chip
        const int64_t per = std::max<int64_t>(16, (na * sp->rdm_nslices + 4095) / 4096);
        hipLaunchKernelGGL(k_rdm_occ, dim3(sp->rdm_nslices, nblk(na, (int)per)), dim3(64),
                           (size_t)norb * 64 * sizeof(double), s, t, tab, A.str, sp->nw, na, per, norb, rdm2);
    }
    SQD_HIP(ctx, hipGetLastError());
    return SQD_OK;
}
