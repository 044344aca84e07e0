// Host side of the sliced tables: the order of the rows, how many lanes a long
// row takes and which wave of a workgroup walks which slice.
#pragma once

#include <algorithm>
#include <cstring>
#include <vector>

#include "sqd_internal.h"

// Arrays planned on the host, side by side in one device allocation.  *mem is set
// when all of them are there: after a failure nothing is held and *mem is as it was.
struct host_part {
    const void* data;
    size_t bytes;
};
inline int upload_parts(sqd_ctx* ctx, const host_part* parts, int n, void** mem, size_t* off, int64_t* counter) {
    size_t total = 0;
    for (int k = 0; k < n; ++k) {
        off[k] = total;
        total += (parts[k].bytes + 255) & ~(size_t)255;
    }
    total += 256;
    std::vector<char> all(total);
    for (int k = 0; k < n; ++k)
        if (parts[k].bytes) std::memcpy(all.data() + off[k], parts[k].data, parts[k].bytes);
    void* p = nullptr;
    const int rc = sqd_alloc(ctx, &p, total, nullptr);
    if (rc) return rc;
    const hipError_t e = sqd_copy_now(ctx, p, all.data(), total, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(p);
        return sqd_hip_fail(ctx, e, "upload of a host plan");
    }
    *mem = p;
    *counter += (int64_t)total;
    return SQD_OK;
}

// The schedule s from chunks of G; the one it replaces is freed once the new one
// is whole, and stays if that fails.
template <typename K>
int upload_schedule(sqd_ctx* ctx, int G, const std::vector<int2>& grp, const std::vector<K>& key, ab_schedule<K>& s,
                    int64_t* counter) {
    const host_part parts[] = {{grp.data(), sizeof(int2) * grp.size()}, {key.data(), sizeof(K) * key.size()}};
    size_t off[2];
    ab_schedule<K> t;
    const int rc = upload_parts(ctx, parts, 2, &t.mem, off, &t.bytes);
    if (rc) return rc;
    t.G = G;
    t.n = (int)key.size();
    t.grp = reinterpret_cast<const int2*>(static_cast<char*>(t.mem) + off[0]);
    t.key = reinterpret_cast<const K*>(static_cast<char*>(t.mem) + off[1]);
    if (s.mem) (void)hipFree(s.mem);
    *counter += t.bytes - s.bytes;
    s = t;
    return SQD_OK;
}

// Rows by decreasing length (ties by index): a counting sort.
inline std::vector<int> rows_longest_first(const std::vector<int>& len) {
    const int most = len.empty() ? 0 : *std::max_element(len.begin(), len.end());
    std::vector<int> at(most + 2, 0), rows(len.size());
    for (int l : len) at[most - l + 1] += 1;
    for (int k = 0; k <= most; ++k) at[k + 1] += at[k];
    for (size_t r = 0; r < len.size(); ++r) rows[at[most - len[r]]++] = (int)r;
    return rows;
}

// Lanes per row (log2): the fewest that keep a lane's entries at or below cap.
inline int split_of(int len, int cap) {
    int k = 0;
    while (k < 6 && ((len + (1 << k) - 1) >> k) > cap) ++k;
    return k;
}

// Slices dealt into bins, the costliest into the lightest bin; the heaviest
// bins are placed beside the lightest, so that pairs and fours of adjacent
// bins are even too.
inline std::vector<std::vector<int>> deal_bins(const std::vector<int>& cost) {
    std::vector<int> order(cost.size()), load(kBins, 0), rank(kBins);
    for (size_t k = 0; k < order.size(); ++k) order[k] = (int)k;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost[x] > cost[y]; });
    std::vector<std::vector<int>> in(kBins), out(kBins);
    for (int k : order) {
        const int q = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        in[q].push_back(k);
        load[q] += cost[k];
    }
    for (int q = 0; q < kBins; ++q) rank[q] = q;
    std::stable_sort(rank.begin(), rank.end(), [&](int x, int y) { return load[x] > load[y]; });
    static constexpr int kPlace[kBins] = {0, 15, 7, 8, 3, 12, 4, 11, 1, 14, 6, 9, 2, 13, 5, 10};
    for (int q = 0; q < kBins; ++q) out[q] = in[rank[kPlace[q]]];
    return out;
}

// Entries a lane of a table with split rows takes at most.  A wavefront walks
// a slice at the pace of its longest lane, and the rows of sampled sets are
// uneven: the Hartree-Fock string reaches half of the set, the mean row a
// tenth.  A thirty-second of all columns leaves each of sixteen waves about
// two slices of that length, so the waves of a workgroup end together, and
// only the long rows pay for the sums across lanes.
inline int split_cap(int64_t entries, int least) { return (int)std::max<int64_t>(least, (entries + 2047) / 2048); }

// Slices of the sliced singles (ab_table) over rows sorted by length, dealt into bins.
struct ab_plan {
    std::vector<int> perm, split, blk{0}, cols, slot, bin, order;
};
inline ab_plan plan_ab(const std::vector<int>& rows, const int* off, int cap) {
    const int n = (int)rows.size();
    struct slice { int split, at, cols; };
    std::vector<slice> sl;
    std::vector<int> cost;
    for (int at = 0; at < n;) {
        const int len = off[rows[at] + 1] - off[rows[at]];   // the longest of the slice
        const int k = split_of(len, cap);
        sl.push_back({k, at, (len + (1 << k) - 1) >> k});
        cost.push_back(sl.back().cols + 2);
        at += 64 >> k;
    }
    const auto in = deal_bins(cost);
    ab_plan p;
    p.order.resize(sl.size());
    for (int q = 0; q < kBins; ++q) {
        p.bin.push_back((int)p.split.size());
        for (int k : in[q]) {
            p.order[k] = (int)p.split.size();   // (sl: the longest rows first)
            p.slot.push_back((int)p.perm.size());
            for (int j = 0; j < (64 >> sl[k].split); ++j)
                p.perm.push_back(sl[k].at + j < n ? rows[sl[k].at + j] : n);
            p.split.push_back(sl[k].split);
            p.cols.push_back(sl[k].cols);
            p.blk.push_back(p.blk.back() + (sl[k].cols + 3) / 4);
        }
    }
    p.bin.push_back((int)p.split.size());
    for (int q = 0; q <= kBins; ++q) p.bin.push_back(p.blk[p.bin[q]]);
    while (p.perm.size() % 64) p.perm.push_back(n);
    return p;
}

// Cross-spin tables (spin_tables::ws64, ws32) of the spins whose rows of C fit the
// LDS four at a time, up to 256 MiB each, in one allocation.  Elsewhere, and where
// that allocation fails, the row-staged kernel sums them itself (norb reads per value
// and workgroup); the windowed kernel has its own.
inline void alloc_cross_tables(sqd_ctx* ctx, sqd_space* sp) {
    const size_t n2 = (size_t)sp->norb * sp->norb;
    size_t total = 0, bytes64[2] = {}, bytes32[2] = {};
    for (int spin = 0; spin < 2; ++spin) {
        const spin_tables& t = sp->sp[spin];
        if (t.alias) continue;
        const size_t lds4 = ((size_t)sp->sp[1 - spin].n + 1 + n2) * 4;   // four rows, elements
        const size_t m = (size_t)t.n * n2;
        if (lds4 * sizeof(double) <= (size_t)ctx->max_lds && m * sizeof(double) <= (256u << 20))
            bytes64[spin] = (m * sizeof(double) + 255) & ~(size_t)255;
        if (lds4 * sizeof(float) <= (size_t)ctx->max_lds && m * sizeof(float) <= (256u << 20))
            bytes32[spin] = (m * sizeof(float) + 255) & ~(size_t)255;
        total += bytes64[spin] + bytes32[spin];
    }
    const std::string err = ctx->err;
    if (!total || sqd_alloc(ctx, &sp->cross_mem, total, &sp->bytes) != SQD_OK) {
        ctx->err = err;   // no failure of the call
        return;
    }
    char* at = static_cast<char*>(sp->cross_mem);
    for (int spin = 0; spin < 2; ++spin) {
        spin_tables& t = sp->sp[spin];
        if (bytes64[spin]) t.ws64 = reinterpret_cast<double*>(at);
        at += bytes64[spin];
        if (bytes32[spin]) t.ws32 = reinterpret_cast<float*>(at);
        at += bytes32[spin];
        if (t.alias) {
            t.ws64 = sp->sp[0].ws64;
            t.ws32 = sp->sp[0].ws32;
        }
    }
}

// (counting bits with the instruction: every host of these devices has it)
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#pragma clang attribute push(__attribute__((target("popcnt"))), apply_to = function)
#endif
inline int bits_in_common(const uint64_t* a, const uint64_t* b, size_t words) {
    int c = 0;
    for (size_t w = 0; w < words; ++w) c += __builtin_popcountll(a[w] & b[w]);
    return c;
}

// Blocks of G alpha singles of one pair, or of G sources by two pairs that both
// excite, from the singles in gather form (nbr | pair << 19 | negative << 31, in
// CSR order): grp lists 2 G singles a block (CSR position, gather form; -1 where
// none), pairs the one or two pairs.  In a round the pairs of each orbital are
// matched, the one with the most sources left with the one that shares most of
// them, as long as they fill a block; the rounds go over the created and the
// annihilated orbital by turns, until one adds less than 4% of the singles (eight
// at most).  What is left goes to blocks of one pair.  2000 strings of 24
// orbitals: 62% of the singles in blocks of two pairs and 6100 walks of the beta
// table instead of 8800, planned in 0.6 ms; choosing the best two of all pairs
// each time finds 76% in 2.4 ms (5000 strings of 36 orbitals: 3.6 and 38 ms), and
// four pairs to a block save 2% of the reads more.
inline void plan_ab_blocks(const std::vector<uint32_t>& pk, int64_t n, int norb, int G, std::vector<int2>& grp,
                           std::vector<int2>& pairs) {
    const int npair = norb * norb;
    const size_t words = (size_t)(n + 63) / 64;
    auto src_of = [&](int e) { return pk[e] & SQD_NBR_MASK; };
    auto pair_of = [&](int e) { return (int)((pk[e] >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK); };
    // the sources of each pair as bits, and its singles by source: the single of
    // source j is at the rank of its bit
    std::vector<uint64_t> all((size_t)npair * words, 0);
    std::vector<int> rank((size_t)npair * words), first(npair + 1, 0), ent(pk.size()), count(npair);
    for (size_t e = 0; e < pk.size(); ++e) {
        const uint32_t j = src_of((int)e);
        all[pair_of((int)e) * words + (j >> 6)] |= 1ull << (j & 63);
        first[pair_of((int)e) + 1] += 1;
    }
    for (int p = 0; p < npair; ++p) {
        count[p] = first[p + 1];
        first[p + 1] += first[p];
        int at = first[p];
        if (!count[p]) continue;
        for (size_t w = 0; w < words; ++w) {
            rank[p * words + w] = at;
            at += __builtin_popcountll(all[p * words + w]);
        }
    }
    auto place = [&](int p, uint32_t j) {
        return rank[p * words + (j >> 6)] + __builtin_popcountll(all[p * words + (j >> 6)] & ((1ull << (j & 63)) - 1));
    };
    for (size_t e = 0; e < pk.size(); ++e) ent[place(pair_of((int)e), src_of((int)e))] = (int)e;
    std::vector<uint64_t> left = all;
    grp.reserve(pk.size() * 2);
    auto add = [&](int p, int q, const uint32_t* src, int m) {
        for (int half = 0; half < 2; ++half)
            for (int r = 0; r < G; ++r) {
                if (r < m && (half == 0 || q >= 0)) {
                    const int e = ent[place(half ? q : p, src[r])];
                    grp.push_back(make_int2(e, (int)pk[e]));
                } else {
                    grp.push_back(make_int2(-1, 0));
                }
            }
        pairs.push_back(make_int2(p, q));
    };
    std::vector<uint32_t> src(n);
    std::vector<int> line;
    size_t before = 0;
    for (int round = 0; round < 8; ++round) {
        for (int i = 0; i < norb; ++i) {
            // the pairs of one orbital: by turns with i created and annihilated
            line.clear();
            for (int a = 0; a < norb; ++a) {
                const int p = round % 2 ? a * norb + i : i * norb + a;
                if (count[p] >= G) line.push_back(p);
            }
            while (line.size() > 1) {
                size_t at = 0, with = 0;
                for (size_t k = 1; k < line.size(); ++k)
                    if (count[line[k]] > count[line[at]]) at = k;
                const int p = line[at];
                std::swap(line[at], line.back());
                line.pop_back();
                uint64_t* lp = left.data() + p * words;
                int most = G - 1;
                for (size_t k = 0; k < line.size(); ++k) {
                    if (count[line[k]] <= most) continue;
                    const int c = bits_in_common(lp, left.data() + line[k] * words, words);
                    if (c > most) most = c, with = k;
                }
                if (most < G) continue;
                const int q = line[with];
                std::swap(line[with], line.back());
                line.pop_back();
                uint64_t* lq = left.data() + q * words;
                const int m = most / G * G;
                int got = 0;
                for (size_t w = 0; w < words && got < m; ++w) {
                    uint64_t taken = 0;
                    for (uint64_t x = lp[w] & lq[w]; x && got < m; x &= x - 1) {
                        src[got++] = (uint32_t)(64 * w + __builtin_ctzll(x));
                        taken |= x & (~x + 1);
                    }
                    lp[w] &= ~taken;
                    lq[w] &= ~taken;
                }
                for (int k = 0; k < m; k += G) add(p, q, src.data() + k, G);
                count[p] -= m;
                count[q] -= m;
            }
        }
        if ((grp.size() - before) * 25 < pk.size()) break;
        before = grp.size();
    }
    for (int p = 0; p < npair; ++p) {
        int got = 0;
        for (size_t w = 0; w < words && got < count[p]; ++w)
            for (uint64_t x = left[p * words + w]; x; x &= x - 1) src[got++] = (uint32_t)(64 * w + __builtin_ctzll(x));
        for (int k = 0; k < got; k += G) add(p, -1, src.data() + k, std::min(G, got - k));
    }
}
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#pragma clang attribute pop
#endif
