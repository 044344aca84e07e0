// Host side of the sliced tables: the order of the rows, how many lanes a long
// row takes and which wave of a workgroup walks which slice.
#pragma once

#include <algorithm>
#include <cstring>
#include <memory>
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
    void* p = nullptr;
    const int rc = sqd_alloc(ctx, &p, total, nullptr);
    if (rc) return rc;
    hipError_t e = hipSuccess;
    // neighbours of up to 64 KiB in all in one copy (of 10 us each); gathering more costs
    // as much (a first RDM on 350 x 283 strings, whose plan has seven arrays: 395 us with
    // a copy each, 335 so)
    constexpr size_t kGather = 64 * 1024;
    std::vector<char> all;
    for (int k = 0; k < n && e == hipSuccess;) {
        int last = k + 1;
        while (last < n && off[last] + parts[last].bytes - off[k] <= kGather) ++last;
        const void* src = parts[k].data;
        size_t bytes = parts[k].bytes;
        if (last > k + 1) {
            bytes = off[last - 1] + parts[last - 1].bytes - off[k];
            all.assign(bytes, 0);
            for (int q = k; q < last; ++q)
                if (parts[q].bytes) std::memcpy(all.data() + off[q] - off[k], parts[q].data, parts[q].bytes);
            src = all.data();
        }
        e = sqd_copy_now(ctx, static_cast<char*>(p) + off[k], src, bytes, hipMemcpyHostToDevice);
        k = last;
    }
    if (e != hipSuccess) {
        (void)hipFree(p);
        return sqd_hip_fail(ctx, e, "upload of a host plan");
    }
    *mem = p;
    *counter += (int64_t)total;
    return SQD_OK;
}

// The schedule s from chunks of G (n2 of them: ab_schedule::n2); the one it replaces
// is freed once the new one is whole, and stays if that fails.
template <typename K>
int upload_schedule(sqd_ctx* ctx, int G, const int2* grp, size_t size, int n2, const std::vector<K>& key,
                    ab_schedule<K>& s, int64_t* counter) {
    const host_part parts[] = {{grp, sizeof(int2) * size}, {key.data(), sizeof(K) * key.size()}};
    size_t off[2];
    ab_schedule<K> t;
    const int rc = upload_parts(ctx, parts, 2, &t.mem, off, &t.bytes);
    if (rc) return rc;
    t.G = G;
    t.n = (int)key.size();
    t.n2 = n2;
    t.grp = reinterpret_cast<const int2*>(static_cast<char*>(t.mem) + off[0]);
    t.key = reinterpret_cast<const K*>(static_cast<char*>(t.mem) + off[1]);
    if (s.mem) (void)hipFree(s.mem);
    *counter += t.bytes - s.bytes;
    s = t;
    return SQD_OK;
}

template <typename K>
int upload_schedule(sqd_ctx* ctx, int G, const std::vector<int2>& grp, const std::vector<K>& key, ab_schedule<K>& s,
                    int64_t* counter) {
    return upload_schedule(ctx, G, grp.data(), grp.size(), 0, key, s, counter);
}

// Device arrays in few allocations, listed in mem as they are made.  The runtime keeps
// blocks of less than 2 MiB at hand; each larger one costs up to 0.3 ms to map and as
// much to unmap.  So arrays below that go side by side into blocks of as much, and the
// larger ones all into one.  Building and freeing a space of other strings each time,
// ms, an allocation an array / one for all / so: 1600 + 1600 strings of 16 orbitals
// 2.1 / 3.2 / 2.1, 2300 + 2300: 7.0 / 5.6 / 4.7, 4000 + 4000 of 20: 10.9 / 6.0 / 5.9.
using array_list = std::vector<std::pair<void**, size_t>>;
constexpr size_t kBlock = 2000u << 10;
inline int alloc_arrays(sqd_ctx* ctx, const array_list& arrays, std::vector<void*>& mem, int64_t* counter) {
    auto padded = [](size_t bytes) { return (bytes + 255) & ~(size_t)255; };
    auto place = [&](const std::vector<size_t>& which) -> int {
        size_t total = 0;
        for (size_t k : which) total += padded(arrays[k].second);
        void* p = nullptr;
        const int rc = sqd_alloc(ctx, &p, total, counter);
        if (rc) return rc;
        mem.push_back(p);
        char* at = static_cast<char*>(p);
        for (size_t k : which) {
            *arrays[k].first = at;
            at += padded(arrays[k].second);
        }
        return SQD_OK;
    };
    std::vector<size_t> large, block;
    size_t filled = 0;
    int rc;
    for (size_t k = 0; k < arrays.size(); ++k) {
        const size_t bytes = padded(arrays[k].second);
        if (bytes > kBlock) {
            large.push_back(k);
            continue;
        }
        if (filled + bytes > kBlock) {
            if ((rc = place(block))) return rc;
            block.clear();
            filled = 0;
        }
        block.push_back(k);
        filled += bytes;
    }
    if (!block.empty() && (rc = place(block))) return rc;
    return large.empty() ? SQD_OK : place(large);
}

// The sliced tables and values of a spin, as above; but the runtime also keeps up to 64
// MiB of freed larger allocations, by size, and those of a space with up to 18 MiB a spin
// are found there again if each array has its own.  Build and free, one space after the
// other, ms, larger arrays in one allocation / in one each: 1800 + 1800 strings of 16
// orbitals (13 MiB a spin) 3.1 / 2.5, 2000 + 2000 (16) 3.9 / 2.7, 2200 + 2200 (18.5) 4.1 /
// 4.3, 2400 + 2400 (21) 4.2 / 7.2.
inline int alloc_tables(sqd_ctx* ctx, const array_list& arrays, std::vector<void*>& mem, int64_t* counter) {
    size_t total = 0;
    for (const auto& q : arrays) total += q.second;
    if (total > (size_t)18 << 20) return alloc_arrays(ctx, arrays, mem, counter);
    array_list small;
    for (const auto& q : arrays) {
        int rc;
        if (q.second <= kBlock) small.push_back(q);
        else if ((rc = alloc_arrays(ctx, {q}, mem, counter))) return rc;
    }
    return alloc_arrays(ctx, small, mem, counter);
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
// LDS four at a time, up to 256 MiB each, in one allocation.  Elsewhere (one-launch
// products that stage two rows among them), and where that allocation fails, the
// workgroups sum them themselves (norb reads per value); the windowed kernel has its
// own.
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
// Blocks of G alpha singles of one pair, or of G sources by two pairs that both
// excite, from the singles in gather form (nbr | pair << 17 | negative << 31, in
// CSR order).  In a round the pairs of each orbital are matched, the one with the
// most sources left with the one that shares most of them, as long as they fill a
// block; the rounds go over the created and the annihilated orbital by turns, until
// one adds less than 4% of the singles (eight at most).  What is left goes to blocks
// of one pair.  2000 strings of 16 orbitals: 62% of the singles in blocks of two pairs
// and 6100 walks of the beta table instead of 8800 (24 orbitals: 36%); choosing the
// best two of all pairs each time finds 76% in four times the time, and four pairs to
// a block save 2% of the reads more.
struct ab_block_plan {
    std::unique_ptr<int2[]> grp;   // 2 G singles of each block of two pairs, then G of each of one (sqd_space::abb)
    size_t size = 0;
    int n2 = 0;                    // blocks of two pairs
    std::vector<int2> pairs;       // the pairs of each block (second -1: one)
};
inline ab_block_plan plan_ab_blocks(const std::vector<uint32_t>& pk, int64_t n, int norb, int G) {
    const int npair = norb * norb;
    const size_t words = (size_t)(n + 63) / 64;
    // the singles by pair.  The strings of a pair's targets are those of its sources
    // plus one number, and the strings ascend, so CSR order is the order of the sources
    std::vector<int> first(npair + 1, 0), count(npair), at(npair);
    for (uint32_t x : pk) first[((x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK) + 1] += 1;
    size_t blocks = 0;   // at most
    for (int p = 0; p < npair; ++p) {
        count[p] = first[p + 1];
        blocks += (size_t)(count[p] + G - 1) / G;
        first[p + 1] += first[p];
        at[p] = first[p];
    }
    // all: the sources of each pair as bits; left: those not in a block; rank: the
    // single of the first source of a word
    std::unique_ptr<int2[]> one(new int2[pk.size() + 1]);
    std::vector<uint64_t> all((size_t)npair * words, 0);
    for (size_t e = 0; e < pk.size(); ++e) {
        const uint32_t x = pk[e], j = x & SQD_NBR_MASK;
        const int p = (int)((x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK);
        one[at[p]++] = make_int2((int)e, (int)x);
        all[p * words + (j >> 6)] |= 1ull << (j & 63);
    }
    std::vector<uint64_t> left = all, any(words), many(words), bits;
    std::unique_ptr<int[]> rank(new int[(size_t)npair * words]);
    std::vector<int> line, used, most_of(npair);
    for (int p = 0; p < npair; ++p) {
        if (count[p] < G) continue;   // (never matched)
        int r = first[p];
        for (size_t w = 0; w < words; ++w) {
            rank[p * words + w] = r;
            r += __builtin_popcountll(all[p * words + w]);
        }
    }
    ab_block_plan plan;
    plan.grp.reset(new int2[blocks * G + 1]);
    plan.pairs.reserve(blocks);
    int2* out = plan.grp.get();
    int matched = 0;
    for (int round = 0, before = 0; round < 8; ++round) {
        for (int i = 0; i < norb; ++i) {
            // the pairs of one orbital: by turns with i created and annihilated
            line.clear();
            for (int a = 0; a < norb; ++a) {
                const int p = round % 2 ? a * norb + i : i * norb + a;
                if (count[p] >= G) line.push_back(p);
            }
            if (line.size() < 2) continue;
            // many: the sources that two pairs or more share; most_of: as many can a
            // pair share with another
            std::fill(any.begin(), any.end(), 0);
            std::fill(many.begin(), many.end(), 0);
            for (int p : line)
                for (size_t w = 0; w < words; ++w) {
                    const uint64_t x = left[p * words + w];
                    many[w] |= any[w] & x;
                    any[w] |= x;
                }
            size_t keep = 0;
            for (int p : line) {
                int c = 0;
                for (size_t w = 0; w < words; ++w) c += __builtin_popcountll(left[p * words + w] & many[w]);
                most_of[p] = c;
                if (c >= G) line[keep++] = p;
            }
            line.resize(keep);
            while (line.size() > 1) {
                size_t big = 0, with = 0;
                for (size_t k = 1; k < line.size(); ++k)
                    if (count[line[k]] > count[line[big]]) big = k;
                const int p = line[big];
                std::swap(line[big], line.back());
                line.pop_back();
                uint64_t* lp = left.data() + p * words;
                // (a pair of few sources: the words that hold them)
                const bool few = (size_t)most_of[p] < words;
                if (few) {
                    used.clear();
                    bits.clear();
                    for (size_t w = 0; w < words; ++w)
                        if (lp[w] & many[w]) used.push_back((int)w), bits.push_back(lp[w] & many[w]);
                }
                int most = G - 1;
                for (size_t k = 0; k < line.size(); ++k) {
                    if (most_of[line[k]] <= most) continue;
                    const uint64_t* lk = left.data() + line[k] * words;
                    int c = 0;
                    if (few)
                        for (size_t u = 0; u < used.size(); ++u) c += __builtin_popcountll(bits[u] & lk[used[u]]);
                    else
                        for (size_t w = 0; w < words; ++w) c += __builtin_popcountll(lp[w] & lk[w]);
                    if (c > most) most = c, with = k;
                }
                if (most < G) continue;
                const int q = line[with];
                std::swap(line[with], line.back());
                line.pop_back();
                uint64_t* lq = left.data() + q * words;
                const uint64_t *ap = all.data() + p * words, *aq = all.data() + q * words;
                const int *rp = rank.get() + p * words, *rq = rank.get() + q * words;
                const int m = most / G * G;
                int got = 0;
                for (size_t w = 0; w < words && got < m; ++w) {
                    const uint64_t both = lp[w] & lq[w];
                    uint64_t x = both;
                    for (; x && got < m; x &= x - 1) {
                        const uint64_t below = (x & (~x + 1)) - 1;
                        out[0] = one[rp[w] + __builtin_popcountll(ap[w] & below)];
                        out[G] = one[rq[w] + __builtin_popcountll(aq[w] & below)];
                        ++out;
                        if (++got % G == 0) out += G;
                    }
                    lp[w] &= ~(both & ~x);
                    lq[w] &= ~(both & ~x);
                }
                plan.pairs.insert(plan.pairs.end(), m / G, make_int2(p, q));
                count[p] -= m;
                count[q] -= m;
                matched += 2 * m;
            }
        }
        if ((matched - before) * (int64_t)25 < (int64_t)pk.size()) break;
        before = matched;
    }
    plan.n2 = (int)plan.pairs.size();
    for (int p = 0; p < npair; ++p) {
        const int2* from = one.get() + first[p];
        int2* const to = out;
        if (count[p] == first[p + 1] - first[p]) {
            out = std::copy(from, from + count[p], out);
        } else {
            for (size_t w = 0; w < words; ++w)
                for (uint64_t x = left[p * words + w]; x; x &= x - 1)
                    *out++ = one[rank[p * words + w] + __builtin_popcountll(all[p * words + w] & ((x & (~x + 1)) - 1))];
        }
        while ((out - to) % G) *out++ = make_int2(-1, 0);
        plan.pairs.insert(plan.pairs.end(), (out - to) / G, make_int2(p, -1));
    }
    plan.size = out - plan.grp.get();
    return plan;
}
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#pragma clang attribute pop
#endif
