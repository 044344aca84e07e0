"""The host side of the kernels' plans (csrc/slices.h), compiled for the host and
run without a GPU: device memory is host memory, and allocations and copies fail
where a test wants them to."""
import os
import subprocess

import pytest

from paper_2601_16169_amd import build

STUBS = r"""
#include <cstdio>
#include <cstdlib>
#include "slices.h"

static int allocs_left = 1 << 30, copies_left = 1 << 30, held = 0;
int sqd_fail(sqd_ctx*, int code, const std::string&) { return code; }
int sqd_hip_fail(sqd_ctx*, hipError_t, const char*) { return SQD_E_HIP; }
int sqd_alloc(sqd_ctx*, void** p, size_t bytes, int64_t* counter) {
    if (allocs_left-- <= 0) return SQD_E_OOM;
    *p = std::malloc(bytes);
    ++held;
    if (counter) *counter += (int64_t)bytes;
    return SQD_OK;
}
hipError_t sqd_copy_now(sqd_ctx*, void* dst, const void* src, size_t bytes, hipMemcpyKind) {
    if (copies_left-- <= 0) return hipErrorUnknown;
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
    std::free(p);
    --held;
    return hipSuccess;
}
#define REQUIRE(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
"""


def _run(tmp_path, body):
    src = tmp_path / "main.cpp"
    src.write_text(STUBS + body)
    exe = tmp_path / "main"
    cmd = [build.hipcc(), "--offload-host-only", "-x", "hip", "-O1", "-fPIC", "-std=c++17", "-w", "-I", build.CSRC, "-c",
           str(src), "-o", str(tmp_path / "main.o")]
    subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=120)
    subprocess.run(["g++", str(tmp_path / "main.o"), "-o", str(exe)], check=True, capture_output=True, text=True,
                   timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


def test_schedule_is_whole_or_as_before(tmp_path):
    """A schedule that cannot be allocated or copied leaves the one before it (or
    none) in place, and holds no memory."""
    _run(tmp_path, r"""
int main() {
    ab_schedule<int2> s;
    int64_t bytes = 0;
    std::vector<int2> grp(16, make_int2(3, 4)), key(2, make_int2(5, -1));
    for (int which = 0; which < 2; ++which) {          // the first schedule of a space
        (which ? copies_left : allocs_left) = 0;
        REQUIRE(upload_schedule(nullptr, 4, grp, key, s, &bytes) != SQD_OK);
        REQUIRE(!s.mem && !s.built(4) && s.n == 0 && held == 0 && bytes == 0);
        allocs_left = copies_left = 1 << 30;
    }
    REQUIRE(upload_schedule(nullptr, 4, grp, key, s, &bytes) == SQD_OK);
    REQUIRE(s.built(4) && s.n == 2 && held == 1 && bytes == s.bytes);
    REQUIRE(s.grp[15].x == 3 && s.key[1].x == 5 && s.key[1].y == -1);
    const void* mem = s.mem;
    std::vector<int2> grp2(4, make_int2(7, 8)), key2(1, make_int2(9, 10));
    for (int which = 0; which < 2; ++which) {          // one that replaces it
        (which ? copies_left : allocs_left) = 0;
        REQUIRE(upload_schedule(nullptr, 2, grp2, key2, s, &bytes) != SQD_OK);
        REQUIRE(s.mem == mem && s.built(4) && s.n == 2 && s.key[1].x == 5 && held == 1 && bytes == s.bytes);
        allocs_left = copies_left = 1 << 30;
    }
    REQUIRE(upload_schedule(nullptr, 2, grp2, key2, s, &bytes) == SQD_OK);
    REQUIRE(s.built(2) && !s.built(4) && s.n == 1 && s.grp[3].y == 8 && s.key[0].y == 10 && held == 1);
    REQUIRE(upload_schedule(nullptr, 2, {}, {}, s, &bytes) == SQD_OK);      // no singles: built and empty
    REQUIRE(s.built(2) && s.n == 0 && held == 1 && bytes == s.bytes);
    return 0;
}
""")


def test_slices_of_whole_rows_are_listed_longest_first(tmp_path):
    """The order in which the row-staged alpha-beta kernel deals its slices: every
    slice once, by decreasing columns, so that eight waves of eight slices each end a
    pass within one slice of each other.  Uneven rows (the first reaches all others),
    rows of one length, one string."""
    _run(tmp_path, r"""
int main() {
    for (int n : {1, 64, 65, 700, 5000}) {
        for (int uneven = 0; uneven < 2; ++uneven) {
            std::vector<int> len(n), off(n + 1, 0);
            for (int r = 0; r < n; ++r) len[r] = uneven ? n / (1 + r) : 7;
            for (int r = 0; r < n; ++r) off[r + 1] = off[r] + len[r];
            const ab_plan p = plan_ab(rows_longest_first(len), off.data(), 1 << 30);
            const int ns = (int)p.split.size();
            REQUIRE((int)p.order.size() == ns && ns == (n + 63) / 64);
            std::vector<int> seen(ns, 0);
            for (int k = 0; k < ns; ++k) {
                REQUIRE(p.order[k] >= 0 && p.order[k] < ns && !seen[p.order[k]]++);
                REQUIRE(p.split[p.order[k]] == 0);
                REQUIRE(k == 0 || p.cols[p.order[k]] <= p.cols[p.order[k - 1]]);
            }
            const int groups = (ns + 63) / 64;
            std::vector<int> load(8 * groups, 0);
            for (int k = 0; k < ns; ++k) load[k % (8 * groups)] += p.cols[p.order[k]];
            int lo = 1 << 30, hi = 0;
            for (int x : load) lo = std::min(lo, x), hi = std::max(hi, x);
            REQUIRE(hi - lo <= p.cols[p.order[0]]);
        }
    }
    return 0;
}
""")


def test_cross_tables_are_optional(tmp_path):
    """A space whose cross-spin tables cannot be allocated is built without them (the
    kernels then sum them), and the call leaves no error; where they can, each spin has
    its own, aligned, within one allocation."""
    _run(tmp_path, r"""
int main() {
    sqd_ctx ctx;
    ctx.max_lds = 160 * 1024;
    ctx.err = "earlier";
    for (int alias = 0; alias < 2; ++alias) {
        sqd_space sp;
        sp.norb = 10;
        sp.sp[0].n = 77;
        sp.sp[1].n = alias ? 77 : 4000;      // rows of 4000: four fit, and four of 77
        sp.sp[1].alias = alias;
        allocs_left = 0;
        alloc_cross_tables(&ctx, &sp);
        REQUIRE(!sp.cross_mem && sp.bytes == 0 && ctx.err == "earlier");
        for (const auto& t : sp.sp) REQUIRE(!t.ws64 && !t.ws32);
        allocs_left = 1 << 30;
        alloc_cross_tables(&ctx, &sp);
        REQUIRE(sp.cross_mem && held == 1 && ctx.err == "earlier");
        const char *from = (const char*)sp.cross_mem, *to = from + sp.bytes;
        for (const auto& t : sp.sp) {
            REQUIRE((const char*)t.ws64 >= from && (const char*)(t.ws64 + t.n * 100) <= to);
            REQUIRE((const char*)t.ws32 >= from && (const char*)(t.ws32 + t.n * 100) <= to);
            REQUIRE(((const char*)t.ws64 - from) % 256 == 0 && ((const char*)t.ws32 - from) % 256 == 0);
        }
        REQUIRE((sp.sp[0].ws64 == sp.sp[1].ws64) == (alias == 1));
        hipFree(sp.cross_mem);
    }
    sqd_space sp;                             // rows too long for four: FP32 alone, or none
    sp.norb = 10;
    sp.sp[0].n = 6000;
    sp.sp[1].n = 12000;
    alloc_cross_tables(&ctx, &sp);
    REQUIRE(sp.cross_mem && !sp.sp[0].ws64 && !sp.sp[0].ws32 && !sp.sp[1].ws64 && sp.sp[1].ws32);
    hipFree(sp.cross_mem);
    sqd_space none;
    none.norb = 10;
    none.sp[0].n = none.sp[1].n = 12000;
    alloc_cross_tables(&ctx, &none);
    REQUIRE(!none.cross_mem && held == 0);
    return 0;
}
""")


def test_parts_arrive_whole(tmp_path):
    """Host arrays side by side on the device, copied singly or gathered: all bytes
    arrive, aligned, whatever the sizes around the limit of a gathered copy, empty ones
    among them; where a copy fails nothing is held and the caller's pointer stays."""
    _run(tmp_path, r"""
int main() {
    const size_t lim = 64 << 10;
    const std::vector<std::vector<size_t>> cases = {
        {}, {0, 0}, {1}, {lim}, {lim + 1}, {lim - 256, 256}, {lim - 256, 257}, {1, 0, 255, 256, 257, 0},
        {3 * lim, 5, 0, lim / 2, lim / 2, 7, 2 * lim, 9}, {5, 3 * lim, 8, 8}, {lim / 2, lim / 2, lim / 2, lim / 2, lim / 2}};
    for (const auto& sizes : cases) {
        std::vector<std::vector<unsigned char>> data;
        std::vector<host_part> parts;
        size_t sum = 0;
        for (size_t b : sizes) {
            data.emplace_back(b);
            for (size_t i = 0; i < b; ++i) data.back()[i] = (unsigned char)(1 + (i * 7 + data.size()) % 251);
            sum += b;
        }
        for (const auto& d : data) parts.push_back({d.data(), d.size()});
        for (int fail = 0;; ++fail) {
            std::vector<size_t> off(sizes.size() + 1, 0);
            void* mem = nullptr;
            int64_t bytes = 0;
            copies_left = fail;
            const int rc = upload_parts(nullptr, parts.data(), (int)parts.size(), &mem, off.data(), &bytes);
            const int copies = fail - copies_left;
            copies_left = 1 << 30;
            if (rc) {
                REQUIRE(!mem && !held && !bytes);
                continue;
            }
            REQUIRE(mem && held == 1 && bytes >= (int64_t)sum);
            for (size_t k = 0; k < sizes.size(); ++k) {
                REQUIRE(off[k] % 256 == 0 && off[k] + sizes[k] <= (size_t)bytes);
                REQUIRE(!std::memcmp((char*)mem + off[k], data[k].data(), sizes[k]));
            }
            if (sizes.empty() || off[sizes.size() - 1] + sizes.back() <= lim) REQUIRE(copies <= 1);
            hipFree(mem);
            break;
        }
    }
    REQUIRE(held == 0);
    return 0;
}
""")


def test_arrays_share_few_allocations(tmp_path):
    """Arrays of a space in few allocations: each in one of them, aligned and clear of
    the others; small ones in blocks that stay within the size that the runtime keeps at
    hand, the larger ones in one; where an allocation fails, those made are listed.  Sizes
    around that limit, none large, none small, empty arrays, no arrays."""
    _run(tmp_path, r"""
int main() {
    const size_t lim = 2000u << 10;
    const std::vector<std::vector<size_t>> cases = {
        {}, {0}, {1, 255, 256, 257}, {lim, 1, lim - 256, 256, 1}, {lim + 1}, {5, 3 * lim, lim - 255, lim + 256, 7},
        {lim / 2, lim / 2 - 256, 256, 256, lim / 2}, {4 * lim, 0, 0, 9}};
    for (const auto& sizes : cases) {
        size_t used = 0;
        for (int fail = 0;; ++fail) {                  // the allocations that succeed first
            std::vector<void*> at(sizes.size(), nullptr), mem;
            array_list arrays;
            for (size_t k = 0; k < sizes.size(); ++k) arrays.push_back({&at[k], sizes[k]});
            int64_t bytes = 0;
            allocs_left = fail;
            const int rc = alloc_arrays(nullptr, arrays, mem, &bytes);
            allocs_left = 1 << 30;
            REQUIRE((int)mem.size() == held);
            if (rc == SQD_OK) {
                int nlarge = 0, from_block = 0;
                for (size_t k = 0; k < sizes.size(); ++k) {
                    const size_t pad = (sizes[k] + 255) / 256 * 256;
                    nlarge += pad > lim;
                    int owner = -1;
                    for (size_t m = 0; m < mem.size(); ++m)
                        if ((char*)at[k] >= (char*)mem[m] && (owner < 0 || mem[m] > mem[owner])) owner = (int)m;
                    REQUIRE(owner >= 0 && ((char*)at[k] - (char*)mem[owner]) % 256 == 0);
                    if (pad <= lim) {
                        REQUIRE((char*)at[k] + pad <= (char*)mem[owner] + lim);
                        from_block += (char*)at[k] == (char*)mem[owner];
                    }
                    std::memset(at[k], (int)k + 1, sizes[k]);
                }
                for (size_t k = 0; k < sizes.size(); ++k)
                    for (size_t i = 0; i < sizes[k]; ++i) REQUIRE(((unsigned char*)at[k])[i] == k + 1);
                REQUIRE((int)mem.size() <= from_block + (nlarge > 0) && bytes % 256 == 0);
                used = mem.size();
            }
            for (void* p : mem) hipFree(p);
            REQUIRE(held == 0);
            if (rc == SQD_OK) {
                REQUIRE((size_t)fail == used);
                break;
            }
        }
    }
    return 0;
}
""")


def test_tables_of_a_spin_are_allocated_once(tmp_path):
    """The tables of a spin, small and large in all: every array set and clear of the
    others, the larger ones of small tables each at the start of an allocation, and after
    a failed allocation those made are listed.  Totals around the limit between the two."""
    _run(tmp_path, r"""
int main() {
    const size_t lim = 2000u << 10, all = (size_t)18 << 20;
    const std::vector<std::vector<size_t>> cases = {
        {}, {100, lim, lim + 1, lim + 2, 7}, {3 * lim, 5, all - 3 * lim - 5}, {3 * lim, 6, all - 3 * lim - 5}, {lim, 4096}};
    for (const auto& sizes : cases) {
        size_t total = 0;
        for (size_t b : sizes) total += b;
        for (int fail = 0;; ++fail) {
            std::vector<void*> at(sizes.size(), nullptr), mem;
            array_list arrays;
            for (size_t k = 0; k < sizes.size(); ++k) arrays.push_back({&at[k], sizes[k]});
            int64_t bytes = 0;
            allocs_left = fail;
            const int rc = alloc_tables(nullptr, arrays, mem, &bytes);
            allocs_left = 1 << 30;
            REQUIRE((int)mem.size() == held);
            if (rc == SQD_OK) {
                size_t starts = 0;
                for (size_t k = 0; k < sizes.size(); ++k) {
                    const bool first = std::find(mem.begin(), mem.end(), at[k]) != mem.end();
                    starts += first;
                    REQUIRE(at[k] && (first || sizes[k] <= lim || total > all));
                    std::memset(at[k], (int)k + 1, sizes[k]);
                }
                REQUIRE(mem.size() == starts);
                for (size_t k = 0; k < sizes.size(); ++k)
                    for (size_t i = 0; i < sizes[k]; ++i) REQUIRE(((unsigned char*)at[k])[i] == k + 1);
            }
            for (void* p : mem) hipFree(p);
            REQUIRE(held == 0);
            if (rc == SQD_OK) break;
        }
    }
    return 0;
}
""")


@pytest.mark.parametrize("norb", [12, 70])
def test_blocks_hold_every_single_once(tmp_path, norb):
    """Blocks of the alpha-beta term: the singles of a block share their pair and, side
    by side in blocks of two pairs, their source; blocks of two pairs come first; every
    single is in one block; padding only fills the last block of a pair.  Strings of one
    and two words, sets from one string to most of all, around the 64 bits of a word."""
    _run(tmp_path, r"""
#include <map>
#include <random>
typedef unsigned __int128 str;
int main() {
    const int norb = NORB, nel = norb > 64 ? 3 : 6;
    std::mt19937_64 rng(5);
    for (int n : {1, 3, 63, 64, 65, 129, 500}) {
        std::map<str, int> at;
        while ((int)at.size() < n) {      // most from the lowest orbitals: dense in singles
            str s = 0;
            for (int left = nel; left;) {
                const int k = (int)(rng() % (rng() % 4 ? nel + 5 : norb));
                const int o = norb > 64 && rng() % 2 ? norb - 1 - k : k;
                if (!(s >> o & 1)) s |= (str)1 << o, --left;
            }
            at[s] = 0;
        }
        int idx = 0;
        for (auto& x : at) x.second = idx++;
        std::vector<uint32_t> pk;
        for (const auto& t : at) {
            std::map<int, uint32_t> row;
            for (int a = 0; a < norb; ++a)
                for (int i = 0; i < norb; ++i) {
                    if (!(t.first >> a & 1) || (t.first >> i & 1)) continue;
                    const auto s = at.find(t.first ^ ((str)1 << a) ^ ((str)1 << i));
                    if (s == at.end()) continue;
                    row[s->second] = (uint32_t)s->second | (uint32_t)(a * norb + i) << SQD_PAIR_SHIFT | (uint32_t)(rng() % 2) << 31;
                }
            for (const auto& e : row) pk.push_back(e.second);
        }
        for (int G : {2, 4}) {
            const ab_block_plan p = plan_ab_blocks(pk, n, norb, G);
            REQUIRE(p.size == (size_t)p.n2 * 2 * G + (p.pairs.size() - p.n2) * G);
            std::vector<int> seen(pk.size(), 0);
            for (size_t k = 0; k < p.pairs.size(); ++k) {
                const bool two = k < (size_t)p.n2;
                const int2* g = p.grp.get() + (k + (two ? k : (size_t)p.n2)) * G;
                REQUIRE((p.pairs[k].y >= 0) == two);
                for (int r = 0; r < (two ? 2 * G : G); ++r) {
                    if (g[r].x < 0) {
                        REQUIRE(!two && r > 0 && (k + 1 == p.pairs.size() || p.pairs[k + 1].x != p.pairs[k].x));
                        continue;
                    }
                    const uint32_t x = pk[g[r].x];
                    REQUIRE((uint32_t)g[r].y == x && !seen[g[r].x]++);
                    REQUIRE((int)((x >> SQD_PAIR_SHIFT) & SQD_PAIR_MASK) == (r < G ? p.pairs[k].x : p.pairs[k].y));
                    if (r >= G) REQUIRE((x & SQD_NBR_MASK) == ((uint32_t)g[r - G].y & SQD_NBR_MASK));
                }
            }
            for (int s : seen) REQUIRE(s == 1);
            if (n == 500) REQUIRE(p.n2 > 0);
        }
    }
    return 0;
}
""".replace("NORB", str(norb)))
