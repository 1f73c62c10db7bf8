"""Host tests of the index arithmetic that the kernels share with the host.  csrc/aa_rows.h: byte offsets of K / V rows that the
bf16 engines' tile loads use, every lane's, for token strides up to the largest the library accepts (N * stride * 2 < 2^31),
against 64-bit arithmetic; csrc/aa_items.h: the blocks a persistent work-group walks; csrc/aa_lists.h; csrc/aa_div.h."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "aa_rows.h"

typedef unsigned long long u64;

int main() {
    long long checked = 0, bad = 0;
    const int lens[] = {1, 2, 3, 5, 15, 16, 17, 30, 31, 32, 33, 47, 62, 63, 64, 65, 127, 128, 129, 1000, 4097};
    for (int N : lens) {
        const u64 most = ((1ull << 31) - 1) / N / 16 * 16;            // bytes between tokens
        const u64 strides[] = {most, most / 2 / 16 * 16, most / 3 / 16 * 16, 134217600, 68174080, 68157440, 33554432,
                               33554416, 1073741824, 1073741808, 256, 272};
        for (u64 st : strides) {
            if (st > most || st < 256) continue;
            for (int len : {N, (N + 1) / 2, 1}) {                      // a packed batch has shorter sequences
                for (int start = 0; start < len; start += 64)
                    for (int row = 0; row < 64; ++row)
                        for (int piece = 0; piece < 16; ++piece) {
                            const u64 want = (u64)std::min(start + row, len - 1) * st + 16 * piece;
                            const unsigned last = (unsigned)((len - 1) * st + 16 * piece);
                            // 256-row engine: the lane part holds the row; 128-row engine: rows 0..3 in the tile part
                            const unsigned a = aa::clamped_row_offset(aa::lane_row_offset(row, len, (unsigned)st, piece),
                                                                      aa::tile_row_offset(start, 0, (unsigned)st), last);
                            const unsigned b = aa::clamped_row_offset(aa::lane_row_offset(row & ~3, len, (unsigned)st, piece),
                                                                      aa::tile_row_offset(start, row & 3, (unsigned)st), last);
                            ++checked;
                            if (a != want || b != want) {
                                if (!bad++) printf("N %d len %d stride %llu start %d row %d: %u %u, not %llu\n", N, len, st,
                                                   start, row, a, b, want);
                            }
                        }
            }
        }
    }
    printf("%lld checked, %lld wrong\n", checked, bad);
    return bad || checked < 100000;
}
"""


DIVISIONS = r"""
#include <cstdio>
#include <initializer_list>
#include "aa_div.h"

int main() {
    long long bad = 0;
    unsigned long long x = 88172645463325252ull;
    for (unsigned k = 0; k < 4000; ++k) {
        x ^= x << 13; x ^= x >> 7; x ^= x << 17;
        // small divisors, powers of two and their neighbours, and any up to 2^31
        const unsigned d = k < 1500 ? k + 1 : k < 1593 ? (1u << ((k - 1500) / 3)) - 1 + (k - 1500) % 3 : (unsigned)(x >> 33) + 1;
        if (!d || d > (1u << 31)) continue;
        aa::FastDiv f{};
        f.set(d);
        for (unsigned e = 0; e < 400; ++e) {
            x ^= x << 13; x ^= x >> 7; x ^= x << 17;
            const unsigned q = (unsigned)(x >> 33) / d;
            const unsigned ns[] = {(unsigned)(x >> 33), e, 0x7fffffffu - e, q * d, q * d + d - 1, q * d - 1};
            for (unsigned n : ns)
                if (n < (1u << 31) && f.div(n) != n / d && !bad++) printf("%u / %u: %u\n", n, d, f.div(n));
        }
    }
    for (unsigned long long d : {1ull << 31, (1ull << 31) + 1, 1ull << 32, (1ull << 32) + 5, 65536ull * 65534, 1ull << 44}) {
        aa::FastDiv f{};
        f.set(d);
        for (unsigned n : {0u, 1u, 12345u, 0x7ffffffeu, 0x7fffffffu})
            if (f.div(n) != 0 && !bad++) printf("%u / %llu: %u\n", n, d, f.div(n));
    }
    return bad != 0;
}
"""


PLACES = r"""
#include <cstdio>
#include <initializer_list>
#include "aa_lists.h"

int main() {
    long long bad = 0;
    for (long long span : {64, 128, 192, 256, 512, 1152, 2048, 16384})
        for (long long n_init : {0, 1, 16, 63, 64, 100, 128, 1000, 5000})
            for (long long window : {0, 1, 30, 64, 65, 128, 300, 2047, 2048, 40000}) {
                long long sum = 0;
                for (long long n = 0; n < 300; ++n) {
                    if (aa::padded_places(n, span, n_init + window) != sum && !bad++)
                        printf("span %lld n_init %lld window %lld n %lld\n", span, n_init, window, n);
                    const long long W = n * span - window > n_init ? n * span - window : n_init;
                    sum += (W - n_init + 63) / 64 * 64;
                }
            }
    return bad != 0;
}
"""


ITEMS = r"""
#include <cstdio>
#include <vector>
#include "aa_items.h"

// packed batches of query blocks, numbered as if every sequence were as long as the longest
struct Block { int seq, i, len; };

int main() {
    long long bad = 0, walked = 0;
    const std::vector<std::vector<int>> batches = {{5}, {1, 0}, {0, 3}, {7, 26, 0}, {0, 0, 4, 0, 0}, {8, 0, 27, 2}, {0, 1, 0, 1}};
    for (const auto& blocks : batches)                   // blocks of every sequence
        for (int heads : {1, 3, 8})
            for (unsigned stride : {1u, 3u, 8u, 64u, 768u}) {
                int most = 0, all = 0;
                for (int n : blocks) { most = n > most ? n : most; all += n * heads; }
                const unsigned total = (unsigned)(most * heads * (int)blocks.size());
                auto block_of = [&](unsigned id) {
                    const int seq = (int)(id / (unsigned)(most * heads));
                    return Block{seq, most - 1 - (int)(id % (unsigned)(most * heads)) / heads, blocks[seq]};
                };
                auto exists = [](const Block& x) { return x.i < x.len; };
                std::vector<int> seen(total, 0);
                for (unsigned wg = 0; wg < stride; ++wg) {       // as a work-group walks: requests ahead, then takes
                    unsigned id = wg;
                    Block cur{0, 0, 0};
                    if (!aa::next_item(id, stride, total, cur, block_of, exists)) continue;
                    for (;;) {
                        ++seen[id];
                        id += stride;
                        Block nx = cur;
                        const bool more = aa::next_item(id, stride, total, nx, block_of, exists);
                        if (!exists(nx)) ++bad;                  // its rows are loaded
                        if (more != (id < total)) ++bad;
                        if (!more) break;
                        cur = nx;
                    }
                }
                for (unsigned id = 0; id < total; ++id) {
                    if (seen[id] != (exists(block_of(id)) ? 1 : 0)) ++bad;
                    walked += seen[id];
                }
                for (unsigned id = 0; id < total; ++id) all -= seen[id];
                if (all) ++bad;
            }
    printf("%lld walked, %lld wrong\n", walked, bad);
    return bad != 0 || walked < 1000;
}
"""


def test_walk_over_blocks_requests_only_blocks_that_exist(tmp_path):
    src, exe = tmp_path / "items.cpp", tmp_path / "items"
    src.write_text(ITEMS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2505_23520_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_places_of_the_lists(tmp_path):
    src, exe = tmp_path / "places.cpp", tmp_path / "places"
    src.write_text(PLACES)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2505_23520_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_divisions_by_known_divisors(tmp_path):
    src, exe = tmp_path / "div.cpp", tmp_path / "div"
    src.write_text(DIVISIONS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2505_23520_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_row_offsets_match_64_bit_arithmetic(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2505_23520_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
