"""Host test of the byte offsets of K / V rows that the bf16 engines' tile loads use (csrc/aa_rows.h): every lane's
offset, for token strides up to the largest the library accepts (N * stride * 2 < 2^31), against 64-bit arithmetic."""
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


def test_row_offsets_match_64_bit_arithmetic(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2505_23520_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
