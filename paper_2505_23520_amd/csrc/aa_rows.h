// Byte offsets of K / V rows of contiguous tiles (bf16 engines).  A tile's last keys may lie past the end of the
// sequence: their loads are sent to the last row.  The clamp works on 32-bit byte offsets (one addition and one minimum per
// load; clamping the key first takes a quarter-rate multiplication as well), and an offset before the clamp does not
// fit 32 bits where few tokens lie far apart (N * stride < 2^31 bytes leaves (N + 63) * stride open), so everything up to
// the clamp saturates.  constexpr: the same code on the host, where it can be compared with 64-bit arithmetic.
#pragma once

namespace aa {

// offset of 16-byte piece `piece` of row `row` (below 64) from the tile's first row
constexpr unsigned lane_row_offset(int row, unsigned stride, int piece) {
    const unsigned long long x = (unsigned long long)row * stride + 16ull * piece;
    return x > 0xffffffffull ? 0xffffffffu : (unsigned)x;
}

// scalar part: row `j` (0..3) after key `start`, the tile's first, in a sequence of `len` rows.  With more than one tile,
// stride < 2^25; else start = 0, and a stride above 2^30 has one row only, which every other offset exceeds already.
constexpr unsigned tile_row_offset(int start, int len, unsigned j, unsigned stride) {
    return (unsigned)(start < len ? start : len - 1) * stride + j * (stride < (1u << 30) ? stride : 1u << 30);
}

// their sum, at most `last` (the lane's piece of the sequence's last row)
constexpr unsigned clamped_row_offset(unsigned lane_part, unsigned tile_part, unsigned last) {
    const unsigned x = lane_part + tile_part;
    const unsigned sum = x < lane_part ? 0xffffffffu : x;
    return sum < last ? sum : last;
}

}  // namespace aa
