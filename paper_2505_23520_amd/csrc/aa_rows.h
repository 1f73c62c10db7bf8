// Byte offsets of K / V rows of contiguous tiles (bf16 engines).  A tile's last keys may lie past the end of the
// sequence: their loads are sent to the last row.  The clamp works on 32-bit byte offsets (one addition and one minimum per
// load; clamping the key first takes a quarter-rate multiplication as well), and an offset before the clamp does not
// fit 32 bits where few tokens lie far apart (N * stride < 2^31 bytes leaves (N + 63) * stride open): its parts are kept
// below 2^32 and their sum saturates.  constexpr: the same code on the host, where it can be compared with 64-bit arithmetic.
#pragma once

namespace aa {

// piece `piece` (16 bytes) of row `row` after the tile's first key; a row that lies past the end whatever the tile's
// first key is counts as row `len`, which keeps the product below 2^31
constexpr unsigned lane_row_offset(int row, int len, unsigned stride, int piece) {
    return (unsigned)(row < len ? row : len) * stride + 16u * (unsigned)piece;
}

// scalar part: row `j` (0..3) after key `start` (below `len`), the tile's first.  With more than one tile stride < 2^25;
// else start = 0, and a stride above 2^30 has one row only, which every other offset exceeds already.
constexpr unsigned tile_row_offset(int start, unsigned j, unsigned stride) {
    return (unsigned)start * stride + j * (stride < (1u << 30) ? stride : 1u << 30);
}

// their sum, at most `last` (the lane's piece of the sequence's last row)
constexpr unsigned clamped_row_offset(unsigned lane_part, unsigned tile_part, unsigned last) {
    const unsigned x = lane_part + tile_part;
    const unsigned sum = x < lane_part ? 0xffffffffu : x;
    return sum < last ? sum : last;
}

}  // namespace aa
