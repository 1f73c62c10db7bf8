// Where the fused call puts the lists of selected columns: every group at a place of its own, as long as its candidates, so that
// no scan over the counts stands between the mask and the lists.  constexpr: the same code on the host.
#pragma once

namespace aa {

constexpr int kIdxPad = 64;        // list chunks are 64 entries (one K/V tile)

// Entries of the candidates of a sequence's first n groups, each group's rounded up to a list chunk: group g has
// g span - c candidates, c = n_init + window, where that is positive.  span: rows of a group, a multiple of kIdxPad.
constexpr long long padded_places(long long n, long long span, long long c) {
    const long long g0 = c / span + 1;               // first group with candidates
    if (n <= g0) return 0;
    return span * ((g0 + n - 1) * (n - g0) / 2) - (n - g0) * (c / kIdxPad * kIdxPad);
}

}  // namespace aa
