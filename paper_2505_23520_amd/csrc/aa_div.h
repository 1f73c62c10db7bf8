// Division of numbers below 2^31 by a positive divisor that the host knows: a high product, an addition and a shift
// (Granlund and Montgomery, division by invariant integers) where the compiler's general division is some forty dependent
// instructions.  Five of them stood at the head of every work-group, 2100 cycles up to its first load.
// constexpr: the same code on the host, where it can be compared with the division itself.
#pragma once

namespace aa {

struct FastDiv {
    unsigned d, mul, shift;
    constexpr void set(unsigned long long divisor) {     // above 2^31 every quotient is 0, as with 2^31
        d = divisor < (1ull << 31) ? (unsigned)divisor : 1u << 31;
        shift = 0;
        while (shift < 31 && (1u << shift) < d) ++shift;
        mul = (unsigned)((((1ull << shift) - d) << 32) / d) + 1u;
    }
    constexpr unsigned div(unsigned n) const {
        return ((unsigned)((unsigned long long)n * mul >> 32) + n) >> shift;
    }
};

}  // namespace aa
