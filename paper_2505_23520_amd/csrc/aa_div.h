// Division of numbers below 2^31 by a divisor (1 .. 2^31) that the host knows: a high product, an addition and a shift
// (Granlund and Montgomery, division by invariant integers) where the compiler's general division is some forty dependent
// instructions.  Five of them stood at the head of every work-group, 2100 cycles up to its first load.
// constexpr: the same code on the host, where it can be compared with the division itself.
#pragma once

namespace aa {

struct FastDiv {
    unsigned d, mul, shift;
    constexpr void set(unsigned divisor) {
        d = divisor;
        shift = 0;
        while (shift < 31 && (1u << shift) < divisor) ++shift;
        mul = (unsigned)((((1ull << shift) - divisor) << 32) / divisor) + 1u;
    }
    constexpr unsigned div(unsigned n) const {
        return ((unsigned)((unsigned long long)n * mul >> 32) + n) >> shift;
    }
};

}  // namespace aa
