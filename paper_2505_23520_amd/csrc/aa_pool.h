// Block mean of the queries, qbar_i (arXiv 2505.23520 Sec. 3.2; Algorithm 2, avgpool(Q)), from query
// fragments held in registers in the layout of the bf16 tile engines: lane (n, hf) of a wave holds,
// for one query row, the eight 16-byte pieces Q[row][16 ks + 8 hf .. + 8), ks = 0..7.
// The stage-1 engines pool the block they have just attended (its Q fragments are still in
// registers); stripe_select's own pooling kernel loads the same fragments and runs the same code, so
// both produce the same bits: the order of every floating-point addition is fixed here.
#pragma once
#include "aa_common.h"

namespace aa {

typedef __bf16 pool_bf16x8 __attribute__((ext_vector_type(8)));

// The value of the lane whose number differs in one bit, without a trip through LDS (as __shfl_xor takes it): data-parallel
// primitives inside a row of 16 lanes.  With these and row swaps instead of 62 exchanges through LDS, and one barrier instead of three,
// what stage 2 needs of a block takes the step-1 maximum kernel 4450 cycles instead of 8100, stage 1 3800.
template <int CTRL> __device__ __forceinline__ int dpp_mov(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false);
}
template <int CTRL> __device__ __forceinline__ float dpp_mov(float x) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, false));
}
template <int DIST, class T> __device__ __forceinline__ T lane_xor(T x) {
    static_assert(DIST == 1 || DIST == 2 || DIST == 4 || DIST == 8, "inside a row of 16 lanes");
    if constexpr (DIST == 1) return dpp_mov<0xB1>(x);        // quad_perm [1, 0, 3, 2]
    if constexpr (DIST == 2) return dpp_mov<0x4E>(x);        // quad_perm [2, 3, 0, 1]
    if constexpr (DIST == 4) return dpp_mov<0x1B>(dpp_mov<0x141>(x));    // half a row mirrored, then each quad: 7 ^ 3
    if constexpr (DIST == 8) return dpp_mov<0x128>(x);       // row rotated by 8
}
// x combined over the wave by a commutative op, the distances in the order 32, 16, 8, 4, 2, 1 (down to LAST)
template <int LAST, class T, class Op> __device__ __forceinline__ T wave_reduce(T x, Op op) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = op(__builtin_bit_cast(T, (unsigned)r[0]), __builtin_bit_cast(T, (unsigned)r[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = op(__builtin_bit_cast(T, (unsigned)q[0]), __builtin_bit_cast(T, (unsigned)q[1]));
    x = op(x, lane_xor<8>(x));
    x = op(x, lane_xor<4>(x));
    x = op(x, lane_xor<2>(x));
    if constexpr (LAST == 1) x = op(x, lane_xor<1>(x));
    return x;
}

// fp32 path.  Sum over the 32 lanes of a wave's half, and, for eight values per lane, a reduce-scatter of their sums: lane n
// of the half returns that of value n / 4 (n % 4 = 0: the others hold the same).  The order of the additions is fixed here:
// stage 1 and the pooling kernel give the same bits.
__device__ __forceinline__ float half_sum(float x) {
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    x += lane_xor<8>(x);
    x += lane_xor<4>(x);
    x += lane_xor<2>(x);
    return x + lane_xor<1>(x);
}
__device__ __forceinline__ float half_sums8(float (&f)[8], int n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(f[i]), __float_as_uint(f[4 + i]), false, false);
        f[i] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    }
    const bool b8 = n & 8, b4 = n & 4;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = b8 ? f[2 + i] : f[i], send = b8 ? f[i] : f[2 + i];
        f[i] = keep + lane_xor<8>(send);
    }
    const float keep = b4 ? f[1] : f[0], send = b4 ? f[0] : f[1];
    float x = keep + lane_xor<4>(send);
    x += lane_xor<2>(x);
    return x + lane_xor<1>(x);
}

// Column sums over the 32 rows of a wave's half (lanes with the same hf): a reduce-scatter over
// the lane bits 16, 8, 4, 2, 1 -- at every level a lane keeps one half of its values and receives
// its partner's partial sums for that half.  On return lane (n, hf) holds the sums of columns
// 16 (n / 4) + 8 hf + 2 (n % 4) and that + 1.  Rows that do not exist must hold zeros.
__device__ __forceinline__ void pool_wave_columns(const pool_bf16x8 (&qf)[8], int n, float& s0, float& s1) {
    float f[64];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) f[8 * ks + e] = (float)qf[ks][e];
    // level 16: the swap hands a lane the values it keeps in one register and its partner's in the other
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(f[i]), __float_as_uint(f[32 + i]), false, false);
        f[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#define AA_POOL_LEVEL(width, dist)                                   \
    {                                                                \
        const bool upper = (n & (dist)) != 0;                        \
        _Pragma("unroll") for (int i = 0; i < (width); ++i) {        \
            const float keep = upper ? f[(width) + i] : f[i];        \
            const float send = upper ? f[i] : f[(width) + i];        \
            f[i] = keep + lane_xor<(dist)>(send);                    \
        }                                                            \
    }
    AA_POOL_LEVEL(16, 8)
    AA_POOL_LEVEL(8, 4)
    AA_POOL_LEVEL(4, 2)
    AA_POOL_LEVEL(2, 1)
#undef AA_POOL_LEVEL
    s0 = f[0];
    s1 = f[1];
}

// Work-group part: part[tile][column] receives every wave's column sums (tile = the wave's 32-row
// tile inside its query block, 0..3); after a barrier one wave adds
// the four tiles in the order (0 + 1) + (2 + 3), scales by 1 / nrows, splits the mean into bf16 hi +
// lo parts and writes rows `bi` of qp_hi / qp_lo (128 entries each) and the Euclidean norm of the
// lo row.  part points at the block's float[4][128].
__device__ __forceinline__ void pool_block_put(float (*part)[128], int tile, int n, int hf, float s0, float s1) {
    const int c0 = 16 * (n >> 2) + 8 * hf + 2 * (n & 3);
    part[tile][c0] = s0;
    part[tile][c0 + 1] = s1;
}
__device__ __forceinline__ void pool_block_write(float (*part)[128], int lane, int nrows, long long bi,
                                                 void* qp_hi, void* qp_lo, float* qlo_norm) {
    const float inv = 1.f / (float)nrows;
    const float m0 = ((part[0][2 * lane] + part[1][2 * lane]) + (part[2][2 * lane] + part[3][2 * lane])) * inv;
    const float m1 = ((part[0][2 * lane + 1] + part[1][2 * lane + 1]) +
                      (part[2][2 * lane + 1] + part[3][2 * lane + 1])) * inv;
    auto to_bf16 = [](float x) -> unsigned short {          // round to nearest even
        unsigned u = __float_as_uint(x);
        u += 0x7fffu + ((u >> 16) & 1u);
        return (unsigned short)(u >> 16);
    };
    auto from_bf16 = [](unsigned short b) -> float { return __uint_as_float((unsigned)b << 16); };
    const unsigned short h0 = to_bf16(m0), h1 = to_bf16(m1);
    const unsigned short l0 = to_bf16(m0 - from_bf16(h0)), l1 = to_bf16(m1 - from_bf16(h1));
    ((unsigned*)qp_hi)[bi * 64 + lane] = (unsigned)h0 | ((unsigned)h1 << 16);
    ((unsigned*)qp_lo)[bi * 64 + lane] = (unsigned)l0 | ((unsigned)l1 << 16);
    // what hi + lo leave out (below 2^-16 of an entry) is far inside the tolerance of the
    // decision; the norm of lo bounds what leaving out the lo products would change
    float ln = from_bf16(l0) * from_bf16(l0) + from_bf16(l1) * from_bf16(l1);
    ln = wave_reduce<1>(ln, [](float x, float y) { return x + y; });
    if (lane == 0) qlo_norm[bi] = sqrtf(ln);
}

// Largest key norm of a key block (the mask kernel bounds |<lo, k>| by |lo| |k| to decide whether the lo
// products are needed): rows r0 .. r1 - 1 (at most 128) of the head whose row r starts at k + r * stride, two
// threads per row, so that a row's sum takes one exchange.  All 256 threads of the work-group load and put their wave's
// largest square into part[wave]; after a barrier one thread writes the result.
struct KeyNorm {
    typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
    uintx4 x[8];
    __device__ __forceinline__ void load(const unsigned short* k, long long stride, int r0, int r1, int tid) {
        const unsigned short* src = k + (long long)min(r0 + (tid >> 1), r1 - 1) * stride + 8 * (tid & 1);
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = *(const uintx4*)(src + 16 * c);
    }
    __device__ __forceinline__ float wave_max() const {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = __uint_as_float(x[c][e] << 16), hi = __uint_as_float(x[c][e] & 0xffff0000u);
                s0 = fmaf(lo, lo, s0);
                s1 = fmaf(hi, hi, s1);
            }
        float big = s0 + s1;
        big += lane_xor<1>(big);
        return wave_reduce<2>(big, [](float a, float b) { return fmaxf(a, b); });
    }
    static __device__ __forceinline__ float block(const float* part) {
        return sqrtf(fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3])));
    }
};

// Clears the counters that the mask kernels of both types (and count_kernel) add to, and, where they are given, the sums
// that the fused call's fill kernel adds to (the padded lists' total, the caller's statistics); called by every thread of a
// kernel that runs before them.
__device__ __forceinline__ void clear_counters(int* counts, long long groups, int* segcount, int nseg, long long* total,
                                               long long* stats, long long thread, long long nthreads) {
    for (long long e = thread; e < groups * (nseg + 1); e += nthreads) {
        if (e < groups) counts[e] = 0;
        else segcount[e - groups] = 0;
    }
    if (thread < 4) {
        if (total && thread == 0) *total = 0;
        if (stats) stats[thread] = 0;
    }
}

}  // namespace aa
