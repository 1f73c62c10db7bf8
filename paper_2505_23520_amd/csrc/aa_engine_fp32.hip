// fp32 tile engine: the same online-softmax walk as the bf16 engines (stage 1
// anchor computation, Algorithm 1; stage 3 gathered sparse attention, Algorithm 3;
// dense causal comparator -- arXiv 2505.23520) with fp32 inputs, fp32 products and
// fp32 probabilities, on the bf16 matrix instruction.
//
// Products: an fp32 value is the exact sum of three bf16 parts (h, m, l: 3 x 8 bits; 0 and magnitudes from 2^-110 to 3.39e38,
// what lies outside is looked for after the loop and falls back to the fp32 instruction), and a product of two values
// is six products of parts, hh + hm + mh + mm + hl + lh; the other three are below 2^-24 of it.  Six instructions of
// 32 matrix cycles for 16 columns take 192 cycles where v_mfma_f32_32x32x2_f32 takes 512.  Scores: the hh products have an
// accumulator of their own, which sees 8 roundings at d = 128 (64 with the fp32 instruction); relative error of the output
// against 64 bits, 4000 tokens, d = 128: 8.8e-7 with the fp32 instruction, 5.9e-7 so, and smaller by a third on every size tried.
//
// Fragments (the layout of the bf16 engines): lane (n, hf) = (lane % 32, lane / 32).  S^T = K Q^T: keys = M, query
// rows = N; lane (n, hf) holds columns 16 j + 8 hf .. + 8 of row n.  Score register v of lane (n, hf) belongs to query
// row n and key 8 (v / 4) + 4 hf + v % 4 -- which is exactly the B operand of O^T = V^T P^T if those are the keys of
// the k slots: the probabilities never move between lanes.
// V^T rows are columns of V in any order: row c of column block db is column T c + db (T = d / 32),
// so a lane's T columns are one wide load and a wave reads two whole V rows at once.
//
// Shape: work-group = one tile of 32 query rows = 4 waves that share the rows and split the 32-key
// blocks among them (block b belongs to wave b % 4); each keeps its own (m, l, O) and they are merged
// once, through LDS, at the end.  The loop has no barrier: K goes to LDS of the wave's own, a block ahead, V straight to
// registers.  32 rows per work-group keep the chip filled at small sizes, and splitting the keys
// shortens the chain of a short sequence.
// Bound: the split is 11 vector instructions for two values and nothing shares it between work-groups, 700 of the 1000
// vector instructions of a block at d = 128 (5.5 cycles each for a lone wave); they run beside the 3072 matrix cycles
// (8192 with the fp32 instruction).  On short sequences the chain of one wave's blocks, and 15000 cycles of prologue and merge.
// Measured against the fp32 instruction with K and V straight to registers, kernel times: prefill of 4000 tokens, 8 / 2 heads,
// d = 128: stage 1 112 -> 68 us (the products 112 -> 84, the order of the tiles 84 -> 75, K through LDS 75 -> 68),
// stage 3 29 -> 26; 1024 tokens, 1 head, d = 64: 15.1 -> 11.6 and 8.4 -> 7.5; dense causal, 2313 tokens, 2 heads, d = 64:
// 60 -> 37 us.
#include "aa_common.h"
#include "aa_engine.h"
#include "aa_pool.h"

#include <type_traits>

namespace aa {

namespace {
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr floatx16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
constexpr int KB = 32;   // keys per block
constexpr int RT = 32;   // query rows per work-group
constexpr int NW = 4;    // waves per work-group

// Work-groups per grid row: a launch takes fewer than 2^32 threads in x, and 256 threads per 32 rows (per 16 at a block of
// 16) reach that with 5e8 (2.7e8) rows times heads.  A multiple of 8, so that decode_tile's XCD of a work-group holds.
constexpr unsigned kGridX = 1u << 23;

template <int T> struct vcols;
template <> struct vcols<1> { typedef float type; };
template <> struct vcols<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct vcols<4> { typedef float type __attribute__((ext_vector_type(4))); };
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float comp(float x, int) { return x; }
template <class V> __device__ __forceinline__ float comp(const V& x, int i) { return x[i]; }

// A row's two lanes (n, 0) and (n, 1) combined, without a trip through LDS
template <class Op> __device__ __forceinline__ float both_halves(float x, Op op) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) { return both_halves(x, [](float a, float b) { return a + b; }); }

// Eight fp32 values as three bf16 parts, x = h + m + l exactly (8 + 8 + 8 bits, each rounded to nearest, so the
// subtractions are exact) for 0 and |x| from 2^-110 to 3.39e38; below, l lies among bf16's last subnormals and up to 2^-134 is lost.
struct Split {
    uintx4 h, m, l;
    __device__ __forceinline__ void pair(int i, float x0, float x1) {        // elements 2 i, 2 i + 1
        auto pack = [](float a, float b) {
            return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
        };
        const unsigned ph = pack(x0, x1);
        x0 -= __uint_as_float(ph << 16);
        x1 -= __uint_as_float(ph & 0xffff0000u);
        const unsigned pm = pack(x0, x1);
        x0 -= __uint_as_float(pm << 16);
        x1 -= __uint_as_float(pm & 0xffff0000u);
        h[i] = ph; m[i] = pm; l[i] = pack(x0, x1);
    }
};
__device__ __forceinline__ floatx16 mfma_bf16(const uintx4& a, const uintx4& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Work-group id -> (batch, query head, row tile), the tiles with the longest key ranges first.  Dense attention and lists: the
// later the tile, the longer.  Anchor region alone: the later in its group, the longer, and the groups side by side.
// A wave has the chip's matrix and vector pipes nearly to itself at these sizes, so the last round of work-groups lasts as
// long as its longest tile.  All query heads of a KV head stay on one XCD (its L2) where the heads divide among the XCDs.
struct TileMap {
    unsigned tiles;                                  // of the longest sequence
    FastDiv rts, pair, heads, heads8;                // row tiles of a block; tiles x Hq / Hkv; B x Hq, and an eighth of it
    FastDiv hq;
    // anchor region alone: tiles of a group; the groups, and the groups but the last; tiles at positions in a group that the
    // last group does not have, over all groups
    FastDiv per, groups, groups1;
    unsigned head, rem;
    void set(const KParams& p) {
        const unsigned r = (unsigned)((p.bq + RT - 1) / RT);
        tiles = (unsigned)p.nblk_max * r;
        rts.set(r);
        pair.set((unsigned long long)tiles * p.grp);
        heads.set((unsigned)(p.B * p.Hq));
        heads8.set(heads.d >= 8 ? heads.d / 8 : 1);
        hq.set((unsigned)p.Hq);
        per.set((unsigned)p.step * r);
        groups.set((tiles + per.d - 1) / per.d);
        groups1.set(groups.d > 1 ? groups.d - 1 : 1);
        rem = tiles - (groups.d - 1) * per.d;
        head = (per.d - rem) * (groups.d - 1);
    }
};
__device__ __forceinline__ Work decode_tile(const KParams& p, const TileMap& m, bool anchor_only, unsigned id) {
    unsigned x, hb;
    if ((unsigned)(p.B * p.Hkv) % 8 == 0) {
        const unsigned slot = id >> 3, q = m.pair.div(slot), within = slot - q * m.pair.d;
        x = p.by_grp.div(within);
        hb = ((id & 7) + 8 * q) * p.grp + within - x * p.grp;
    } else if (m.heads.d % 8 == 0) {
        const unsigned slot = id >> 3;
        x = m.heads8.div(slot);
        hb = (id & 7) * m.heads8.d + slot - x * m.heads8.d;
    } else {
        x = m.heads.div(id);
        hb = id - x * m.heads.d;
    }
    Work wk;
    wk.b = (int)m.hq.div(hb);
    wk.h = (int)hb - wk.b * p.Hq;
    wk.i = (int)(m.tiles - 1 - x);
    if (anchor_only) {
        unsigned pos, gr;
        if (x < m.head) {
            const unsigned q = m.groups1.div(x);
            pos = m.per.d - 1 - q;
            gr = x - q * m.groups1.d;
        } else {
            const unsigned q = m.groups.div(x - m.head);
            pos = m.rem - 1 - q;
            gr = x - m.head - q * m.groups.d;
        }
        wk.i = (int)(gr * m.per.d + pos);
    }
    return wk;
}

// FLAGS (a combination of kEng*) as in engine_bf16_kernel
template <int T> __device__ __forceinline__ typename vcols<T>::type buffer_load(__amdgpu_buffer_rsrc_t rs, unsigned off) {
    typedef typename vcols<T>::type vec;
    if constexpr (T == 1) return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
    else if constexpr (T == 2) return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0));
    else return __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }     // vmcnt(0)

// WIDE: a head's rows of K or V span 4 GiB or more (64-bit addresses instead of buffer offsets).  The compiler waits for
// every load in flight wherever it needs one of them then (its rule for loads of the flat encoding that write to LDS).
template <int D, int FLAGS, bool WIDE>
__global__ __launch_bounds__(64 * NW, D == 128 || WIDE ? 2 : 3) void engine_fp32_kernel(EngineArgs a, TileMap map) {
    constexpr int flags = FLAGS;
    constexpr int T = D / 32;                        // column blocks of O
    constexpr int KS = D / 16;                       // 16-column pieces of a K / Q row
    constexpr int VK = 8 / KS;                       // V rows requested per piece of K consumed
    typedef typename vcols<T>::type vec;
    // Slot j holds piece j of every wave's K block (2 KB a wave) and, after the loop, 8 of every wave's O^T registers.  One
    // object per slot, so that the compiler can tell that the asynchronous loads into one do not alias the reads from another.
    __shared__ __attribute__((aligned(16))) floatx4 K0[NW][128], K1[NW][128], K2[NW][128], K3[NW][128], K4[NW][128],
        K5[NW][128], K6[NW][128], K7[NW][128];
    auto slot = [&](int j) -> floatx4(*)[128] {      // (j is a constant everywhere: slots beyond KS - 1 do not exist)
        return j == 0 ? K0 : j == 1 ? K1 : j == 2 ? K2 : j == 3 ? K3 : j == 4 ? K4 : j == 5 ? K5 : j == 6 ? K6 : K7;
    };
    constexpr bool QREG = D == 128;                  // the queries' first parts in registers: two work-groups fill the LDS
    __shared__ union {
        uintx4 q[QREG ? 2 : 3][KS][64];              // the other parts (m, l) of the query rows
        struct { float m[NW][RT], l[NW][RT]; } st;   // after the loop
    } sm;
    const KParams& p = a.p;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 31, hf = lane >> 5;

    if (flags & kEngStoreState) {
        store_dense_stats(a);
        if (flags & kEngParts) {
            const long long wg = blockIdx.x + (long long)gridDim.x * blockIdx.y;
            clear_counters(a.zero_counts, a.groups_total, a.zero_seg, a.nseg, a.zero_total, a.zero_stats,
                           wg * (64 * NW) + threadIdx.x, (long long)gridDim.x * gridDim.y * (64 * NW));
        }
    }
    if ((flags & kEngList) && !engine_selected(a)) return;
    const unsigned id = blockIdx.y * kGridX + blockIdx.x;
    if (id >= map.tiles * map.heads.d) return;
    const Work wk = decode_tile(p, map, !(flags & (kEngDense | kEngList)), id);
    const Seq sq = seq_of(p, wk.b);
    const int blk = (int)map.rts.div(wk.i);
    const int row0 = blk * p.bq + (wk.i - blk * (int)map.rts.d) * RT;        // first row of the tile
    const int rend = min(min(blk * p.bq + p.bq, row0 + RT), sq.len);
    if (row0 >= rend) return;
    const int hk = (int)p.by_grp.div(wk.h);
    const int g = (int)p.by_step.div(blk);
    const bool direct = a.direct && window_start(p, g) <= p.n_init;   // no candidates: stage 1 finishes the rows
    if ((flags & kEngLoadState) && direct) return;
    const int r = row0 + n;
    const bool rok = r < rend;
    const int rlast = rend - 1;

    // ---- block sequence: [initial tokens][window .. diagonal][list]
    int W = 0, ninit = 0, T1 = 0, t2s = 0, nA = 0;
    if (flags & kEngAnchorRegion) {
        if (!(flags & kEngDense)) { W = window_start(p, g); ninit = p.n_init; }
        const int e1 = min(ninit, rlast + 1);
        T1 = (e1 + KB - 1) / KB;
        t2s = max(T1, W / KB);
        nA = T1 + max(0, rlast / KB + 1 - t2s);
    }
    int cnt = 0;
    long long lbase = 0;
    if (flags & kEngList) {
        const long long t = grp_index(p, sq, wk.b, wk.h, g);
        cnt = a.counts[t];
        lbase = a.offsets[t];
    }
    const int nT = nA + (cnt + KB - 1) / KB;
    auto block_start = [&](int t) -> int { return KB * (t < T1 ? t : t2s + (t - T1)); };
    // key of this lane's K row in block t (lists are padded to 64 entries, so every slot read exists)
    auto key_of = [&](int t) -> int {
        if (t >= nT) return 0;
        return t < nA ? min(block_start(t) + n, sq.len - 1) : a.idx[lbase + (long long)(t - nA) * KB + n];
    };

    const float* kb_ = (const float*)a.k + tok_offset(p, p.ks, sq, wk.b, hk, 0);
    const float* vb_ = (const float*)a.v + tok_offset(p, p.vs, sq, wk.b, hk, 0);
    const float* qsrc = (const float*)a.q + tok_offset(p, p.qs, sq, wk.b, wk.h, rok ? r : row0) + 8 * hf;

    int key = key_of(wave), key_next = key_of(wave + NW);
    // K: piece j of a block (16 columns of its 32 keys) is two direct-to-LDS loads, in each of which four lanes fetch 64
    // bytes of a row together: lane 4 i + s the 16 bytes s ^ (i / 2 % 4) of row i, or 16 + i.  (Every lane fetching its own row's
    // bytes into registers is 64 accesses to the L1 an instruction instead of 16.)  The fragments, lane (n, hf) columns
    // 8 hf .. + 8 of key n, are read from the slot that only this wave uses; the exchange of the 16-byte places spreads
    // the reads of eight consecutive rows over the banks.
    floatx4 frag[2][2];
    vec vf[16];
    const unsigned kstb = (unsigned)p.ks[2] * 4u, vstb = (unsigned)p.vs[2] * 4u;   // token strides in bytes (not WIDE)
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)kb_, 0, (int)((unsigned)(sq.len - 1) * kstb + 4u * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)vb_, 0, (int)((unsigned)(sq.len - 1) * vstb + 4u * D), 0x00020000);
    const float *krow0 = nullptr, *krow1 = nullptr;  // of the block whose pieces are being requested (WIDE)
    unsigned koff0 = 0, koff1 = 0;
    auto k_rows = [&](int kk) {
        int src = lane & ~3;                         // byte address of lane (lane / 4)
        asm volatile("" : "+v"(src));
        const int k0 = __builtin_amdgcn_ds_bpermute(src, kk), k1 = __builtin_amdgcn_ds_bpermute(src + 64, kk);
        const int c = 4 * ((lane & 3) ^ (lane >> 3 & 3));
        if (WIDE) {
            krow0 = kb_ + (long long)k0 * p.ks[2] + c;
            krow1 = kb_ + (long long)k1 * p.ks[2] + c;
        } else {
            koff0 = (unsigned)k0 * kstb + 4u * c;
            koff1 = (unsigned)k1 * kstb + 4u * c;
        }
    };
    auto load_k = [&](int j) {                       // asynchronous
        lds_void *d0 = (lds_void*)&slot(j)[wave][0], *d1 = (lds_void*)&slot(j)[wave][64];
        if (WIDE) {
            __builtin_amdgcn_global_load_lds((const global_void*)(krow0 + 16 * j), d0, 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const global_void*)(krow1 + 16 * j), d1, 16, 0, 0);
        } else {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, d0, 16, (int)koff0, 64 * j, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, d1, 16, (int)koff1, 64 * j, 0, 0);
        }
    };
    const int kr0 = 4 * n + (2 * hf ^ (n >> 1 & 3)), kr1 = 4 * n + ((2 * hf + 1) ^ (n >> 1 & 3));
    auto read_k = [&](int j) {
        frag[j & 1][0] = slot(j)[wave][kr0];
        frag[j & 1][1] = slot(j)[wave][kr1];
    };
    // The lane's row of V, as a byte offset; it goes to the lanes that read it (a product per row and lane instead would be
    // 64 bits wide in the WIDE form).  A lane's T columns are one load, a wave reads two whole rows with each.
    int vlo = 0, vhi = 0;
    auto v_rows = [&](int kk) {
        if (WIDE) {
            const long long off = (long long)kk * p.vs[2] * 4;
            vlo = (int)off; vhi = (int)(off >> 32);
        } else {
            vlo = (int)((unsigned)kk * vstb);
        }
    };
    // rows of loads v .. v + N - 1: every exchange is issued before the first result is waited for
    // src: byte address of lane 4 hf, made opaque for every block: 16 sums are not kept in registers
    auto v_lane = [&]() -> int {
        int src = 16 * hf;
        asm volatile("" : "+v"(src));
        return src;
    };
    auto load_v = [&](int src, int v, auto count) {
        constexpr int N = decltype(count)::value;
        unsigned lo[N], hi[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int from = src + 4 * (8 * ((v + i) >> 2) + ((v + i) & 3));
            lo[i] = (unsigned)__builtin_amdgcn_ds_bpermute(from, vlo);
            if (WIDE) hi[i] = (unsigned)__builtin_amdgcn_ds_bpermute(from, vhi);
        }
        return [=, &vf](int i) {                     // the load itself
            if (WIDE) vf[v + i] = *(const vec*)((const char*)(vb_ + T * n) + (long long)((unsigned long long)hi[i] << 32 | lo[i]));
            else vf[v + i] = buffer_load<T>(vrs, lo[i] + 4u * T * n);
        };
    };
    k_rows(key);
#pragma unroll
    for (int j = 0; j < KS; ++j) load_k(j);
    auto part_index = [&]() -> long long { return blk_index(p, sq, wk.b, wk.h, blk) * map.rts.d + (row0 - blk * p.bq) / RT; };
    // the waves share the rows: each splits its part of them
    uintx4 qreg[QREG ? KS : 1];
    Split own[(KS + NW - 1) / NW];
#pragma unroll
    for (int i = 0; i < (KS + NW - 1) / NW; ++i) {
        const int j = i * NW + wave;
        if (j >= KS) break;
        const floatx4 x = *(const floatx4*)(qsrc + 16 * j), y = *(const floatx4*)(qsrc + 16 * j + 4);
        if ((flags & kEngParts) && !direct) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = rok ? (e < 4 ? x[e & 3] : y[e & 3]) : 0.f;
            const float sum = half_sums8(f, n);
            if (n % 4 == 0) ((float*)a.qp_hi)[part_index() * D + 16 * j + 8 * hf + n / 4] = sum;
        }
        own[i].pair(0, x[0], x[1]); own[i].pair(1, x[2], x[3]); own[i].pair(2, y[0], y[1]); own[i].pair(3, y[2], y[3]);
        // Queries outside [2^-100, 2^40] but for 0: a part that is not a number makes the row's results so (see below the loop)
        float big = 0.f;
        unsigned small = ~0u;                        // twice the smallest magnitude but 0, less 1
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float c = e < 4 ? x[e & 3] : y[e & 3];
            big = __builtin_elementwise_maximum(big, fabsf(c));
            small = min(small, (__float_as_uint(c) << 1) - 1u);
        }
        if (small < (__float_as_uint(0x1p-100f) << 1) - 1u || !(big <= 0x1p40f)) own[i].l[0] = 0x7fc07fc0u;
        sm.q[0][j][lane] = own[i].h;
        sm.q[1][j][lane] = own[i].l;
        if (!QREG) sm.q[QREG ? 0 : 2][j][lane] = own[i].m;
    }
    if (QREG) {                                      // the first parts go on to every wave's registers, the second in their place
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KS; ++j) qreg[QREG ? j : 0] = sm.q[0][j][lane];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < (KS + NW - 1) / NW; ++i) sm.q[0][i * NW + wave][lane] = own[i].m;
    }

    const float c2 = p.sigma * 1.4426950408889634f;  // exp(sigma*x) = exp2(c2*x)
    float m = -INFINITY, l = 0.f;                    // l: this lane's keys only
    float smin = INFINITY;                           // of the lane's scores, hidden keys' too (loop only)
    floatx16 o[T];
    auto reset = [&]() {
        m = -INFINITY; l = 0.f;
#pragma unroll
        for (int db = 0; db < T; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    };
    reset();
    // The sum of a block's scores is made before the branches of its masks.  Left alone, the compiler moves it behind them and then
    // counts the wait states between the last matrix instruction and the first addition along the longer arm only: on
    // the other, 12 instead of 18 in the fp32 form below, where a row's keys 27 and 31 had the score of earlier instructions, and 9
    // instead of 12 in the loop.
    auto keep_here = [](floatx16& s) __attribute__((always_inline)) { asm volatile("" : "+v"(s)); };
    // Scores of block t -> probabilities; updates m and l, rescales o.  parts: of the loop, whose wave takes its blocks again if a
    // score is not a number, so it may get lost here or not; fmaxf, which passes it over, costs an instruction
    // more for every operand of unknown origin.
    auto softmax = [&](auto parts, int t, floatx16& s) {
        if (decltype(parts)::value) {
#pragma unroll
            for (int v = 0; v < 16; ++v) smin = __builtin_elementwise_minimum(smin, s[v]);
        }
        if (t < nA) {
            // key j is visible to row r iff j <= r and (j < ninit or j >= W); the lane's part of j,
            // 4 hf, is taken off the limits instead
            const int t0 = block_start(t);
            if (t0 + KB - 1 > row0 || !(t0 + KB <= ninit || t0 >= W)) {
                int jr = r - t0 - 4 * hf;
                asm volatile("" : "+v"(jr));         // opaque: nothing is hoisted out of the loop
                const int jn = ninit - t0 - 4 * hf, jw = W - t0 - 4 * hf;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int jc = 8 * (v >> 2) + (v & 3);
                    if (!(jc <= jr && (jc < jn || jc >= jw))) s[v] = -INFINITY;
                }
            }
        } else {
            int jr = cnt - (t - nA) * KB - 1 - 4 * hf;
            asm volatile("" : "+v"(jr));
            if ((t + 1 - nA) * KB > cnt) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + (v & 3) > jr) s[v] = -INFINITY;
            }
        }
        const auto larger = [](float a, float b) {
            return decltype(parts)::value ? __builtin_elementwise_maximum(a, b) : fmaxf(a, b);
        };
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = larger(mx, s[v]);
        mx = both_halves(mx, larger);
        if (__any(mx > m)) {
            const float mnew = fmaxf(m, mx);
            const float alpha = (mnew == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((m - mnew) * c2);
            m = mnew;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < T; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
        }
        const float mc = (m == -INFINITY) ? 0.f : m * c2;
        float rs = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], c2, -mc));
            rs += s[v];
        }
        l += rs;
    };

    // K pieces are requested a block ahead, into the slot whose contents have just been split, V rows half during the scores of
    // their block, half before its softmax.  The split of a piece is spread between the products of the one before; the order is pinned with
    // scheduling fences.
    Split sp[2];
    auto split_k = [&](Split& d, int j, int i) {     // elements 2 i, 2 i + 1 of piece j
        const floatx4& x = frag[j & 1][i >> 1];
        d.pair(i, x[2 * (i & 1)], x[2 * (i & 1) + 1]);
    };
    auto split_v = [&](Split& d, int u, int i) {     // piece u: 16-key half u / T, column block u % T
        const int v = 8 * (u / T) + 2 * i;
        d.pair(i, comp(vf[v], u % T), comp(vf[v + 1], u % T));
    };
    __syncthreads();                                 // the query parts are there
    read_k(0);
    read_k(1);
#pragma unroll
    for (int i = 0; i < 4; ++i) split_k(sp[0], 0, i);
#pragma unroll 1
    for (int t = wave; t < nT; t += NW) {
        // Two accumulation chains.  Of the nine products of the parts the three below 2^-24 of the largest are left out.
        floatx16 s2[2] = {kZero16, kZero16};
        v_rows(key);
        const int src = v_lane();
        key = key_next;
        key_next = key_of(t + 2 * NW);
        k_rows(key);
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            const Split& k = sp[j & 1];
            Split& nx = sp[(j + 1) & 1];
            const uintx4 qh = QREG ? qreg[QREG ? j : 0] : sm.q[0][j][lane];
            const uintx4 qm = sm.q[QREG ? 0 : 2][j][lane], ql = sm.q[1][j][lane];
            const auto next_v = load_v(src, j * VK, std::integral_constant<int, VK>());
            const bool more = j + 1 < KS;
            __builtin_amdgcn_sched_barrier(0);
            load_k(j);                               // of the next block: piece j of this one has been split
            if (j + 2 < KS) read_k(j + 2);
            __builtin_amdgcn_sched_barrier(0);
            s2[1] = mfma_bf16(k.l, qh, s2[1]);
            if (more) split_k(nx, j + 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            s2[1] = mfma_bf16(k.h, ql, s2[1]);
            if (more) split_k(nx, j + 1, 1);
            __builtin_amdgcn_sched_barrier(0);
            s2[1] = mfma_bf16(k.m, qm, s2[1]);
            if (more) split_k(nx, j + 1, 2);
            __builtin_amdgcn_sched_barrier(0);
            s2[1] = mfma_bf16(k.m, qh, s2[1]);
            if (more) split_k(nx, j + 1, 3);
            __builtin_amdgcn_sched_barrier(0);
            s2[0] = mfma_bf16(k.h, qh, s2[0]);
            s2[1] = mfma_bf16(k.h, qm, s2[1]);
#pragma unroll
            for (int u = 0; u < VK; ++u) next_v(u);
            __builtin_amdgcn_sched_barrier(0);
        }
        floatx16 s = s2[0] + s2[1];
        {
            const auto next_v = load_v(src, 8, std::integral_constant<int, 8>());
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 8; ++v) next_v(v);   // (requested with the others they spill)
        }
        keep_here(s);
        __builtin_amdgcn_sched_barrier(0);
        softmax(std::true_type(), t, s);
        Split pr[2];                                 // probabilities of the block's 16-key halves
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) pr[c].pair(i, s[8 * c + 2 * i], s[8 * c + 2 * i + 1]);
#pragma unroll
        for (int i = 0; i < 4; ++i) split_v(sp[0], 0, i);
#pragma unroll
        for (int u = 0; u < 2 * T; ++u) {
            const Split& v = sp[u & 1];
            Split& nx = sp[(u + 1) & 1];
            const Split& x = pr[u / T];
            floatx16& acc = o[u % T];
            auto next = [&](int i) {
                if (u + 1 < 2 * T) split_v(nx, u + 1, i);
                else split_k(nx, 0, i);              // of the next block
            };
            __builtin_amdgcn_sched_barrier(0);
            if (u == 2 * T - 1) { read_k(0); read_k(1); }        // of the next block
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_bf16(v.l, x.h, acc);
            next(0);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_bf16(v.h, x.l, acc);
            next(1);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_bf16(v.m, x.m, acc);
            next(2);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_bf16(v.m, x.h, acc);
            next(3);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma_bf16(v.h, x.m, acc);
            acc = mfma_bf16(v.h, x.h, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    wait_loads();                                    // (of a block that does not exist; the slots are about to be written)
    // the cached state that this lane merges, requested before the waves wait for each other (before the loop: 16 more registers)
    const long long ri = row_index(p, sq, wk.b, wk.h, rok ? r : row0);
    const long long col0 = T * (8 * wave + 4 * hf);
    floatx4 acc0[T];
    float m0 = -INFINITY, l0 = 0.f;
    if (flags & kEngLoadState) {
        m0 = a.Min[ri];
        l0 = a.Lin[ri];
#pragma unroll
        for (int c = 0; c < T; ++c) acc0[c] = *(const floatx4*)(a.Accin + ri * D + col0 + 4 * c);
    }
    // What the parts do not hold.  An infinite input, or one that its first part rounds to infinity, has none (inf - inf): results
    // that are not finite, as with queries out of range.  What lies below 2^-110 loses up to 2^-134:
    //  - an entry of V: at most 2^-134 l in a result, less than 2^-24 of one that is at least 2^-96 l;
    //  - an entry of K, with queries of at most 2^40: less than 2^-86 in a score, 2^-23 of a row's largest that is at
    //    least 2^-63, and nothing in a probability;
    //  - a probability, 2^100 times smaller than a row's largest or more: less than 2^-48 of every result and key, if no entry of
    //    V is above 2^86 times the smallest result.
    // Where a result or a largest score is smaller, but not 0 (made of zeros, as in padded columns; entries below 2^-134 count as
    // such beside others), where all of a row is 0 or scores lie that far apart, the wave looks whether its rows of V or K
    // hold such entries.  If so, and where results are not finite, it takes its blocks again with the fp32 instruction.
    // d = 128, 4000 tokens, 8 heads, dense: 214 us; half of V zeros 206; scores 90 nats apart 320 (every row of V looked at);
    // V below 2^-115 604 (fp32 instruction alone, with K and V straight to registers: 327 to 343).
    {
        const float lt = sum_halves(l);
        float least = INFINITY, most = 0.f;          // (of numbers only: else these are not)
#pragma unroll
        for (int db = 0; db < T; ++db)
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const float x = fabsf(o[db][v]), y = fabsf(o[db][v + 1]);
                least = __builtin_elementwise_minimum(__builtin_elementwise_minimum(x, y), least);
                most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), most);
            }
        const bool odd = !(__builtin_elementwise_maximum(most, lt) < INFINITY);
        const bool low_s = m != 0.f && fabsf(m) < 0x1p-63f, deep = (m - smin) * c2 > 100.f;
        bool again = __any(odd);
        if (__builtin_expect(__any(odd || least < 0x1p-96f * lt || low_s || deep), 0) && !again) {
            float small = INFINITY;                  // the smallest result of the row but 0
#pragma unroll
            for (int db = 0; db < T; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) small = o[db][v] != 0.f ? fminf(small, fabsf(o[db][v])) : small;
            const bool low_o = small < 0x1p-96f * lt || (most == 0.f && lt > 0.f);
            const float limit = __any(deep) ? 0x1p86f * wave_reduce<1>(small, [](float a, float b) { return fminf(a, b); }) : INFINITY;
            // an entry below 2^-100 but 0, or above the limit (always_inline: outlined, it would take o through memory)
            auto holds = [&](const float* rows, long long stride, float top) __attribute__((always_inline)) -> bool {
                bool found = false;
#pragma unroll 1
                for (int t = wave; t < nT && !found; t += NW) {
                    const int kk = key_of(t);
                    floatx4 x[KB * D / 256];
#pragma unroll
                    for (int i = 0; i < KB * D / 256; ++i) {
                        const int e = 256 * i + 4 * lane;
                        x[i] = *(const floatx4*)(rows + __shfl(kk, e / D, 64) * stride + e % D);
                    }
#pragma unroll
                    for (int i = 0; i < KB * D / 256; ++i)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            found |= x[i][c] != 0.f && (fabsf(x[i][c]) < 0x1p-100f || fabsf(x[i][c]) > top);
                    found = __any(found);
                }
                return found;
            };
            again = (__any(low_s) && holds(kb_, p.ks[2], INFINITY)) || (__any(low_o || deep) && holds(vb_, p.vs[2], limit));
        }
        l = lt;
        if (__builtin_expect(again, 0)) {
            reset();
#pragma unroll 1
            for (int t = wave; t < nT; t += NW) {
                const int kk = key_of(t);
                const float* ksrc = kb_ + 4 * hf + (long long)kk * p.ks[2];
                floatx16 s2[2] = {kZero16, kZero16};
#pragma unroll 1
                for (int c = 0; c < D; c += 8) {     // k slot hf of step e is column c + 4 hf + e
                    const floatx4 x = *(const floatx4*)(ksrc + c), y = *(const floatx4*)(qsrc - 4 * hf + c);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s2[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], s2[e & 1], 0, 0, 0);
                }
                floatx16 s = s2[0] + s2[1];
                keep_here(s);
                softmax(std::false_type(), t, s);
                v_rows(kk);
#pragma unroll
                for (int v = 0; v < 16; ++v) {       // k slot hf of step v is key 8 (v / 4) + 4 hf + v % 4
                    load_v(v_lane(), v, std::integral_constant<int, 1>())(0);
#pragma unroll
                    for (int db = 0; db < T; ++db)
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(vf[v], db), s[v], o[db], 0, 0, 0);
                }
            }
            l = sum_halves(l);
        }
    }

    // ---- merge the four waves' states.  Wave w finishes O^T registers 4 w .. 4 w + 3 of every column
    // block: of row n the columns T (8 w + 4 hf) .. + 4 T - 1.
    __syncthreads();                                 // the query parts are no longer read
#pragma unroll
    for (int db = 0; db < T; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) ((float*)slot(2 * db + (v >> 3))[wave])[64 * (v & 7) + lane] = o[db][v];
    if (hf == 0) { sm.st.m[wave][n] = m; sm.st.l[wave][n] = l; }
    __syncthreads();

    float mall = -INFINITY;
    if (flags & kEngLoadState) {
        m0 = m0 / p.sigma;
        mall = m0;
    }
    float mw[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mw[w] = sm.st.m[w][n];
        mall = fmaxf(mall, mw[w]);
    }
    auto scale_of = [&](float x) -> float {          // a part that has seen no key counts for nothing
        return x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x - mall) * c2);
    };
    float lall = 0.f, res[4 * T];                    // res[T e + db]: column T (8 wave + 4 hf) + T e + db
    if (flags & kEngLoadState) {
        const float f0 = scale_of(m0);
        lall = l0 * f0;
#pragma unroll
        for (int c = 0; c < 4 * T; ++c) res[c] = acc0[c / 4][c % 4] * f0;
    } else {
#pragma unroll
        for (int c = 0; c < 4 * T; ++c) res[c] = 0.f;
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = scale_of(mw[w]);
        lall = fmaf(sm.st.l[w][n], f, lall);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int db = 0; db < T; ++db) {
                const float* ow = (const float*)(wave < 2 ? slot(2 * db)[w] : slot(2 * db + 1)[w]);      // registers 4 wave + e
                res[T * e + db] = fmaf(ow[64 * ((4 * wave + e) & 7) + lane], f, res[T * e + db]);
            }
    }

    float ms = mall * p.sigma;
    if ((flags & kEngParts) && !direct && wave == 0) {
        const float sum = half_sum(rok ? ms : 0.f);
        if (lane == 0) a.qlo_norm[part_index()] = sum;
    }
    if (!rok) return;
    const bool first = wave == 0 && hf == 0;
    bool store_out = (flags & kEngStoreOut) != 0;
    if ((flags & kEngStoreState) && direct) {
        // what stage 3 makes of a cached state and an empty list, bit for bit
        ms = ms / p.sigma * p.sigma;
        store_out = true;
    } else if (flags & kEngStoreState) {
        if (first) { a.Mout[ri] = ms; a.Lout[ri] = lall; }
        if (a.Accout) {
            float* dst = a.Accout + ri * D + col0;
#pragma unroll
            for (int c = 0; c < 4 * T; c += 4) *(floatx4*)(dst + c) = floatx4{res[c], res[c + 1], res[c + 2], res[c + 3]};
        }
    }
    if (store_out) {
        const float inv = 1.f / lall;
        float* dst = (float*)a.out + tok_offset(p, p.os, sq, wk.b, wk.h, r) + col0;
#pragma unroll
        for (int c = 0; c < 4 * T; c += 4)
            *(floatx4*)(dst + c) = floatx4{res[c] * inv, res[c + 1] * inv, res[c + 2] * inv, res[c + 3] * inv};
        if (a.lse && first) a.lse[ri] = ms + logf(lall);
    }
}
}  // namespace

int launch_engine_fp32(const EngineArgs& ea, hipStream_t st) {
    const KParams& p = ea.p;
    const long long total = (long long)p.nblk_max * ((p.bq + RT - 1) / RT) * p.Hq * p.B;
    const dim3 grid((unsigned)(total < kGridX ? total : kGridX), (unsigned)((total + kGridX - 1) / kGridX));
    TileMap map;
    map.set(p);
    const long long stride = p.ks[2] > p.vs[2] ? p.ks[2] : p.vs[2];
    const bool wide = stride >= (1ll << 30) || (long long)p.N * stride >= (1ll << 30);
    switch ((p.d * 128 + ea.flags) * 2 + wide) {
#define AA_ENGINE_CASE(d, F, w) \
    case (((d) * 128 + (F)) * 2 + w): return (int)launch_kernel(engine_fp32_kernel<(d), (F), w>, grid, dim3(64 * NW), 0, st, ea, map);
#define AA_ENGINE_CASES(d, w)                                            \
    AA_ENGINE_CASE(d, kEngAnchorRegion | kEngStoreState, w)              \
    AA_ENGINE_CASE(d, kEngAnchorRegion | kEngStoreState | kEngParts, w)  \
    AA_ENGINE_CASE(d, kEngList | kEngLoadState | kEngStoreOut, w)        \
    AA_ENGINE_CASE(d, kEngList | kEngAnchorRegion | kEngStoreOut, w)     \
    AA_ENGINE_CASE(d, kEngAnchorRegion | kEngDense | kEngStoreOut, w)
    AA_ENGINE_CASES(32, false)
    AA_ENGINE_CASES(64, false)
    AA_ENGINE_CASES(128, false)
    AA_ENGINE_CASES(32, true)
    AA_ENGINE_CASES(64, true)
    AA_ENGINE_CASES(128, true)
#undef AA_ENGINE_CASES
#undef AA_ENGINE_CASE
    default: return -1;
    }
}

}  // namespace aa
