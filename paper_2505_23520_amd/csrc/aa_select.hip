// Stage 2 of AnchorAttention, difference-aware stripe identification
// (arXiv 2505.23520 Sec. 3.2 mask, Algorithm 2, and the step rule of Sec. 3.4):
//   pool_q   : qbar_i = mean of query block i's rows               (Alg. 2, avgpool(Q))
//   mask     : bit (g, j) = OR_{i in g} [ xbar_i - sigma <qbar_i, k_j> <= theta ],  j in C_g
//   count    : |I_g| = popcount of the group's bits (added up by the stripe mask kernels as they write them; a kernel of its
//              own for block granularity only)
//   scan     : offsets = exclusive prefix sum of the counts rounded up to 64 (not in the fused call, see fill_kernel)
//   fill     : ballot / prefix-popcount stream compaction of the bits into ascending lists
// The bf16 mask kernel is a skinny MFMA GEMM (pooled rows x keys); the pooled
// query, an fp32 mean, is split into bf16 hi + lo parts so that the products with
// the (exactly bf16) keys carry ~16 mantissa bits and the threshold decision does
// not depend on bf16 rounding of the mean.
#include "aa_common.h"
#include "aa_pool.h"
#include "aa_select.h"

namespace aa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
constexpr floatx16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

namespace {
__device__ __forceinline__ float bf16_to_f(unsigned short b) { return __uint_as_float((unsigned)b << 16); }
__device__ __forceinline__ unsigned short f_to_bf16_rne(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
}  // namespace

namespace {
// c more selected columns in segment seg of group t.  The group's total is added up here only if the scan does not
// do it from the segments.
__device__ __forceinline__ void add_counts(const SelectArgs& a, long long t, int seg, int c) {
    atomicAdd(&a.segcount[t * a.nseg + seg], c);
    if (!a.sum_segs) atomicAdd(&a.counts[t], c);
}
}  // namespace

// ------------------------------------------------------------------ pool_q
// grid (nblk_max, Hq [+ Hkv], B).  bf16: 256 threads = the four waves of the tile engines; writes
// hi/lo bf16 rows of 128 and the norm of the lo row (aa_pool.h).  With kmax_blk set (stripe granularity)
// the grid has Hkv more rows in y, whose work-groups write the largest key norm of their key block, and the
// mask kernel's counters are cleared.  pool_skip_q: the queries were pooled by stage 1 already, the
// grid holds the Hkv key rows only.
__global__ __launch_bounds__(256) void pool_q_bf16_kernel(SelectArgs a) {
    const KParams& p = a.p;
    const int i = blockIdx.x, b = blockIdx.z, tid = threadIdx.x;
    if (a.kmax_blk) {
        const long long wg = blockIdx.x + (long long)gridDim.x * (blockIdx.y + (long long)gridDim.y * blockIdx.z);
        clear_counters(a.counts, a.groups_total, a.segcount, a.nseg, a.total, a.total ? a.stats : nullptr, wg * 256 + tid,
                       (long long)gridDim.x * gridDim.y * gridDim.z * 256);
    }
    const Seq sq = seq_of(p, b);
    const int r0 = i * p.bq;
    if (r0 >= sq.len) return;
    const int r1 = min(r0 + p.bq, sq.len);
    __shared__ float red[4][128];
    const int y = blockIdx.y + (a.pool_skip_q ? p.Hq : 0);
    if (y >= p.Hq) {
        const int hk = y - p.Hq;
        KeyNorm kn;
        kn.load((const unsigned short*)a.k + tok_offset(p, p.ks, sq, b, hk, 0), p.ks[2], r0, r1, tid);
        const float big = kn.wave_max();
        if ((tid & 63) == 0) red[0][tid >> 6] = big;
        __syncthreads();
        if (tid == 0) a.kmax_blk[kblk_index(p, sq, b, hk, i)] = KeyNorm::block(red[0]);
        return;
    }
    // query block i of head h: the fragments of the tile engines (wave w: rows 32 w .. 32 w + 31, lane
    // (n, hf): the 16-byte pieces 16 ks + 8 hf of row n), pooled by the code the engines use
    const int h = y;
    const int lane = tid & 63, wave = tid >> 6, n = lane & 31, hf = lane >> 5;
    const int r = r0 + 32 * wave + n;
    bf16x8 qf[8];
    {
        const __bf16* src = (const __bf16*)a.q + tok_offset(p, p.qs, sq, b, h, r < r1 ? r : r0);
        const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 x = *(const bf16x8*)(src + 16 * ks + 8 * hf);
            qf[ks] = r < r1 ? x : zero8;
        }
    }
    float s0, s1;
    pool_wave_columns(qf, n, s0, s1);
    pool_block_put(red, wave, n, hf, s0, s1);
    __syncthreads();
    if (tid < 64) pool_block_write(red, lane, r1 - r0, blk_index(p, sq, b, h, i), a.qp_hi, a.qp_lo, a.qlo_norm);
}

// fp32: 256 threads per query block.  With qp_f32 set, the block mean of the queries; with m_rows set, the pooled anchor (mean of
// M over the block's rows): the fp32 engine's work-groups own 32 rows each, not a block; with segcount set, the
// counters of stage 2 are cleared.  Sums per 32-row tile and their order are those of stage 1, which adds rows 16, 8, 4, 2 and 1
// apart (half_sum): a thread holds 16 bytes of every other row of a tile, a row's threads fetch it together.
__device__ __forceinline__ float block_sum(float t0, float t1, float t2, float t3) { return (t0 + t1) + (t2 + t3); }

__global__ __launch_bounds__(256) void pool_fp32_kernel(SelectArgs a) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    const KParams& p = a.p;
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (a.segcount) {
        const long long wg = blockIdx.x + (long long)gridDim.x * (blockIdx.y + (long long)gridDim.y * blockIdx.z);
        clear_counters(a.counts, a.groups_total, a.segcount, a.nseg, a.total, a.total ? a.stats : nullptr, wg * 256 + tid,
                       (long long)gridDim.x * gridDim.y * gridDim.z * 256);
    }
    // fused prefill: stage 1 has finished the rows of groups without candidates and left no M for them; stage 2 reads neither
    // their pooled anchors nor their pooled queries
    if (i < a.first_block) return;
    const Seq sq = seq_of(p, b);
    const int r0 = i * p.bq;
    if (r0 >= sq.len) return;
    const int nrows = min(p.bq, sq.len - r0);
    const long long bi = blk_index(p, sq, b, h, i);
    const float inv = 1.f / (float)nrows;
    __shared__ __attribute__((aligned(16))) float part[4][2][128];
    __shared__ float mpart[4];
    if (a.m_rows) {                                      // a wave per tile; rows that do not exist count 0
        const int r = 32 * wave + (lane & 31);
        const float sum = half_sum(r < nrows ? a.m_rows[row_index(p, sq, b, h, r0 + r)] : 0.f);
        if (lane == 0) mpart[wave] = sum;
    }
    if (a.qp_f32) {
        const int d4 = p.d / 4, c = tid % d4, odd = tid / d4 & 1, tile = tid / d4 >> 1;
        if (tile < 4) {
            const float* src = (const float*)a.q + tok_offset(p, p.qs, sq, b, h, r0) + 4 * c;
            floatx4 x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int r = 32 * tile + 2 * k + odd;
                x[k] = *(const floatx4*)(src + (long long)min(r, nrows - 1) * p.qs[2]);
                if (r >= nrows) x[k] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int w = 8; w >= 1; w /= 2)
#pragma unroll
                for (int k = 0; k < w; ++k) x[k] += x[k + w];
            *(floatx4*)&part[tile][odd][4 * c] = x[0];
        }
    }
    __syncthreads();
    if (a.m_rows && tid == 0) a.xa_out[bi] = block_sum(mpart[0], mpart[1], mpart[2], mpart[3]) * inv;
    if (a.qp_f32 && tid < p.d) {
        float t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = part[e][0][tid] + part[e][1][tid];
        a.qp_f32[bi * p.d + tid] = block_sum(t[0], t[1], t[2], t[3]) * inv;
    }
}

// ------------------------------------------------------------------ mask, bf16 MFMA
// One work-group = one (query head, row tile, key chunk): 256 threads = 4 waves, three work-groups
// per CU.  A row tile holds RT = 128 - 128 % step pooled rows, so no group straddles two tiles; wave
// w owns its rows 32 w .. 32 w + 31.  The chunk's keys pass through LDS in 64-key tiles (16-byte
// direct-to-LDS loads, two stages, same padded group layout as the attention engine).
// C[key][row] = K qbar^T: keys are the M dimension, pooled rows the N dimension, so one lane owns
// one pooled row and collects the compare bits of its row in registers.
//
// Grid: one dimension.  Every launched work-group has exactly one chunk of work (row tiles only
// count the chunks below their last group's window).  A key chunk (256 KB of K) is needed by the
// query heads of its KV head times the row tiles at or above it -- up to 32 work-groups at 128k
// tokens -- and is read from HBM once if those run at the same time on one XCD (each XCD has its
// own L2).  The hardware deals consecutive work-group ids round-robin to the 8 XCDs, so id
// -> logical index L = (id % 8) * per_xcd + id / 8 gives each XCD a contiguous range of L, walked
// in order; L enumerates sequences, inside a sequence the KV heads, inside a (sequence, KV head)
// pair the key chunks in ascending order, inside a chunk the row tiles that need it, and the
// query heads of the KV head fastest.
constexpr int kMaskTileKeys = 64;
constexpr int kMaskChunkTiles = kMaskChunkKeys / kMaskTileKeys;   // tiles per work-group
constexpr int kKGrp = 1024 + 16;                         // bytes per group of four K rows + pad
constexpr int kKTile = 16 * kKGrp;
typedef __attribute__((address_space(3))) void lds_void;

namespace {
// Work-group barrier that makes LDS writes visible but leaves vector-memory operations in flight
// (__syncthreads() also waits for every outstanding load, the prefetched tiles included).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
}  // namespace

__global__ __launch_bounds__(256, 3) void mask_bf16_kernel(SelectArgs a) {
    const KParams& p = a.p;
    // Work items that exist: per sequence, items(len) x Hq (a packed batch's shorter sequences have
    // fewer than the longest one, for which the host sized the grid).  Every XCD gets an equal,
    // contiguous share of them, so the load is balanced whatever the mix of lengths.
    const int span_blk = p.bq;
    unsigned real = 0;                                   // (the host has checked that 31 bits hold it)
    if (p.packed) {
        for (int s = 0; s < p.B; ++s)
            real += (unsigned)mask_pair_items((p.cu[s + 1] - p.cu[s] + span_blk - 1) / span_blk, p.step, p.bq, p.w, p.n_init,
                                              a.mask_span);
        real *= (unsigned)p.Hq;
    } else {
        real = (unsigned)a.mask_items * (unsigned)p.Hq * (unsigned)p.B;
    }
    const unsigned per_xcd = (real + 7u) / 8u;
    const unsigned slot = blockIdx.x >> 3;
    unsigned L = (blockIdx.x & 7u) * per_xcd + slot;
    if (slot >= per_xcd || L >= real) return;
    // L -> sequence b, then inside the sequence KV head, item, query head of the KV head
    int b = 0, items_b = a.mask_items;
    if (p.packed) {
        for (;; ++b) {
            items_b = mask_pair_items((p.cu[b + 1] - p.cu[b] + span_blk - 1) / span_blk, p.step, p.bq, p.w, p.n_init,
                                      a.mask_span);
            const unsigned n = (unsigned)items_b * (unsigned)p.Hq;
            if (L < n) break;
            L -= n;
        }
    } else if (p.B > 1) {
        const unsigned n = (unsigned)items_b * (unsigned)p.Hq;
        b = (int)(L / n);
        L -= (unsigned)b * n;
    }
    const int per_pair = items_b * p.grp;
    const int hk = (int)(L / (unsigned)per_pair), e = (int)(L % (unsigned)per_pair);
    const int h = hk * p.grp + e % p.grp;
    const Seq sq = seq_of(p, b);
    const int nblk = (sq.len + p.bq - 1) / p.bq;
    const int RT = mask_row_tile(p.step);
    const int ny = (nblk + RT - 1) / RT;
    // item e / grp of this sequence -> (chunk, row tile).  Row tile y has candidates in its first
    // n(y) chunks and n is non-decreasing in y, so chunks n(y-1) .. n(y)-1 are needed by the
    // ny - y row tiles y .. ny-1: walk these levels.
    int rt = -1, chunk = 0;
    {
        int item = e / p.grp, prev = 0;
        for (int y = 0; y < ny; ++y) {
            const int n = mask_tile_chunks(nblk, y, p.step, p.bq, p.w, p.n_init, a.mask_span);
            const int width = ny - y, items = (n - prev) * width;
            if (item < items) {
                chunk = prev + item / width;
                rt = y + item % width;
                break;
            }
            item -= items;
            prev = n;
        }
    }
    if (rt < 0) return;                                  // a shorter sequence of a packed batch
    const int row_t0 = rt * RT;                          // first pooled row (query block) of the tile
    if (row_t0 >= nblk) return;
    const int rows_here = min(RT, nblk - row_t0);
    const int g_first = row_t0 / p.step;
    const int g_last = (row_t0 + rows_here - 1) / p.step;
    const int Wmax = window_start(p, g_last);            // candidates of the tile end before Wmax
    const int key_lo = (p.n_init / kMaskTileKeys) * kMaskTileKeys;
    if (key_lo + chunk * a.mask_span >= Wmax) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hf = lane >> 5;
    // one LDS object per stage: the compiler can then tell that the asynchronous loads into one stage
    // do not alias the operand reads from another (with a single array it waits for the loads it
    // has just issued before every tile's first read)
    __shared__ __attribute__((aligned(16))) char kt0[kKTile], kt1[kKTile];
    // compare words of the whole chunk: [tile][pooled row][word]
    __shared__ unsigned rowword[kMaskChunkTiles][128][2];
    __shared__ int gcount[128];                          // selected columns of each group in this work-group's keys

    // B operand: this lane's pooled query row, hi and lo parts, columns 16 ks + 8 hf .. +8
    bf16x8 bhi[8], blo[8];
    const int lr = 32 * wave + n;                        // row inside the tile
    const bool rok = lr < rows_here;
    const long long bi = blk_index(p, sq, b, h, row_t0 + (rok ? lr : 0));
    {
        const unsigned short* hi = (const unsigned short*)a.qp_hi + bi * 128;
        const unsigned short* lo = (const unsigned short*)a.qp_lo + bi * 128;
        const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 x = *(const bf16x8*)(hi + 16 * ks + 8 * hf);
            const bf16x8 y = *(const bf16x8*)(lo + 16 * ks + 8 * hf);
            bhi[ks] = rok ? x : zero8;
            blo[ks] = rok ? y : zero8;
        }
    }
    // The threshold test xbar - sigma s <= theta is the sign of s + (theta - xbar) / sigma: that
    // constant of the lane's row is the initial accumulator of the score MFMAs, so the accumulators
    // come out as margins (in raw dot-product units) and their sign bits are the decisions.
    // -inf = no such row (never selects).
    const float toff = rok ? (p.theta - (p.use_anchor ? a.xa[bi] : 0.f)) / p.sigma : -INFINITY;
    floatx16 cinit;
#pragma unroll
    for (int v = 0; v < 16; ++v) cinit[v] = toff;
    const float lo_norm = rok ? a.qlo_norm[bi] : 0.f;

    const unsigned short* kbase = (const unsigned short*)a.k + tok_offset(p, p.ks, sq, b, hk, 0);
    const unsigned kstb = (unsigned)p.ks[2] * 2u;
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)kbase, 0, (int)((unsigned)(sq.len - 1) * kstb + 256u), 0x00020000);
    // loader: in the load of group gi lane l fetches the 16-byte chunk l % 16 of key 16 (l / 16) + gi
    auto load_tile = [&](int t0, char* buf) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int gi = 4 * wave + j;
            const int key = min(t0 + 16 * (lane >> 4) + gi, sq.len - 1);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, (lds_void*)(buf + gi * kKGrp), 16,
                                                     (int)((unsigned)key * kstb + 16u * (lane & 15)), 0, 0, 0);
        }
    };
    const int nwords = a.nwords;
    const int ngrp = (nblk + p.step - 1) / p.step;
    const int ngt = g_last - g_first + 1;
    // OR the rows of each group, clip to the group's candidate range, write the bit words of a tile
    // a work-group walks its mask_span keys in chunks of at most kMaskChunkKeys: the pooled rows stay in
    // registers, the compare words of a chunk are combined and written before the next one starts
    const int koff = (n & 15) * kKGrp + (n >> 4) * 256 + 16 * hf;   // K row of key 32 kb + n
    if (tid < 128) gcount[tid] = 0;                      // (the first tile's barrier publishes it)
    const int span_end = min(key_lo + (chunk + 1) * a.mask_span,
                             ((Wmax + kMaskTileKeys - 1) / kMaskTileKeys) * kMaskTileKeys);
    for (int chunk0 = key_lo + chunk * a.mask_span; chunk0 < span_end; chunk0 += kMaskChunkKeys) {
    const int chunk1 = min(chunk0 + kMaskChunkKeys, span_end);
    const int ntiles = (chunk1 - chunk0) / kMaskTileKeys;
    // |sigma <lo, k>| <= sigma |lo| max|k| over the chunk's keys: a score whose margin from the hi
    // products alone is farther from zero than that keeps its sign whatever the lo products add
    // (the chunk's key blocks side by side, behind the first tile's loads: a loop over them waits out one load after the
    // other; all of stage 2 with this and the 32-bit index arithmetic above: 16k tokens 54.2 -> 53.7 us, 128k 879 -> 874)
    load_tile(chunk0, kt0);
    float kbig = 0.f;
    {
        const float* kn = a.kmax_blk + kblk_index(p, sq, b, hk, 0);
        const int J0 = chunk0 / 128, J1 = min(chunk1 - 1, sq.len - 1) / 128;
#pragma unroll
        for (int j = 0; j <= kMaskChunkKeys / 128; ++j) kbig = fmaxf(kbig, kn[min(J0 + j, J1)]);
    }
    const float lo_bound = 1.001f * lo_norm * kbig;
    // After the tile loop: OR the rows of each group, clip to the group's candidate range, write the
    // bit words of the chunk.  (This stays outside the tile loop: before an inner loop that reads
    // LDS, and before an LDS atomic, the compiler waits for every outstanding asynchronous load
    // into LDS, which would serialise the tile loads with the arithmetic.)
    auto combine_all = [&]() {
        // consecutive threads take consecutive words of one group (coalesced stores); each starts
        // its walk over the group's rows at a different row, which spreads a wave's LDS reads over
        // the banks (from the same row they would be 16 reads to one bank)
        for (int e = tid; e < ngt * 2 * ntiles; e += 256) {
            const int wi = e & 1, tl = (e >> 1) % ntiles, gi = (e >> 1) / ntiles;
            const int g = g_first + gi;
            const int lr0 = g * p.step - row_t0;
            const int nr = min(p.step, rows_here - lr0);
            unsigned wd = 0;
            int s = tl % nr;
            for (int c = 0; c < nr; ++c) {
                wd |= rowword[tl][lr0 + s][wi];
                s = s + 1 == nr ? 0 : s + 1;
            }
            const int j0 = chunk0 + tl * kMaskTileKeys + 32 * wi;
            const int Wg = window_start(p, g);
            const int lo = max(p.n_init - j0, 0), hi = min(Wg - j0, 32);   // keep n_init <= j0 + bit < Wg
            unsigned keep = 0;
            if (hi > lo) keep = (hi - lo >= 32) ? 0xffffffffu : (((1u << (hi - lo)) - 1u) << lo);
            wd &= keep;
            if (g < ngrp && j0 / 32 < nwords) {
                a.bits[grp_index(p, sq, b, h, g) * nwords + j0 / 32] = wd;
                if (wd) atomicAdd(&gcount[gi], __popc(wd));
            }
        }
    };

    // two stages: the loads of tile t + 1 are issued at the start of tile t and awaited at its end.
    // (Three stages with a two-tile lead were 12 % slower: 50 KB of LDS per work-group leave room for
    // three work-groups per CU, 66 KB only for two, and the third hides both the load latency and
    // the 4 us a CU needs to replace a finished work-group.)  Every tile issues its four loads
    // unconditionally (past the chunk's end the last tile is fetched again into the stage nobody
    // reads any more), so no statically possible path reads a stage whose loads might be pending.
    __builtin_amdgcn_s_waitcnt(0x0F70);              // tile 0 is there
    lds_barrier();
    auto tile_step = [&](int t, const char* Kcur, char* Kld) {
        load_tile(chunk0 + min(t + 1, ntiles - 1) * kMaskTileKeys, Kld);
        // higher issue priority for the MFMA block than for the bit packing: a wave with matrix work
        // wins over the SIMD's other waves that are in their vector-ALU part (-3 %)
        __builtin_amdgcn_s_setprio(2);
        const char* Kb = Kcur + koff;
        floatx16 c[2];
        // hi products first.  The two accumulators alternate, so no MFMA waits for the one issued
        // just before it
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 kf0 = *(const bf16x8*)(Kb + 32 * ks);
            const bf16x8 kf1 = *(const bf16x8*)(Kb + 512 + 32 * ks);
            c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, bhi[ks], ks == 0 ? cinit : c[0], 0, 0, 0);
            c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf1, bhi[ks], ks == 0 ? cinit : c[1], 0, 0, 0);
        }
        // operand reads run ahead of their MFMAs
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        __builtin_amdgcn_s_setprio(0);
        float nearest = INFINITY;                    // smallest |margin| of the lane's 32 scores
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; v += 2)
                nearest = fminf(fminf(nearest, fabsf(c[kb][v])), fabsf(c[kb][v + 1]));       // v_min3_f32
        if (__any(nearest <= lo_bound)) {
            // some decision of this wave's tile hangs on the lo products: add them (rare: only
            // margins within ~1e-2 of zero get here)
            __builtin_amdgcn_s_setprio(2);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const bf16x8 kf0 = *(const bf16x8*)(Kb + 32 * ks);
                const bf16x8 kf1 = *(const bf16x8*)(Kb + 512 + 32 * ks);
                c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, blo[ks], c[0], 0, 0, 0);
                c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf1, blo[ks], c[1], 0, 0, 0);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        // Sign bits shifted into a word (one instruction per score, no compare / select chains).
        // The lane gathers the bits of its 16 keys per 32-key block (accumulator register v holds
        // key 8 (v / 4) + 4 hf + v % 4, i.e. its nibbles alternate with those of the lane 32 away,
        // which holds the other 16 keys of the same row).
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            unsigned neg = 0;                        // bit v = sign of score v's margin
#pragma unroll
            for (int v = 15; v >= 0; --v)
                neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(c[kb][v]), 31);
            unsigned wd = ~neg & 0xffffu;
            wd = (wd | (wd << 8)) & 0x00ff00ffu;     // nibble i of the 16 bits -> nibble 2 i of the word
            wd = (wd | (wd << 4)) & 0x0f0f0f0fu;
            wd <<= 4 * hf;
            const auto both = __builtin_amdgcn_permlane32_swap(wd, wd, false, false);
            if (hf == 0) rowword[t][lr][kb] = both[0] | both[1];
        }
        // tile t + 1 has landed
        __builtin_amdgcn_s_waitcnt(0x0F70);
        lds_barrier();
    };
    static_assert(kMaskChunkTiles % 2 == 0, "the tile loop below alternates two stages");
#pragma unroll 1
    for (int t2 = 0; t2 < ntiles; t2 += 2) {
        tile_step(t2, kt0, kt1);
        if (t2 + 1 >= ntiles) break;
        tile_step(t2 + 1, kt1, kt0);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);              // the trailing loads have landed before LDS is reused
    combine_all();
    __syncthreads();                                 // rowword is reused by the next chunk
    }
    // a work-group's keys lie in one segment
    if (tid < ngt && gcount[tid])
        add_counts(a, grp_index(p, sq, b, h, g_first + tid), chunk * a.mask_span / kSegKeys, gcount[tid]);
}

// ------------------------------------------------------------------ mask, fp32 MFMA
// grid (key blocks of 32 / 4, Hq, B), 256 threads = 4 waves, one 32-key block per wave.  The wave keeps
// its keys in registers (B operand of v_mfma_f32_32x32x2_f32: lane (n, hf) holds the 16-byte pieces
// 8 j + 4 hf of key n) and walks the pooled rows of the groups that have the block among their
// candidates, 32 rows at a time; a lane then holds 16 rows' products with its key.  Its decisions
// become one 32-bit word of rows, and a ballot per group gives the bit word of the 32 keys.
// Latency-bound at the sizes of fp32 use; 4000 tokens, 8 / 2 heads, d = 128: 59 us with one key per thread and
// vector FMAs (every thread streaming its own key row), 9 us so; the pooling kernel 32 -> 5 us.
// PARTS > 0: the pooled rows are made here from stage 1's sums per 32-row tile (fused call: a launch less, 4 us; 1024 tokens, 1 head,
// d = 64: 31.0 -> 28.4 us for the whole call).
// At most PARTS tiles a block.
template <int D, int PARTS>
__global__ __launch_bounds__(256) void mask_fp32_kernel(SelectArgs a) {
    constexpr int NK = D / 8;
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    const KParams& p = a.p;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 31, hf = lane >> 5;
    const int h = blockIdx.y, b = blockIdx.z, hk = h / p.grp;
    const Seq sq = seq_of(p, b);
    const int nblk = (sq.len + p.bq - 1) / p.bq;
    const int j0 = 32 * (4 * (int)blockIdx.x + wave);
    if (j0 >= sq.len || j0 + 32 <= p.n_init) return;
    // first group whose candidates reach into the block: W_g > max(j0, n_init)
    const long long span = (long long)p.bq * p.step;
    const long long g0 = ((long long)max(j0, p.n_init) + p.w) / span + 1;
    if (g0 * p.step >= nblk) return;
    floatx4 kf[NK];
    {
        const float* src = (const float*)a.k + tok_offset(p, p.ks, sq, b, hk, min(j0 + n, sq.len - 1)) + 4 * hf;
#pragma unroll
        for (int j = 0; j < NK; ++j) kf[j] = *(const floatx4*)(src + 8 * j);
    }
    const long long bi0 = blk_index(p, sq, b, h, 0), gi0 = grp_index(p, sq, b, h, 0);
    unsigned carry = 0;                                  // bit word so far of a group that continues in the next tile
    for (int i0 = (int)g0 * p.step; i0 < nblk; i0 += 32) {
        const int rows = min(32, nblk - i0);
        const int blk = i0 + min(n, rows - 1);           // this lane's pooled row
        float xrow = 0.f, inv = 1.f;
        const float* qsrc;
        int nt = 1;                                      // tiles of the block
        if (PARTS > 0) {
            const int rts = (p.bq + 31) / 32, nrows = min(p.bq, sq.len - blk * p.bq);
            const long long t = (bi0 + blk) * rts;
            inv = 1.f / (float)nrows;
            nt = (nrows + 31) / 32;
            float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < PARTS; ++i) m[i] = i < nt ? a.part_m[t + min(i, nt - 1)] : 0.f;
            xrow = block_sum(m[0], m[1], m[2], m[3]) * inv;
            qsrc = a.part_q + t * D + 4 * hf;
        } else {
            qsrc = a.qp_f32 + (bi0 + blk) * D + 4 * hf;
        }
        floatx16 s = kZero16;
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            floatx4 x = *(const floatx4*)(qsrc + 8 * j);
            if (PARTS > 0) {
                floatx4 y[4] = {x, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int i = 1; i < PARTS; ++i) {
                    const floatx4 z = *(const floatx4*)(qsrc + min(i, nt - 1) * D + 8 * j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[i][e] = i < nt ? z[e] : 0.f;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = block_sum(y[0][e], y[1][e], y[2][e], y[3][e]) * inv;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], kf[j][e], s, 0, 0, 0);
        }
        unsigned dec = 0;                                // bit v: decision of row 8 (v / 4) + 4 hf + v % 4
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 8 * (v >> 2) + 4 * hf + (v & 3);
            const float xbar = !p.use_anchor ? 0.f : PARTS > 0 ? __shfl(xrow, row, 64) : a.xa[bi0 + i0 + min(row, rows - 1)];
            dec |= (xbar - p.sigma * s[v] <= p.theta) ? 1u << v : 0u;
        }
        dec = (dec | (dec << 8)) & 0x00ff00ffu;          // nibble i of the 16 bits -> nibble 2 i of the word
        dec = (dec | (dec << 4)) & 0x0f0f0f0fu;
        dec <<= 4 * hf;
        dec |= __shfl_xor(dec, 32, 64);                  // bit i: decision of row i of the tile
        const int g_a = i0 / p.step, g_b = (i0 + rows - 1) / p.step;
        unsigned mine = 0;
        int done = 0;                                    // groups of this tile that end in it
        for (int g = g_a; g <= g_b; ++g) {
            const int lo = max(g * p.step - i0, 0), hi = min((g + 1) * p.step - i0, rows);   // rows lo .. hi - 1
            const unsigned rowmask = (hi - lo >= 32) ? 0xffffffffu : ((1u << (hi - lo)) - 1u) << lo;
            unsigned word = (unsigned)__ballot((dec & rowmask) != 0u);
            if (g == g_a) word |= carry;
            if ((g + 1) * p.step <= i0 + 32 || i0 + 32 >= nblk) {
                if (lane == g - g_a) mine = word;
                done = g - g_a + 1;
            } else {
                carry = word;
            }
        }
        if ((g_b + 1) * p.step <= i0 + 32) carry = 0;
        if (lane < done) {
            const int g = g_a + lane, Wg = window_start(p, g);
            const int lo = max(p.n_init - j0, 0), hi = min(Wg - j0, 32);   // keep n_init <= j0 + bit < Wg
            unsigned keep = 0;
            if (hi > lo) keep = (hi - lo >= 32) ? 0xffffffffu : (((1u << (hi - lo)) - 1u) << lo);
            mine &= keep;
            a.bits[(gi0 + g) * a.nwords + j0 / 32] = mine;
            if (mine) add_counts(a, gi0 + g, (j0 / 32 - seg_word0(p.n_init)) / (kSegKeys / 32), __popc(mine));
        }
    }
}

int launch_mask_fp32(const SelectArgs& a, hipStream_t st) {
    const KParams& p = a.p;
    const dim3 grid((unsigned)((p.N + 127) / 128), (unsigned)p.Hq, (unsigned)p.B);
    const int parts = !a.part_q ? 0 : p.bq <= 32 ? 1 : p.bq <= 64 ? 2 : 4;
    switch (p.d * 8 + parts) {
#define AA_MASK_CASE(d, n) \
    case (d) * 8 + (n): return (int)launch_kernel(mask_fp32_kernel<d, n>, grid, dim3(256), 0, st, a);
#define AA_MASK_CASES(d) AA_MASK_CASE(d, 0) AA_MASK_CASE(d, 1) AA_MASK_CASE(d, 2) AA_MASK_CASE(d, 4)
        AA_MASK_CASES(32)
        AA_MASK_CASES(64)
        AA_MASK_CASES(128)
#undef AA_MASK_CASES
#undef AA_MASK_CASE
        default: return -1;
    }
}

// ------------------------------------------------------------------ block granularity
// One decision per key block (Sec. 2.1.2 / Table 1's block granularity) instead of one per column:
// the difference test of Sec. 3.2 on the block's average key.  Tiny next to the stripe mask
// (pooled rows x pooled keys), so plain fp32 FMAs.

// kbar_J = mean of key block J.  grid (nblk_max, Hkv, B), 256 threads.  bf16 (d = 128): thread
// (c, rs) sums the 16-byte chunk c of rows rs, rs + 16, ...; fp32: one column per thread.
__global__ __launch_bounds__(256) void pool_k_kernel(SelectArgs a) {
    const KParams& p = a.p;
    const int J = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
    const Seq sq = seq_of(p, b);
    const int r0 = J * p.bq;
    if (r0 >= sq.len) return;
    const int r1 = min(r0 + p.bq, sq.len);
    const long long kb = (p.packed ? (long long)hk * p.blk_cap + sq.blk0 : ((long long)b * p.Hkv + hk) * p.blk_cap) + J;
    const long long base = tok_offset(p, p.ks, sq, b, hk, 0);
    const int tid = threadIdx.x;
    if (a.is_bf16) {
        const int c = tid & 15, rs = tid >> 4;
        const unsigned short* src = (const unsigned short*)a.k + base + 8 * c;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int r = r0 + rs; r < r1; r += 16) {
            const uintx4 x = *(const uintx4*)(src + (long long)r * p.ks[2]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[2 * e] += __uint_as_float(x[e] << 16);
                acc[2 * e + 1] += __uint_as_float(x[e] & 0xffff0000u);
            }
        }
        __shared__ float red[16][128];
#pragma unroll
        for (int e = 0; e < 8; ++e) red[rs][8 * c + e] = acc[e];
        __syncthreads();
        if (tid < 128) {
            float s0 = 0.f;
#pragma unroll
            for (int k = 0; k < 16; ++k) s0 += red[k][tid];
            a.kp_f32[kb * 128 + tid] = s0 / (float)(r1 - r0);
        }
    } else {
        const float* src = (const float*)a.k + base;
        for (int c = tid; c < p.d; c += 256) {
            float s0 = 0.f;
            for (int r = r0; r < r1; ++r) s0 += src[(long long)r * p.ks[2] + c];
            a.kp_f32[kb * p.d + c] = s0 / (float)(r1 - r0);
        }
    }
}

// dynamic LDS of mask_block_kernel: step pooled query rows, step anchors, a tile of 64 pooled keys
// (rows padded by 4 floats), one flag per key block
constexpr int kBlkTile = 64;
size_t mask_block_lds_bytes(int N, int d, int bq, int step) {
    return (size_t)step * d * 4 + (size_t)step * 4 + (size_t)kBlkTile * (d + 4) * 4 + (size_t)((N / bq + 15) / 16) * 16;
}

// grid (ngrp_max, Hq, B), 256 threads.  Per pass a tile of 64 pooled keys sits in LDS; lane l of
// every wave owns key block l of the tile, wave w the pooled rows w, w + 4, ... of the group (so
// the query operand is a broadcast read), four rows at a time.
// Needs n_init and the window start to be multiples of bq, so every half word (16 keys) of the
// bit map lies inside one key block and inside or outside C_g as a whole.
__global__ __launch_bounds__(256) void mask_block_kernel(SelectArgs a) {
    const KParams& p = a.p;
    const int g = p.ngrp_max - 1 - (int)blockIdx.x;    // long candidate ranges first
    const int h = blockIdx.y, b = blockIdx.z, hk = h / p.grp;
    const Seq sq = seq_of(p, b);
    const int nblk = (sq.len + p.bq - 1) / p.bq;
    const int i0 = g * p.step;
    if (i0 >= nblk) return;
    const int nb = min(p.step, nblk - i0);
    const int Wg = window_start(p, g);
    if (Wg <= p.n_init) return;
    const int d = p.d, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kst = d + 4;                             // floats per row of the key tile
    extern __shared__ __attribute__((aligned(16))) float bsm[];
    float* qs = bsm;                                   // [step][d]
    float* xs = qs + p.step * d;                       // [step]
    float* kt = xs + p.step;                           // [64][d + 4]
    unsigned char* flag = (unsigned char*)(kt + kBlkTile * kst);   // [key blocks of C_g]
    for (int e = tid; e < nb * d; e += 256) {
        const long long bi = blk_index(p, sq, b, h, i0 + e / d);
        const int c = e % d;
        qs[e] = a.is_bf16 ? bf16_to_f(((const unsigned short*)a.qp_hi)[bi * 128 + c]) +
                                bf16_to_f(((const unsigned short*)a.qp_lo)[bi * 128 + c])
                          : a.qp_f32[bi * d + c];
    }
    for (int s = tid; s < nb; s += 256) xs[s] = p.use_anchor ? a.xa[blk_index(p, sq, b, h, i0 + s)] : 0.f;
    const int J_lo = p.n_init / p.bq, J_hi = Wg / p.bq;
    const long long kb0 = p.packed ? (long long)hk * p.blk_cap + sq.blk0 : ((long long)b * p.Hkv + hk) * p.blk_cap;
    const int d4 = d / 4;
    for (int J0 = J_lo; J0 < J_hi; J0 += kBlkTile) {
        const int nJ = min(kBlkTile, J_hi - J0);
        __syncthreads();                               // previous tile consumed (first pass: qs, xs written)
        for (int e = tid; e < nJ * d4; e += 256) {
            const int r = e / d4, c = e % d4;
            *(float4*)(kt + r * kst + 4 * c) = *(const float4*)(a.kp_f32 + (kb0 + J0 + r) * d + 4 * c);
        }
        __syncthreads();
        int pred = 0;
        if (lane < nJ) {
            const float4* kr = (const float4*)(kt + lane * kst);
            for (int s0 = wave; s0 < nb; s0 += 16) {   // rows s0, s0 + 4, s0 + 8, s0 + 12
                float dot[4] = {0.f, 0.f, 0.f, 0.f};
                for (int c = 0; c < d4; ++c) {
                    const float4 y = kr[c];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int s = min(s0 + 4 * e, nb - 1);
                        const float4 x = *(const float4*)(qs + s * d + 4 * c);
                        dot[e] = fmaf(x.x, y.x, dot[e]); dot[e] = fmaf(x.y, y.y, dot[e]);
                        dot[e] = fmaf(x.z, y.z, dot[e]); dot[e] = fmaf(x.w, y.w, dot[e]);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int s = min(s0 + 4 * e, nb - 1);    // a clamped row repeats a real one: same OR
                    pred |= ((xs[s] - p.sigma * dot[e]) <= p.theta) ? 1 : 0;
                }
            }
        }
        // OR over the four waves: each wave ORs its bit into the block's flag byte
        if (wave == 0 && lane < nJ) flag[J0 - J_lo + lane] = (unsigned char)pred;
        __syncthreads();
        if (wave != 0 && lane < nJ && pred) flag[J0 - J_lo + lane] = 1;   // same value from every writer
    }
    __syncthreads();
    unsigned* bits = a.bits + grp_index(p, sq, b, h, g) * a.nwords;
    for (int w = p.n_init / 32 + tid; w < (Wg + 31) / 32; w += 256) {
        unsigned wd = 0;
#pragma unroll
        for (int hw = 0; hw < 2; ++hw) {
            const int j = 32 * w + 16 * hw;
            if (j >= p.n_init && j < Wg && flag[j / p.bq - J_lo]) wd |= 0xffffu << (16 * hw);
        }
        bits[w] = wd;
    }
}

// ------------------------------------------------------------------ count / scan / fill
// total, stats (nullable): see clear_counters
__global__ void zero_i32_kernel(int* x, long long nelem, long long* total, long long* stats) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0 && total) *total = 0;
    if (i < 4 && stats) stats[i] = 0;
    if (i < nelem) x[i] = 0;
}

// grid (ngrp_max, Hq, B), 256 threads: selected columns of the group per segment of 64 bit words = kSegKeys
// keys from seg_word0 on (block granularity; the stripe mask kernels count what they write themselves)
__global__ __launch_bounds__(256) void count_kernel(SelectArgs a) {
    const KParams& p = a.p;
    const int g = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const Seq sq = seq_of(p, b);
    const int ngrp = (sq.len + p.bq * p.step - 1) / (p.bq * p.step);
    if (g >= ngrp) return;
    const int Wg = window_start(p, g);
    const long long t = grp_index(p, sq, b, h, g);
    const unsigned* bits = a.bits + t * a.nwords;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w_lo = p.n_init / 32, w_hi = Wg > p.n_init ? (Wg + 31) / 32 : w_lo;
    const int w0 = seg_word0(p.n_init);
    for (int seg = wave; w0 + seg * 64 < w_hi; seg += 4) {
        const int w = w0 + seg * 64 + lane;
        int c = (w >= w_lo && w < w_hi) ? __popc(bits[w]) : 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
        if (lane == 0 && c) add_counts(a, t, seg, c);
    }
}

namespace {
__device__ __forceinline__ long long tri(long long m) { return m > 0 ? m * (m + 1) / 2 : 0; }
// pairs of the anchor regions of the rows r0 .. r1-1 of a group with window start W:
// sum over r of min(n_init, r + 1) + max(0, r - W + 1)
__device__ __forceinline__ long long anchor_pairs(long long n_init, long long W, long long r0, long long r1) {
    const long long e = min(r1, n_init);
    long long s = e > r0 ? tri(e) - tri(r0) : 0;            // rows inside the initial tokens see r + 1 of them
    s += n_init * max(0ll, r1 - max(r0, n_init));           // later rows see all of them
    s += tri(r1 - W) - tri(r0 - W);                         // window: W .. r
    return s;
}
}  // namespace

namespace {
__device__ __forceinline__ long long pad_list(int c) { return (c + kIdxPad - 1) / kIdxPad * (long long)kIdxPad; }

// selected columns of group t
__device__ __forceinline__ int group_count(const SelectArgs& a, long long t) {
    if (!a.sum_segs) return a.counts[t];
    const int* sc = a.segcount + t * a.nseg;
    int c = 0;
    if (a.nseg % 4 == 0) {                               // rows of whole 16-byte pieces (the array is aligned)
        for (int s = 0; s < a.nseg; s += 4) {
            const int4 x = *(const int4*)(sc + s);
            c += (x.x + x.y) + (x.z + x.w);
        }
    } else {
        for (int s = 0; s < a.nseg; ++s) c += sc[s];
    }
    return c;
}

// Attended (row, key) pairs of group t with a list of cnt columns: every row's anchor region (closed form) plus the list;
// 0 for a slot past a packed batch's groups.
__device__ __forceinline__ long long group_pairs(const KParams& p, long long t, int cnt) {
    const int span = p.bq * p.step;
    int len = p.N, g = (int)((unsigned)t % (unsigned)p.grp_cap);
    if (p.packed) {
        len = 0;
        for (int b = 0; b < p.B; ++b) {
            const int n = p.cu[b + 1] - p.cu[b], ng = (n + span - 1) / span;
            if (g < ng) { len = n; break; }
            g -= ng;
        }
    }
    if ((long long)g * span >= len) return 0;
    const long long r0 = (long long)g * span, r1 = min(r0 + span, (long long)len);
    return anchor_pairs(p.n_init, window_start(p, g), r0, r1) + (r1 - r0) * cnt;
}

// At most this many selected columns in any word of a segment: a store per column and lane (else a step per pair of words)
constexpr int kFillLaneBits = 12;

// One work-group of NT threads: offsets[t] = sum_{t' < t} roundup64(counts[t']), the counts themselves where they
// are still in segments, the overflow flag, and, with a.stats set, what the prefill reports:
// attended (row, key) pairs = every row's anchor region (closed form per group) plus its group's list, and
// the selected entries.
template <int NT>
__device__ __forceinline__ void scan_groups(const SelectArgs& a) {
    constexpr int NWV = NT / 64;
    __shared__ long long part[3][NWV];
    const KParams& p = a.p;
    const long long T = a.groups_total;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long per = (T + NT - 1) / NT;
    const long long lo = min(T, per * tid), hi = min(T, lo + per);
    long long s = 0, pairs = 0, entries = 0;
    for (long long t = lo; t < hi; ++t) {
        const int cnt = group_count(a, t);
        if (a.sum_segs) a.counts[t] = cnt;
        s += pad_list(cnt);
        if (a.stats) {
            const long long x = group_pairs(p, t, cnt);
            pairs += x;
            if (x) entries += cnt;
        }
    }
    long long x = s;                                     // inclusive scan over the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const long long y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) part[0][wave] = x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        pairs += __shfl_xor(pairs, off, 64);
        entries += __shfl_xor(entries, off, 64);
    }
    if (lane == 0) { part[1][wave] = pairs; part[2][wave] = entries; }
    __syncthreads();
    long long run = x - s;
    for (int w = 0; w < wave; ++w) run += part[0][w];
    for (long long t = lo; t < hi; ++t) {
        a.offsets[t] = run;
        run += pad_list(a.counts[t]);                    // (written by this thread above, where it was)
    }
    if (tid == NT - 1) {
        a.offsets[T] = run;
        if (a.overflow) *a.overflow = run > a.idx_capacity ? 1 : 0;
    }
    if (a.stats && tid < 4) {
        long long sum = 0;
        if (tid < 2)
            for (int w = 0; w < NWV; ++w) sum += part[1 + tid][w];
        a.stats[tid] = sum;
    }
}
}  // namespace

__global__ __launch_bounds__(1024) void scan_kernel(SelectArgs a) { scan_groups<1024>(a); }

// Places: group t's part of the sums that scan_groups takes, one group per thread of the work-groups of the last grid layer.
namespace {
__device__ __forceinline__ void add_sums(const SelectArgs& a) {
    const long long wg = blockIdx.x + (long long)gridDim.x * blockIdx.y, nwg = (long long)gridDim.x * gridDim.y;
    if (wg * 256 >= a.groups_total) return;
    __shared__ long long part[3][4];
    long long pad = 0, pairs = 0, entries = 0;
    for (long long t = wg * 256 + threadIdx.x; t < a.groups_total; t += nwg * 256) {
        const int cnt = group_count(a, t);
        pad += pad_list(cnt);
        if (a.stats) {
            const long long x = group_pairs(a.p, t, cnt);
            pairs += x;
            if (x) entries += cnt;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        pad += __shfl_xor(pad, off, 64);
        pairs += __shfl_xor(pairs, off, 64);
        entries += __shfl_xor(entries, off, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { part[0][wave] = pad; part[1][wave] = pairs; part[2][wave] = entries; }
    __syncthreads();
    if (threadIdx.x < (a.stats ? 3 : 1)) {
        const long long* x = part[threadIdx.x];
        long long* dst = threadIdx.x == 0 ? a.total : a.stats + (threadIdx.x - 1);
        atomicAdd((unsigned long long*)dst, (unsigned long long)(x[0] + x[1] + x[2] + x[3]));
    }
}
}  // namespace

// grid (ngrp_max, ceil(nseg / 4), B*Hq [+ 1]), 256 threads: each wave expands one segment (64 bit words =
// kSegKeys keys) of the group's bit words into its part of the ascending list; the segment counts give its
// position inside the list.  Where the list begins:
//   kFillOffsets  offsets[t], from scan_kernel;
//   kFillScan     no scan_kernel ran; every work-group adds up the lists before its group's itself, and the first
//                 work-group of one more grid layer does scan_kernel's work beside the others.  For few groups that is a
//                 fraction of what the launch costs (5 us); it grows with groups x groups, so the host draws the line;
//   kFillPlaces   the fused call, where nobody reads the lists but stage 3: at the group's own place.  No scan at all; counts
//                 and offsets are written here, the sums (padded entries, statistics) by one more grid layer beside the others.
//                 16384 tokens at step 1 (4096 groups x 8 segments): scan 12.6 us and its launch.
template <int MODE>
__global__ __launch_bounds__(256) void fill_kernel(SelectArgs a) {
    constexpr bool SCAN = MODE == kFillScan, PLACES = MODE == kFillPlaces;
    const KParams& p = a.p;
    if (MODE != kFillOffsets && blockIdx.z == (unsigned)(p.Hq * p.B)) {
        if (PLACES) add_sums(a);
        else if (blockIdx.x == 0 && blockIdx.y == 0) scan_groups<256>(a);
        return;
    }
    const int g = blockIdx.x, h = blockIdx.z % p.Hq, b = blockIdx.z / p.Hq;
    const Seq sq = seq_of(p, b);
    const int ngrp = (sq.len + p.bq * p.step - 1) / (p.bq * p.step);
    if (g >= ngrp) return;
    const int Wg = window_start(p, g);
    const int lane = threadIdx.x & 63;
    const int seg = __builtin_amdgcn_readfirstlane(4 * blockIdx.y + (threadIdx.x >> 6));
    const long long t = grp_index(p, sq, b, h, g);
    if (Wg <= p.n_init) {
        if (PLACES && seg == 0 && lane == 0) { a.counts[t] = 0; a.offsets[t] = 0; }
        return;
    }
    const int w_lo = p.n_init / 32, w_hi = (Wg + 31) / 32;
    const int w0 = seg_word0(p.n_init) + seg * 64;       // the segment's first word
    const int* segc = a.segcount + t * a.nseg;
    long long base = 0;
    if (SCAN) {
        __shared__ long long part[4];
        for (long long u = threadIdx.x; u < t; u += 256) base += pad_list(group_count(a, u));
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) base += __shfl_xor(base, off, 64);
        if (lane == 0) part[threadIdx.x >> 6] = base;
        __syncthreads();
        base = (part[0] + part[1]) + (part[2] + part[3]);
    }
    if (w0 >= w_hi) return;                              // (never the first segment)
    // every load is issued before the first decision, so the wave pays one memory round trip
    const int own = segc[seg];
    int cnt = 0, pre = 0;                                // selected columns of the group, and in earlier segments
    if (MODE == kFillOffsets) base = a.offsets[t];
    for (int s = lane; s < a.nseg; s += 64) {
        const int c = segc[s];
        cnt += c;
        pre += s < seg ? c : 0;
    }
    const int w = w0 + lane;                             // this lane's word
    const unsigned wd = (w >= w_lo && w < w_hi) ? a.bits[t * a.nwords + w] : 0u;
    if (PLACES) {
        const long long span = (long long)p.bq * p.step, c = (long long)p.n_init + p.w;
        base = (p.packed ? (long long)h : (long long)b * p.Hq + h) * a.list_room + padded_places(g, span, c);
        if (p.packed)
            for (int e = 0; e < b; ++e) base += padded_places((p.cu[e + 1] - p.cu[e] + span - 1) / span, span, c);
    }
    const auto add = [](int x, int y) { return x + y; };
    cnt = wave_reduce<1>(cnt, add);
    if (PLACES && seg == 0 && lane == 0) { a.counts[t] = cnt; a.offsets[t] = base; }
    if (own == 0) return;                                // the group's last entry is never in such a segment
    pre = wave_reduce<1>(pre, add);
    long long pos = base + pre;
    const unsigned long long nzw = __ballot(wd != 0u);
    const int most = wave_reduce<1>((int)__popc(wd), [](int x, int y) { return max(x, y); });
    if (most <= kFillLaneBits) {
        // few columns per word: every lane stores its own word's, one after the other.  Its first entry comes after the
        // columns of the lower lanes, whose numbers are added up bit by bit.
        const unsigned pc = __popc(wd);
        unsigned mine = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {                    // pc <= kFillLaneBits < 16
            const unsigned long long m = __ballot((pc >> k) & 1u);
            mine += __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0)) << k;
        }
        unsigned rest = wd;
        long long dst = pos + mine;
        for (int k = 0; k < most; ++k) {
            if (rest) {
                if (dst < a.idx_capacity) a.idx[dst] = w * 32 + __builtin_ctz(rest);
                rest &= rest - 1;
                ++dst;
            }
        }
    } else {
        // two words per step: lanes 0..31 test word 2 i, lanes 32..63 word 2 i + 1 (coalesced stores); only the word
        // pairs that hold a selected column are visited (scalar loop over a bit mask)
        const int bit = lane & 31, half = lane >> 5;
        unsigned long long pairs = (nzw | (nzw >> 1)) & 0x5555555555555555ull;
        while (pairs) {
            const int i = __builtin_ctzll(pairs) >> 1;
            pairs &= pairs - 1;
            const unsigned first = __builtin_amdgcn_readlane(wd, 2 * i), second = __builtin_amdgcn_readlane(wd, 2 * i + 1);
            const unsigned mine = half ? second : first;
            const bool on = (mine >> bit) & 1u;
            const long long dst = pos + __popc(mine & ((1u << bit) - 1u)) + (half ? __popc(first) : 0);
            if (on && dst < a.idx_capacity) a.idx[dst] = (w0 + 2 * i + half) * 32 + bit;
            pos += __popc(first) + __popc(second);
        }
    }
    // the wave that wrote the group's last entry pads the list to the next multiple of 64 with it
    if (pre + own == cnt) {
        const int top = 63 - __builtin_clzll(nzw);       // own > 0: some word is non-zero
        const unsigned lastw = __builtin_amdgcn_readlane(wd, top);
        const int last_key = (w0 + top) * 32 + 31 - __clz(lastw);
        const int padded = (cnt + kIdxPad - 1) / kIdxPad * kIdxPad;
        for (int e = cnt + lane; e < padded; e += 64)
            if (base + e < a.idx_capacity) a.idx[base + e] = last_key;
    }
}

int launch_fill(const SelectArgs& a, FillMode mode, hipStream_t st) {
    const dim3 grid((unsigned)a.p.ngrp_max, (unsigned)((a.nseg + 3) / 4),
                    (unsigned)(a.p.Hq * a.p.B + (mode == kFillOffsets ? 0 : 1)));
    switch (mode) {
        case kFillScan: return (int)launch_kernel(fill_kernel<kFillScan>, grid, dim3(256), 0, st, a);
        case kFillPlaces: return (int)launch_kernel(fill_kernel<kFillPlaces>, grid, dim3(256), 0, st, a);
        default: return (int)launch_kernel(fill_kernel<kFillOffsets>, grid, dim3(256), 0, st, a);
    }
}

}  // namespace aa
