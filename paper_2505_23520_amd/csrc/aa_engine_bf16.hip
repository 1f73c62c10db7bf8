// bf16 tile engine: one online-softmax (flash-style) kernel that serves
//   * stage 1, anchor computation          (Sec. 3.1 Eq. 1, Algorithm 1),
//   * stage 3, gathered sparse attention   (Sec. 3.3 Eq. 3-5, Algorithm 3),
//   * the dense causal comparator
// of arXiv 2505.23520 on gfx950.  The three differ only in which K/V rows feed
// the tiles (a contiguous masked range or the rows a selected-column list names)
// and in what is read before / written after the loop.
//
// Shape of the computation (d = 128, b_q = 128, bf16 in, fp32 accumulate):
//   work-group = one query block = 4 waves x 32 query rows, three work-groups per CU
//   (three waves per SIMD, so one wave's softmax and LDS latency overlap the others' MFMAs);
//   K/V tile   = 64 keys, two K stages and one V stage in LDS, filled by 16-byte direct-to-LDS
//   buffer loads (no staging registers; a gathered row and a contiguous row cost the same);
//   S^T = K Q^T  with v_mfma_f32_32x32x16_bf16 (keys are the M dimension, query
//   rows the N dimension, so one lane owns one query row and the row max / sum
//   are in-lane reductions; the wave's halves meet only when a reference is raised);
//   O^T = V^T P^T with the same instruction; V stays row-major in LDS and its operand
//   is read with the transposing LDS load ds_read_b64_tr_b16.
// LDS layout of a tile: a direct-to-LDS load writes the 64 lanes' 16 bytes to consecutive
// addresses, i.e. 1 KB = four 256-byte rows per instruction ("group").  Key kk of the tile
// sits in group kk % 16, row kk / 16; groups are padded (K: 16 B, V: 64 B) so that the 16
// lanes of an operand read fall into different banks.
// The running reference m of exp(s - m) is only raised when a row's maximum
// exceeds it by more than 2^8; the accumulators are then rescaled, otherwise they are left
// alone.  The true row maximum, which is the anchor that stage 1 exports, is tracked separately.
//
// What bounds it: a wave's own chain per tile (load issue, 16 score MFMAs, softmax, 16 P V MFMAs,
// two barriers) is about four times as long as its 1024 MFMA cycles, so the matrix pipe needs as many waves per
// SIMD as fit to stay busy.  Three fit if a wave takes at most 168 registers and a work-group a
// third of the LDS.  V therefore has one stage: V tile t is issued when tile t - 1 has been
// consumed and is awaited after the scores and softmax of tile t, behind which its latency hides
// (K tile t + 1 has the whole of tile t).  At 168 registers the compiler left alone issues every LDS operand
// read right before its MFMA, so the read-ahead is written out and pinned with scheduling fences,
// and no load or wait stands under a condition (a path on which fewer loads are outstanding would
// turn the waits into vmcnt(0)).  Nothing may be spilled: a reload is a vector-memory load, too.
// Measured, 131072 tokens x 32 heads, step 16: anchor computation 3.10 -> 2.71 ms (the two-per-CU form
// with two V stages before), matrix pipe 50 -> 65 % busy; the engine clock falls from 1.70 to 1.57 GHz
// at the same time (the card's power limit), which is why the time gains less than the cycles.  Of this the third
// wave alone gave 5 %, the pinned order 4 %.  Inside the tile loop the pipe is 77 % busy (3970 cycles per
// tile and three waves); the rest is a work-group's prologue (5700 cycles), epilogue (6000, of which what stage 2 needs takes 3800)
// and replacement.
// Several blocks per work-group in one loop, which saves the replacement, was 3 to 11 % slower.
#include "aa_engine_bf16_common.h"
#include "aa_items.h"
#include "aa_pool.h"
#include "aa_rows.h"

#include <type_traits>

namespace aa {

using namespace eng;

namespace {
// Work-group barrier that leaves vector-memory operations in flight.  LDS operand reads before it
// have been consumed by their MFMAs and the tile loads it publishes were awaited; the fences only
// keep the compiler from moving work across it.
__device__ __forceinline__ void bare_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// What stage 2 needs of a query block, from the work-group that holds it: the pooled query (Algorithm 2, avgpool of Q) from the
// fragments in registers, the key norms of the block, the pooled anchor (mean of M over its rows).  ms: M of the
// lane's row.  EARLY: the keys are requested ahead of the pooling (32 registers more at its peak).
template <bool EARLY>
__device__ __forceinline__ void stage2_exports(const EngineArgs& a, const Seq& sq, const Work& wk, int hk, const bf16x8 (&qf)[8],
                                               float (*qpart)[128], float* red, float* knorm, int row0, int rlast, int wave,
                                               int lane, bool rok, float ms) {
    const KParams& p = a.p;
    const int tid = 64 * wave + lane, n = lane & 31, hf = lane >> 5;
    // the key norms of block i of a KV head fall to one of the head's query heads, in turn (its rows were the
    // last tiles of the loop)
    const bool norms = a.kmax_blk && wk.h - hk * p.grp == wk.i - (int)p.by_grp.div(wk.i) * p.grp;
    KeyNorm kn;
    auto load_keys = [&]() {
        if (norms)
            kn.load((const unsigned short*)a.k + tok_offset(p, p.ks, sq, wk.b, hk, 0), p.ks[2], row0, rlast + 1, tid);
    };
    if (EARLY) load_keys();
    if (a.qp_hi) {
        float s0, s1;
        pool_wave_columns(qf, n, s0, s1);
        pool_block_put(qpart, wave, n, hf, s0, s1);
    }
    if (!EARLY) load_keys();
    if (a.xa) {
        const float red_m = wave_reduce<1>((rok && hf == 0) ? ms : 0.f, [](float x, float y) { return x + y; });
        if (lane == 0) red[wave] = red_m;
    }
    if (norms) {
        const float big = kn.wave_max();
        if (lane == 0) knorm[wave] = big;
    }
    __syncthreads();                                 // one barrier, then a wave for each of the three
    const int nrows = rlast - row0 + 1;
    const long long bi = blk_index(p, sq, wk.b, wk.h, wk.i);
    if (wave == 0 && a.qp_hi) pool_block_write(qpart, lane, nrows, bi, a.qp_hi, a.qp_lo, a.qlo_norm);
    if (wave == 1 && lane == 0 && a.xa) a.xa[bi] = (red[0] + red[1] + red[2] + red[3]) / (float)nrows;
    if (wave == 2 && lane == 0 && norms) a.kmax_blk[kblk_index(p, sq, wk.b, hk, wk.i)] = KeyNorm::block(knorm);
}
}  // namespace

// FLAGS (a combination of kEng*) is a compile-time parameter: every mode gets its own code without
// the other modes' branches, registers and, above all, merged control-flow paths (where paths with
// different numbers of outstanding loads meet, the compiler's waits assume the shortest).
// QLDS: the query rows come through LDS (see request_q).
template <int FLAGS, bool QLDS>
__global__ __launch_bounds__(256, 3) void engine_bf16_kernel(EngineArgs a) {
    constexpr int flags = FLAGS;
    constexpr int NW = 4;                            // waves per work-group
    static_assert(NW == 4, "the loader deals four groups of a tile to every wave");
    // one LDS object per stage, so that the compiler can tell that the asynchronous loads into
    // one stage do not alias the operand reads from the others
    __shared__ __attribute__((aligned(16))) char Ks0[KBYTES], Ks1[KBYTES], Vs0[VBYTES];
    __shared__ float red[NW], knorm[NW];
    __shared__ float qpart[(FLAGS & kEngStoreState) ? 4 : 1][128];   // pooled-query partial sums (stage 1)
    const KParams& p = a.p;
    int tid = threadIdx.x;
    int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it scalar
    int n = lane & 31, hf = lane >> 5;

    // (calls of few blocks: dense attention of 150 tokens 7.73 -> 7.63 us, the prefill 8.73 -> 8.56; where the chip is full, a
    // work-group finds the lines in the cache)
    if (!QLDS) touch_args(a);
    if (flags & kEngStoreState) {
        store_dense_stats(a);
        if (a.kmax_blk)
            clear_counters(a.zero_counts, a.groups_total, a.zero_seg, a.nseg, a.zero_total, a.zero_stats, blockIdx.x * 256ll + tid, gridDim.x * 256ll);
    }
    if ((flags & kEngList) && !engine_selected(a)) return;
    const Work wk = decode_work(p, p.nblk_max, p.by_pair, blockIdx.x);
    const Seq sq = seq_of(p, wk.b);
    const int row0 = wk.i * BQ;
    if (row0 >= sq.len) return;
    // Three waves share a SIMD (one from each resident work-group).  A wave raises its issue priority
    // for its MFMA blocks and drops it for its softmax, so a wave with matrix work wins over
    // siblings that are in their vector-ALU part, and they do not settle into lockstep.
    __builtin_amdgcn_s_setprio(2);
    const int hk = (int)p.by_grp.div(wk.h);
    const int g = (int)p.by_step.div(wk.i);
    const bool direct = a.direct && window_start(p, g) <= p.n_init;   // no candidates: stage 1 finishes the rows
    if ((flags & kEngLoadState) && direct) return;
    const int rw = row0 + 32 * wave;                 // first row of this wave
    int r = rw + n;                                  // this lane's query row
    bool rok = r < sq.len;
    const int rlast = min(row0 + BQ, sq.len) - 1;    // last row of the block

    // ---- tile sequence: [range 1: initial tokens][range 2: window .. diagonal][list chunks]
    int W = 0, ninit = 0, T1 = 0, t2s = 0, nA = 0;
    if (flags & kEngAnchorRegion) {
        if (!(flags & kEngDense)) { W = window_start(p, g); ninit = p.n_init; }
        const int e1 = min(ninit, rlast + 1);
        T1 = (e1 + TK - 1) / TK;
        t2s = max(T1, W / TK);
        const int T2 = rlast / TK + 1;
        nA = T1 + max(0, T2 - t2s);
    }
    int cnt = 0;
    long long lbase = 0;
    if (flags & kEngList) {
        const long long t = grp_index(p, sq, wk.b, wk.h, g);
        cnt = a.counts[t];
        lbase = a.offsets[t];
    }
    const int nL = (cnt + TK - 1) / TK;

    // K / V rows of this KV head are fetched with raw buffer loads: scalar base, 32-bit byte offsets
    const unsigned short* kb_ = (const unsigned short*)a.k + tok_offset(p, p.ks, sq, wk.b, hk, 0);
    const unsigned short* vb_ = (const unsigned short*)a.v + tok_offset(p, p.vs, sq, wk.b, hk, 0);
    const unsigned kstb = (unsigned)p.ks[2] * 2u, vstb = (unsigned)p.vs[2] * 2u;   // token strides in bytes
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)kb_, 0, (int)((unsigned)(sq.len - 1) * kstb + 2u * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)vb_, 0, (int)((unsigned)(sq.len - 1) * vstb + 2u * D), 0x00020000);

    // ---- loader role of this wave: GPW = 16 / NW groups of every tile.  In the load of group gi
    // lane l fetches the 16-byte chunk l % 16 of key 16 (l / 16) + gi of the tile, so each lane deals
    // with the GPW consecutive keys 16 (l / 16) + GPW wave + j.
    constexpr int GPW = 16 / NW;
    const int lch = lane & 15;
    const int kq0 = 16 * (lane >> 4) + GPW * wave;   // first of this lane's keys inside the tile

    auto tile_start = [&](int t) -> int {            // first key of contiguous tile t (t < nA)
        return TK * (t < T1 ? t : t2s + (t - T1));
    };
    // Keys of a list tile come from the index list.  Tile c's are fetched into kidx0 / kidx1 (by the
    // parity of c) two steps ahead: its K rows are loaded in step c - 1, its V rows in step c.
    // Nothing else ever writes these registers: a vector-ALU write to registers that may still
    // be the target of an outstanding load makes the compiler wait for every outstanding load,
    // the asynchronous tile loads included.  Keys of a contiguous tile are plain arithmetic.
    intx4 kidx0 = {0, 0, 0, 0}, kidx1 = {0, 0, 0, 0};
    auto idx_prefetch = [&](int c, intx4& kidx) {
        if (c < nL) kidx = *(const intx4*)(a.idx + lbase + (long long)c * TK + kq0);
    };
    // asynchronous: completion is awaited by wait_vmem()
    // (no branch: the byte offsets of a contiguous tile are clamped to the sequence's last row)
    // LIST (here and below): tile t of the list, else contiguous tile t
    // (contiguous and list tiles in one kernel: the lane's 16-byte piece is added after the clamp, which leaves the limits in
    // scalar registers; the other modes need no such addition)
    constexpr bool mixed = (FLAGS & kEngList) && (FLAGS & kEngAnchorRegion);
    const unsigned piece = 16u * lch, cpiece = mixed ? 0 : piece;
    const unsigned klane = lane_row_offset(kq0, sq.len, kstb, mixed ? 0 : lch);
    const unsigned vlane = lane_row_offset(kq0, sq.len, vstb, mixed ? 0 : lch);
    const unsigned klast = (unsigned)(sq.len - 1) * kstb + cpiece, vlast = (unsigned)(sq.len - 1) * vstb + cpiece;
    auto rows_load = [&](auto list, int t, const __amdgpu_buffer_rsrc_t& rs, unsigned stb, unsigned lane0, unsigned last,
                         char* dst, int pitch, const intx4& kidx) {
#pragma unroll
        for (int j = 0; j < GPW; ++j) {
            unsigned off;
            if (decltype(list)::value) off = (unsigned)kidx[j] * stb + piece;
            else off = clamped_row_offset(lane0, tile_row_offset(tile_start(t), j, stb), last) + (mixed ? piece : 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(dst + j * pitch), 16, (int)off, 0, 0, 0);
        }
    };
    auto k_load = [&](auto list, int t, char* Kb, const intx4& kidx) {
        rows_load(list, t, krs, kstb, klane, klast, Kb + GPW * wave * KGRP, KGRP, kidx);
    };
    auto v_load = [&](auto list, int t, const intx4& kidx) {
        rows_load(list, t, vrs, vstb, vlane, vlast, Vs0 + GPW * wave * VGRP, VGRP, kidx);
    };

    // The first list indices are requested before everything else: the first tile's loads need them,
    // and only them, so they go out while the Q fragments and the cached state are still on their way
    // (waits are in issue order: behind those loads the indices would arrive last).
    idx_prefetch(0, kidx0);

    constexpr std::integral_constant<bool, false> contiguous{};
    constexpr std::integral_constant<bool, true> listed{};
    // ---- Q fragments (B operand of S^T = K Q^T): lane (n, hf) holds Q[row][16 ks + 8 hf .. +8)
    // (through the stages that the first tiles do not use: Ks1 and Vs0)
    static_assert(KBYTES >= 2 * kQStageBytes && VBYTES >= 2 * kQStageBytes, "two waves' query rows per stage");
    char* const qstg = (wave < 2 ? Ks1 : Vs0) + (wave & 1) * kQStageBytes;
    bf16x8 qf[8];
    if (QLDS) request_q(a, sq, wk.b, wk.h, rw, lane, qstg);
    else load_q_fragments(qf, a, sq, wk.b, wk.h, r, rok, 0, hf);

    // ---- pipeline prologue: the first K tile goes out ahead of the cached state, which is not needed
    // before the first P V block
    if (flags & kEngAnchorRegion) k_load(contiguous, 0, Ks0, kidx0);     // (a block has its diagonal tile)
    else if (nL > 0) k_load(listed, 0, Ks0, kidx0);
    if (!(flags & kEngAnchorRegion)) idx_prefetch(1, kidx1);
    __builtin_amdgcn_sched_barrier(0);

    // ---- running state (see load_state)
    const float c2 = p.sigma * 1.4426950408889634f;  // exp(sigma*x) = exp2(c2*x)
    const float rescale_gap = rescale_limit(c2);
    const long long tile = acc_tile(p, sq, wk.b, wk.h, wk.i, wave);
    float mref, mtrue, l;
    floatx16 o[4];
    if (flags & kEngLoadState) load_state(a, row_index(p, sq, wk.b, wk.h, rok ? r : row0), tile, lane, hf, mref, mtrue, l, o);
    else init_state(mref, mtrue, l, o);
    __builtin_amdgcn_sched_barrier(0);
    // K tile 0 is there; the 16 loads of the cached accumulators are younger and may still be on their way
    if (flags & kEngLoadState) __builtin_amdgcn_s_waitcnt(0x4F70); else wait_vmem();
    if (QLDS) {
        read_q(qf, qstg, rok, n, hf);
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): read before the barrier, behind which V tile 0 takes the place
    }
    bare_barrier();

    // operand addresses inside a stage (bytes): K row of key 32 kb + n; V chunk read by this lane
    // in the transposing load (lane 16 G + s: key offset s / 4, 8-byte piece s % 4 of d-half G % 2)
    const int koff = (n & 15) * KGRP + (n >> 4) * 256 + 16 * hf;
    const int ls = lane & 15, lg = lane >> 4;
    const int voff = (4 * hf + (ls >> 2)) * VGRP + 32 * (lg & 1) + 8 * (ls & 3);

    auto tile_step = [&](auto list, int t, int nT, const char* Kcur, char* Knext, intx4& kcur, intx4& knext)
                         __attribute__((always_inline)) {
        constexpr bool LIST = decltype(list)::value;
        v_load(list, t, kcur);
        if (LIST) idx_prefetch(t + 2, kcur);
        __builtin_amdgcn_sched_barrier(0);           // the wait below counts on this issue order
        // the next K tile (past the end the last one again, into a stage nobody reads): gathered rows go out now,
        // contiguous ones, which L2 serves, after the softmax, out of the way of the V tile (-1 %; gathered rows
        // issued there cost 29 %)
        if (LIST) k_load(list, min(t + 1, nT - 1), Knext, knext);
        const char* Kb = Kcur + koff;
        const char* Vb = Vs0 + voff;

        // S^T = K Q^T : s[kb], 32 keys x 32 rows each.  Masks (tiles that touch a region
        // boundary, the diagonal or a list tail) enter as the initial accumulator: 0 for a
        // visible (key, row) pair, -inf otherwise; the common unmasked tile starts from literal 0.
        const int t0 = LIST ? 0 : tile_start(t);
        const bool masked = LIST ? t == nT - 1 && (cnt & (TK - 1))
                                 : !((t0 + TK - 1 <= rw) && (t0 + TK <= ninit || t0 >= W));
        // a contiguous tile that starts beyond this wave's last row is hidden from all its rows
        // (the work-group still needs it for its later rows): nothing to compute
        const bool on = LIST || t0 <= rw + 31;
        bf16x8 pf[2][2];  // [kb][s16]
        if (on) {
            floatx16 s[2];
            // K operands run four MFMAs ahead of their use; the order is pinned with scheduling fences
            // (left alone, the compiler issues each read right before its MFMA)
            {
                bf16x8 kf[16];
                auto read_k = [&](int i) { kf[i] = *(const bf16x8*)(Kb + 512 * (i & 1) + 32 * (i >> 1)); };
#pragma unroll
                for (int i = 0; i < 4; ++i) read_k(i);
                __builtin_amdgcn_sched_barrier(0);
                if (__builtin_expect(!masked, 1)) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
                        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[0], kZero16, 0, 0, 0);
                } else {
                    // key j = t0 + jl is visible to row r iff j <= r and (j < ninit or j >= W);
                    // entry jl of the last list chunk is real iff jl < rem
                    // (jl = 32 kb + 8 (v / 4) + 4 hf + v % 4: the lane's part is taken off the limits instead)
                    // (with the lane opaque, the 32 comparisons are not hoisted out of the loop either)
                    const int ln = counted_lane(), h4 = 4 * (ln >> 5);
                    const int jr = (LIST ? cnt - t * TK - 1 : rw - t0 + (ln & 31)) - h4;
                    const int jn = ninit - t0 - h4, jw = W - t0 - h4;
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) {
                        floatx16 bias;
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int jc = 32 * kb + 8 * (v >> 2) + (v & 3);
                            bool ok = jc <= jr;
                            if (!LIST) ok = ok & ((jc < jn) | (jc >= jw));
                            bias[v] = ok ? 0.f : -INFINITY;
                        }
                        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[0], bias, 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                read_k(4); read_k(5);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 2; i < 16; ++i) {         // MFMA i: ks = i / 2, kb = i % 2
                    s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[i >> 1], s[i & 1], 0, 0, 0);
                    if (i + 4 < 16) read_k(i + 4);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
            softmax_tile(s, pf, c2, rescale_gap, mref, mtrue, l, o);
            __builtin_amdgcn_s_setprio(2);
        }
        if (!LIST) {
            __builtin_amdgcn_sched_barrier(0);
            k_load(list, min(t + 1, nT - 1), Knext, knext);
            __builtin_amdgcn_sched_barrier(0);
        }
        // V tile t has landed (vmcnt(4): the four loads of the next K tile are younger)
        __builtin_amdgcn_s_waitcnt(0x0F74);
        bare_barrier();
        if (on) {
        // O^T += V^T P^T, V operands four MFMAs ahead
        shortx4 vlo[16], vhi[16];
        auto read_v = [&](int i) {                 // operand of MFMA i: sg = i / 4, db = i % 4
            // keys 16 sg + 8 rd + 4 hf + (0..3) live in groups 8 rd + 4 hf + (0..3), row sg
            vlo[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) shortx4*)(Vb + (i >> 2) * 256 + 64 * (i & 3)));
            vhi[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) shortx4*)(Vb + 8 * VGRP + (i >> 2) * 256 + 64 * (i & 3)));
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) read_v(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const shortx8 vv = __builtin_shufflevector(vlo[i], vhi[i], 0, 1, 2, 3, 4, 5, 6, 7);
            const int sg = i >> 2, db = i & 3;
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), pf[sg >> 1][sg & 1],
                                                             o[db], 0, 0, 0);
            if (i + 4 < 16) read_v(i + 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        }
        wait_vmem();                                 // next K tile has landed in LDS
        bare_barrier();
    };
    auto tile_loop = [&](auto list, int nT) __attribute__((always_inline)) {
        for (int t = 0; t < nT; t += 2) {
            tile_step(list, t, nT, Ks0, Ks1, kidx0, kidx1);
            if (t + 1 < nT) tile_step(list, t + 1, nT, Ks1, Ks0, kidx1, kidx0);
        }
    };
    if (flags & kEngAnchorRegion) tile_loop(contiguous, nA);
    if (mixed) {
        // Anchor region, then list: a loop for each (in one loop for both every list tile pays for the choice between the two).
        // In between the state is put in the form in which stage 1 caches it, so the result is the same with and
        // without a cached state, bit for bit.
        if (nL > 0) k_load(listed, 0, Ks0, kidx0);
        idx_prefetch(1, kidx1);                      // (its registers are needed in the first loop)
        float lt = row_sum(l);
        const float ms = rebase_state(a, c2, mref, mtrue, lt, o);
        mref = mtrue = ms / p.sigma;
        l = hf == 0 ? lt : 0.f;
        wait_vmem();
        bare_barrier();
    }
    if (flags & kEngList) tile_loop(listed, nL);

    // ---- epilogue
    // The tile stages are free now (every wave has passed the barrier that ends the last tile):
    // each wave takes one of them as a private staging area for coalesced stores.  LDS operations
    // of one wave execute in order, so no barrier separates its writes from its reads.
    char* const stg = wave == 0 ? Ks0 : wave == 1 ? Ks1 : Vs0 + (wave - 2) * kOutStageBytes;
    const int wave_rows = min(32, sq.len - rw);      // rows of this wave inside the sequence (<= 0: none)
    float lt = row_sum(l);                           // row sum relative to mref
    lane = counted_lane();                           // (no lane's value but addresses lives through the loop)
    tid = 64 * wave + lane;
    n = lane & 31; hf = lane >> 5;
    r = rw + n;
    rok = r < sq.len;
    const long long ri = row_index(p, sq, wk.b, wk.h, rok ? r : row0);
    if (flags & kEngStoreState) {
        const float ms = rebase_state(a, c2, mref, mtrue, lt, o);
        // (the state goes out last: the barriers in between would wait for its stores to drain)
        if (a.xa) stage2_exports<false>(a, sq, wk, hk, qf, qpart, red, knorm, row0, rlast, wave, lane, rok, ms);
        if (!direct) {
            store_state(a, ri, tile, rok, wave_rows > 0, lane, hf, ms, lt, o);
        } else if (wave_rows > 0) {
            // what stage 3 makes of a cached state and an empty list, bit for bit
            store_out(a, stg, tok_offset(p, p.os, sq, wk.b, wk.h, rw), wave_rows, lane, n, hf, lt, o);
            if (rok && a.lse && hf == 0) a.lse[ri] = ms / p.sigma * p.sigma + __logf(lt);
        }
    }
    if ((flags & kEngStoreOut) && wave_rows > 0) {
        store_out(a, stg, tok_offset(p, p.os, sq, wk.b, wk.h, rw), wave_rows, lane, n, hf, lt, o);
        if (rok && a.lse && hf == 0) a.lse[ri] = mref * p.sigma + __logf(lt);
    }
}

// Stage 1 for a stage 3 that attends the anchor region itself: the row maxima, of which only the pooled anchor is kept, and
// the other things that stage 2 needs.  The scores are those of engine_bf16_kernel, instruction by instruction, so the maxima
// are the same bits.  Bound: a block is six tiles at step 1, 3000 matrix cycles a wave, between the latencies of its query rows
// and of its exports; so a work-group walks every gridDim.x-th block (all blocks cost the same) and requests the next block's
// query rows ahead of the exports of this one.  16384 tokens, 32 heads: 78 us with a work-group per block and exports through LDS, 70
// so (the walk alone makes the whole call 2 % faster); its compulsory bytes take 34 us.
__global__ __launch_bounds__(256, 3) void anchor_max_bf16_kernel(EngineArgs a, unsigned total) {
    __shared__ __attribute__((aligned(16))) char Ks0[KBYTES], Ks1[KBYTES];
    __shared__ float red[4], knorm[4], qpart[4][128];
    const KParams& p = a.p;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hf = lane >> 5;
    if (a.kmax_blk)
        clear_counters(a.zero_counts, a.groups_total, a.zero_seg, a.nseg, a.zero_total, a.zero_stats, blockIdx.x * 256ll + tid, gridDim.x * 256ll);
    const int koff = (n & 15) * KGRP + (n >> 4) * 256 + 16 * hf;
    const int lch = lane & 15, kq0 = 16 * (lane >> 4) + 4 * wave;
    const unsigned kstb = (unsigned)p.ks[2] * 2u;
    const int ninit = p.n_init;

    // the block that work item `id` stands for, if it exists
    struct Block { Work wk; Seq sq; int row0, hk; };
    auto block_of = [&](unsigned id) -> Block {
        Block x;
        x.wk = decode_work(p, p.nblk_max, p.by_pair, id);
        x.sq = seq_of(p, x.wk.b);
        x.row0 = x.wk.i * BQ;
        x.hk = (int)p.by_grp.div(x.wk.h);
        return x;
    };
    auto next_block = [&](unsigned& id, Block& x) -> bool {
        return next_item(id, gridDim.x, total, x, block_of, [](const Block& y) { return y.row0 < y.sq.len; });
    };
    auto load_q = [&](bf16x8 (&qf)[8], const Block& x) {
        const int r = x.row0 + 32 * wave + n;
        load_q_fragments(qf, a, x.sq, x.wk.b, x.wk.h, r, r < x.sq.len, 0, hf);
    };

    unsigned id = blockIdx.x;
    Block cur;
    if (!next_block(id, cur)) return;
    bf16x8 qf[8];
    load_q(qf, cur);
    for (;;) {
        const Seq& sq = cur.sq;
        const int row0 = cur.row0, rw = row0 + 32 * wave;
        const int rlast = min(row0 + BQ, sq.len) - 1;
        const int W = window_start(p, (int)p.by_step.div(cur.wk.i));
        const int T1 = (min(ninit, rlast + 1) + TK - 1) / TK, t2s = max(T1, W / TK);
        const int nA = a.xa ? T1 + max(0, rlast / TK + 1 - t2s) : 0;     // (xa null: the anchors are not compared with)
        auto tile_start = [&](int t) -> int { return TK * (t < T1 ? t : t2s + (t - T1)); };
        const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)((const unsigned short*)a.k + tok_offset(p, p.ks, sq, cur.wk.b, cur.hk, 0)), 0,
            (int)((unsigned)(sq.len - 1) * kstb + 2u * D), 0x00020000);
        const unsigned klane = lane_row_offset(kq0, sq.len, kstb, lch), klast = (unsigned)(sq.len - 1) * kstb + 16u * lch;
        auto k_load = [&](int t, char* Kb) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, (lds_void*)(Kb + (4 * wave + j) * KGRP), 16,
                                                         (int)clamped_row_offset(klane, tile_row_offset(tile_start(t), j, kstb), klast),
                                                         0, 0, 0);
        };
        if (nA > 0) k_load(0, Ks0);                  // (every wave has passed a barrier since the last read of this stage)
        float mtrue = -INFINITY;
        auto tile_step = [&](int t, const char* Kcur, char* Kld) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vmem();                             // tile t is there
            bare_barrier();                          // everywhere, and the stage of tile t - 1 has been read
            k_load(min(t + 1, nA - 1), Kld);
            __builtin_amdgcn_sched_barrier(0);
            const char* Kb = Kcur + koff;
            const int t0 = tile_start(t);
            if (t0 > rw + 31) return;                // hidden from all rows of the wave
            floatx16 s[2];
            bf16x8 kf[16];
            auto read_k = [&](int i) { kf[i] = *(const bf16x8*)(Kb + 512 * (i & 1) + 32 * (i >> 1)); };
#pragma unroll
            for (int i = 0; i < 6; ++i) read_k(i);
            if (__builtin_expect((t0 + TK - 1 <= rw) && (t0 + TK <= ninit || t0 >= W), 1)) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[0], kZero16, 0, 0, 0);
            } else {
                const int ln = counted_lane(), h4 = 4 * (ln >> 5);
                const int jr = rw - t0 + (ln & 31) - h4, jn = ninit - t0 - h4, jw = W - t0 - h4;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    floatx16 bias;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int jc = 32 * kb + 8 * (v >> 2) + (v & 3);
                        bias[v] = ((jc <= jr) & ((jc < jn) | (jc >= jw))) ? 0.f : -INFINITY;
                    }
                    s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[0], bias, 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 2; i < 16; ++i) {
                s[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[i >> 1], s[i & 1], 0, 0, 0);
                if (i + 4 < 16) read_k(i + 4);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) mtrue = fmaxf(fmaxf(mtrue, s[0][v]), s[1][v]);
        };
#pragma unroll 1
        for (int t = 0; t < nA; t += 2) {
            tile_step(t, Ks0, Ks1);
            if (t + 1 < nA) tile_step(t + 1, Ks1, Ks0);
        }
        wait_vmem();
        id += gridDim.x;
        Block nx = cur;                              // (none left: this block's rows again)
        const bool more = next_block(id, nx);
        bf16x8 qn[8];
        load_q(qn, nx);
        float ma, mb;
        both_halves(mtrue, ma, mb);
        stage2_exports<false>(a, sq, cur.wk, cur.hk, qf, qpart, red, knorm, row0, rlast, wave, lane, rw + n < sq.len,
                             fmaxf(ma, mb) * p.sigma);
        if (!more) return;
        cur = nx;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = qn[ks];
        __syncthreads();                             // red, knorm and qpart have been read
    }
}

// Stage 3 recomputing the anchor region: two work-groups per CU instead of three, by 8 KB of unused LDS, where the query blocks
// of the call fill two slots per CU once to one and three quarters times and a group is long (its blocks then have chains of
// uneven length, and the last third of a full chip waits for the longest).  32 heads, three / two per CU, us: step 16, 2500 tokens
// (640 blocks) 51.3 / 51.2, 3000 (768) 63.4 / 60.3, 3500 (896) 70.9 / 69.8, 5000 (1280) 103.2 / 106.0, 8192 (2048) 171.9 /
// 182.3; step 8, 3000 tokens 51.1 / 48.8, 3500 54.4 / 54.0; step 4, 2500 34.4 / 33.3, 4096 48.6 / 50.7; step 2, 2500 29.5 / 32.7;
// every column selected, 2500 64.7 / 62.7; 8 heads, 11000 tokens (688) 85.3 / 78.7.  Towards 1024 blocks it depends on the call:
// 4096 tokens 90.5 / 90.0, every column selected 133.7 / 145.9, two sequences of 2000 82.1 / 79.7, 8 heads, 16000 tokens 106.3 /
// 114.0.  (16 / 2 heads, 5000 tokens (640) 65.6 / 69.5.)  Up to 512 blocks there is no third either way.
static size_t recompute_extra_lds(const KParams& p) {
    const long long blocks = (p.total + BQ - 1) / BQ * p.Hq;
    return p.step >= 8 && blocks > 512 && blocks <= 896 ? 8192 : 0;
}

int launch_engine_bf16(const EngineArgs& ea, unsigned grid, hipStream_t st) {
    switch (ea.flags * 2 + q_through_lds(ea.p)) {
#define AA_ENGINE_CASE(F, lds)                                                                                                 \
    case (F) * 2: return (int)launch_kernel(engine_bf16_kernel<(F), false>, dim3(grid), dim3(256), lds, st, ea);               \
    case (F) * 2 + 1: return (int)launch_kernel(engine_bf16_kernel<(F), true>, dim3(grid), dim3(256), lds, st, ea);
    AA_ENGINE_CASE(kEngAnchorRegion | kEngStoreState, 0)              // stage 1
    AA_ENGINE_CASE(kEngList | kEngLoadState | kEngStoreOut, 0)         // stage 3 from the cached state
    AA_ENGINE_CASE(kEngList | kEngAnchorRegion | kEngStoreOut, recompute_extra_lds(ea.p))   // stage 3 recomputing the anchor region
    AA_ENGINE_CASE(kEngAnchorRegion | kEngDense | kEngStoreOut, 0)     // dense causal attention
#undef AA_ENGINE_CASE
    default: return -1;
    }
}

int launch_anchor_max_bf16(const EngineArgs& ea, unsigned grid, hipStream_t st) {
    // three work-groups per CU, a multiple of 8 (decode_work's XCD of a work item)
    return (int)launch_kernel(anchor_max_bf16_kernel, dim3(grid < 768 ? grid : 768), dim3(256), 0, st, ea, grid);
}

}  // namespace aa
