// Arguments of the online-softmax tile engines (bf16 and fp32 MFMA).
#pragma once
#include "aa_common.h"

namespace aa {

enum : int {
    kEngAnchorRegion = 1,   // walk the tiles of A(r): initial tokens + window .. diagonal
    kEngDense = 2,          // with kEngAnchorRegion: A(r) := [0, r] (dense causal attention)
    kEngList = 4,           // walk the chunks of the group's selected-column list
    kEngLoadState = 8,      // start from (M, L, Acc) instead of (-inf, 0, 0)
    kEngStoreState = 16,    // write M, L, (Acc), pooled anchor
    kEngStoreOut = 32,      // write out = acc / l and lse
    kEngParts = 64          // fp32, with kEngStoreState: write sums per 32-row tile, clear stage 2's counters
};

struct EngineArgs {
    KParams p;
    int flags;
    const void *q, *k, *v;
    const float *Min, *Lin, *Accin;
    const int* counts;
    const long long* offsets;
    const int* idx;
    float *Mout, *Lout, *Accout, *xa;
    // stage 1 only, nullable: pooled queries of stage 2 (bf16 hi / lo rows of 128, norm of lo),
    // written from the Q fragments the block's work-group holds anyway (see aa_pool.h).  fp32 with kEngParts: qp_hi and
    // qlo_norm receive the sums of every 32-row tile's queries (rows of d floats) and maxima, of which mask_fp32_kernel makes the
    // block means; tile t of block i at (block index) * ceil(bq / 32) + t
    void *qp_hi, *qp_lo;
    float* qlo_norm;
    // stage 1 only, nullable: largest key norm per (KV head, key block) for stage 2, and the counters to clear for it
    float* kmax_blk;
    int *zero_counts, *zero_seg;
    long long *zero_total, *zero_stats;
    int nseg;
    void* out;
    float* lse;
    // Fused prefill: rows of a group without candidates (W_g <= n_init) are finished by stage 1, which writes
    // out and lse instead of the state, and left alone by stage 3.  stats (nullable, stage 1): set if no
    // group has candidates, so that nothing else runs; receives the statistics of the call.
    int direct;
    long long* stats;
    // List-driven calls: offsets[groups_total] is the total (padded) list length.  Lists that do not
    // fit the caller's idx buffer (idx_capacity entries) are incomplete: the launch then does nothing.
    // Two engines can be launched for the same list-driven call; each decides on the device from that
    // total whether it is the one to run: sel = 0 runs always, sel = 1 runs iff the total is below
    // sel_entries, sel = 2 iff not.
    long long groups_total, idx_capacity;
    int sel;
    long long sel_entries;
};

// statistics of a call none of whose groups has candidates: every row attends all keys up to itself
__device__ __forceinline__ void store_dense_stats(const EngineArgs& a) {
    if (blockIdx.x != 0 || blockIdx.y != 0 || threadIdx.x != 0 || !a.stats) return;
    long long pairs = 0;
    for (int b = 0; b < a.p.B; ++b) {
        const long long len = a.p.packed ? a.p.cu[b + 1] - a.p.cu[b] : a.p.N;
        pairs += len * (len + 1) / 2;
    }
    a.stats[0] = pairs * a.p.Hq;
    a.stats[1] = 0; a.stats[2] = 0; a.stats[3] = 0;
}

// Requests all cache lines of the kernel arguments at once.  They are in no cache when a launch begins, and where the code
// comes upon them one by one, each is a round trip of its own ahead of the first tile.
__device__ __forceinline__ void touch_args(const EngineArgs& a) {
    static_assert(sizeof(EngineArgs) == 8 * 64, "members of every line are named below");
    asm volatile("" ::"s"(a.p.B), "s"(a.p.qs[2]), "s"(a.p.vs[2]), "s"(a.p.blk_cap), "s"(a.p.by_bq.d), "s"(a.q), "s"(a.idx),
                 "s"(a.kmax_blk), "s"(a.out), "s"(a.sel));
}

// true iff this launch has work to do (uniform over the grid)
__device__ __forceinline__ bool engine_selected(const EngineArgs& a) {
    if (!(a.flags & kEngList)) return true;
    const long long total = a.offsets[a.groups_total];
    if (total > a.idx_capacity) return false;
    if (a.sel == 0) return true;
    return (a.sel == 2) == (total >= a.sel_entries);
}

// Launchers: the launch's hipError_t, or -1 if there is no instantiation for ea.flags.
// 128 query rows per work-group, one instantiation per mode
int launch_engine_bf16(const EngineArgs& ea, unsigned grid, hipStream_t st);
// stage 1 without M, L and Acc: pooled anchors (ea.xa nullable) and what else stage 2 needs, 128 rows per work-group
int launch_anchor_max_bf16(const EngineArgs& ea, unsigned grid, hipStream_t st);
// 256 query rows (two consecutive blocks) per work-group; needs dense mode or an even step
int launch_engine_bf16_pp(const EngineArgs& ea, unsigned grid, hipStream_t st);

// fp32; writes no pooled anchors (ea.xa is not read: pool_fp32_kernel does that from M)
int launch_engine_fp32(const EngineArgs& ea, hipStream_t st);

}  // namespace aa
