// Host side of the C ABI (include/anchor_attention.h): argument checks, buffer
// arithmetic and kernel launches.  Nothing here allocates device memory or waits
// for the stream.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "../../include/anchor_attention.h"
#include "aa_common.h"
#include "aa_engine.h"
#include "aa_select.h"

namespace aa {
namespace {

thread_local char g_hip_err[256] = "";

int hip_fail(hipError_t e, const char* what) {
    snprintf(g_hip_err, sizeof(g_hip_err), "%s: %s", what, hipGetErrorString(e));
    return AA_EHIP;
}
#define AA_HIP(call)                                         \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #call);    \
    } while (0)
// AA_LAUNCH(kernel, grid, block, lds bytes, stream, args...): the launch's own status
#define AA_LAUNCH(kern, ...)                                 \
    do {                                                     \
        hipError_t e_ = launch_kernel(kern, __VA_ARGS__);    \
        if (e_ != hipSuccess) return hip_fail(e_, #kern);    \
    } while (0)

inline long long cdiv(long long a, long long b) { return (a + b - 1) / b; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Plan {
    KParams kp;
    aa_sizes sz;
    int nwords;
    // byte offsets inside the workspaces
    size_t sel_qhi, sel_qlo, sel_qln, sel_kmax, sel_bits, sel_segc, sel_kp;   // stripe_select workspace
    size_t pf_M, pf_L, pf_Acc, pf_xa, pf_counts, pf_offsets, pf_flag, pf_idx, pf_sel;  // prefill workspace
    size_t pf_partq, pf_partm;                                                                  // fp32 only
};

// candidates of the first `ngroups` groups of a sequence, each group's count rounded up to a list
// chunk (a group's candidate range depends on its index alone, not on the sequence's length)
long long padded_candidates(const aa_params* p, long long ngroups) {
    const long long span = (long long)p->block_q * p->step;
    long long tot = 0;
    for (long long g = 0; g < ngroups; ++g) {
        long long W = g * span - p->window;
        if (W < p->n_init) W = p->n_init;
        tot += cdiv(W - p->n_init, kIdxPad) * kIdxPad;
    }
    return tot;
}

int make_plan(const aa_params* p, Plan* pl) {
    if (!p || !pl) return AA_EINVAL;
    if (p->B <= 0 || p->Hq <= 0 || p->Hkv <= 0 || p->N <= 0 || p->d <= 0) return AA_EINVAL;
    if (p->Hq % p->Hkv != 0) return AA_EINVAL;
    if (p->block_q <= 0 || p->block_kv != p->block_q) return AA_EINVAL;
    if (p->n_init < 0 || p->window < 0 || p->step < 1) return AA_EINVAL;
    if (std::isnan(p->theta) || std::isnan(p->softmax_scale) || p->softmax_scale < 0.f) return AA_EINVAL;
    if (p->dtype != AA_FP32 && p->dtype != AA_BF16) return AA_EINVAL;
    if (p->granularity != AA_STRIPE && p->granularity != AA_BLOCK) return AA_EINVAL;
    if (p->granularity == AA_BLOCK && (p->n_init % p->block_kv || p->window % p->block_kv)) return AA_EINVAL;
    if (p->engine != AA_ENGINE_AUTO && p->engine != AA_ENGINE_128 && p->engine != AA_ENGINE_256) return AA_EINVAL;
    if (p->cu_seqlens && (p->total_tokens <= 0 || p->N > p->total_tokens)) return AA_EINVAL;
    if (p->causal != 1) return AA_EUNSUPPORTED;
    if (p->step > 128) return AA_EUNSUPPORTED;
    // the block-granularity mask kernel keeps a group's pooled rows and one flag per key block in LDS
    if (p->granularity == AA_BLOCK && mask_block_lds_bytes(p->N, p->d, p->block_q, p->step) > kMaskBlockLdsMax)
        return AA_EUNSUPPORTED;
    const int vec = p->dtype == AA_BF16 ? 8 : 4;             // elements per 16-byte access
    if (p->dtype == AA_BF16) {
        if (p->d != 128 || p->block_q != 128) return AA_EUNSUPPORTED;
        // K / V rows are addressed with 32-bit byte offsets from the head's first row
        if ((int64_t)p->N * p->k_stride[2] * 2 >= (1ll << 31) || (int64_t)p->N * p->v_stride[2] * 2 >= (1ll << 31))
            return AA_EUNSUPPORTED;
    } else {
        if (p->d != 32 && p->d != 64 && p->d != 128) return AA_EUNSUPPORTED;
        if (p->block_q < 16 || p->block_q > 128 || p->block_q % 16) return AA_EUNSUPPORTED;
    }
    const int64_t* st[4] = {p->q_stride, p->k_stride, p->v_stride, p->o_stride};
    for (int t = 0; t < 4; ++t) {
        if (st[t][2] < p->d || st[t][1] <= 0) return AA_EINVAL;
        for (int e = 0; e < 3; ++e)
            if (st[t][e] < 0 || st[t][e] % vec) return AA_EINVAL;
    }

    KParams& k = pl->kp;
    memset(&k, 0, sizeof(k));
    k.B = p->B; k.Hq = p->Hq; k.Hkv = p->Hkv; k.N = p->N; k.d = p->d;
    k.bq = p->block_q; k.n_init = p->n_init; k.w = p->window; k.step = p->step;
    k.grp = p->Hq / p->Hkv;
    k.packed = p->cu_seqlens != nullptr;
    k.use_anchor = p->use_anchor != 0;
    k.theta = p->theta;
    k.sigma = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->d);
    for (int e = 0; e < 3; ++e) {
        k.qs[e] = p->q_stride[e]; k.ks[e] = p->k_stride[e];
        k.vs[e] = p->v_stride[e]; k.os[e] = p->o_stride[e];
    }
    k.cu = p->cu_seqlens;
    k.total = k.packed ? p->total_tokens : (long long)p->B * p->N;
    const long long span = (long long)p->block_q * p->step;
    k.nblk_max = (int)cdiv(p->N, p->block_q);
    k.ngrp_max = (int)cdiv(p->N, span);
    // launch grids put heads (times sequences) on y / z
    if ((long long)p->Hq * p->B > 65535 || p->Hq + p->Hkv > 65535) return AA_EUNSUPPORTED;
    // no grid of the fp32 path limits the groups; such calls are refused because nothing has run them (from 1048561 tokens on,
    // with 8 GB of bit words per head)
    if (p->dtype == AA_FP32 && k.ngrp_max > 65535) return AA_EUNSUPPORTED;
    k.by_grp.set(k.grp);
    k.by_hkv.set(k.Hkv);
    k.by_step.set(k.step);
    k.by_bq.set(k.bq);
    k.by_pair.set((unsigned long long)k.nblk_max * k.grp);
    k.by_pair2.set((unsigned long long)((k.nblk_max + 1) / 2) * k.grp);

    aa_sizes& s = pl->sz;
    memset(&s, 0, sizeof(s));
    if (k.packed) {
        s.rows = (int64_t)p->Hq * p->total_tokens;
        s.blk_cap = p->total_tokens / p->block_q + p->B;
        s.grp_cap = p->total_tokens / span + p->B;
        s.blocks = (int64_t)p->Hq * s.blk_cap;
        s.groups = (int64_t)p->Hq * s.grp_cap;
        // Worst split of total_tokens into B sequences of at most N tokens.  A group counts in full
        // as soon as it has one row, so the bound goes over group counts: the sequences have at most
        // gtot groups together and at most ngrp_max each, and the candidates of a sequence with n
        // groups, F(n), are convex in n (later groups have longer candidate ranges): the maximum of
        // sum F(n_b) puts as many sequences as possible at ngrp_max and the remainder into one more.
        long long gtot = p->total_tokens / span + p->B;
        if (gtot > (long long)p->B * k.ngrp_max) gtot = (long long)p->B * k.ngrp_max;
        s.idx_capacity_max = (int64_t)p->Hq * ((gtot / k.ngrp_max) * padded_candidates(p, k.ngrp_max) +
                                               padded_candidates(p, gtot % k.ngrp_max));
    } else {
        s.rows = (int64_t)p->B * p->Hq * p->N;
        s.blk_cap = k.nblk_max;
        s.grp_cap = k.ngrp_max;
        s.blocks = (int64_t)p->B * p->Hq * s.blk_cap;
        s.groups = (int64_t)p->B * p->Hq * s.grp_cap;
        s.idx_capacity_max = (int64_t)p->B * p->Hq * padded_candidates(p, k.ngrp_max);
    }
    if (s.idx_capacity_max < kIdxPad) s.idx_capacity_max = kIdxPad;
    // fp32: row-major, d floats per row; bf16: per query block, four 32-row tiles in fragment order
    s.acc_elems = p->dtype == AA_BF16 ? s.blocks * (int64_t)p->block_q * p->d : s.rows * p->d;
    k.blk_cap = s.blk_cap;
    k.grp_cap = s.grp_cap;
    pl->nwords = (int)cdiv(p->N, 32);

    size_t off = 0;
    if (p->dtype == AA_BF16) {
        pl->sel_qhi = off; off += align256((size_t)s.blocks * 128 * 2);
        pl->sel_qlo = off; off += align256((size_t)s.blocks * 128 * 2);
        pl->sel_qln = off; off += align256((size_t)s.blocks * 4);
        pl->sel_kmax = off; off += align256((size_t)(s.blocks / k.grp) * 4);
    } else {
        pl->sel_qhi = off; off += align256((size_t)s.blocks * p->d * 4);
        pl->sel_qlo = off; pl->sel_qln = off; pl->sel_kmax = off;
    }
    pl->sel_bits = off; off += align256((size_t)s.groups * pl->nwords * 4);
    pl->sel_segc = off; off += align256((size_t)s.groups * cdiv(pl->nwords, 64) * 4);
    pl->sel_kp = off;
    if (p->granularity == AA_BLOCK) off += align256((size_t)(s.blocks / k.grp) * p->d * 4);
    s.select_ws_bytes = off;

    off = 0;
    pl->pf_M = off; off += align256((size_t)s.rows * 4);
    pl->pf_L = off; off += align256((size_t)s.rows * 4);
    pl->pf_Acc = off; off += align256((size_t)s.acc_elems * 4);
    pl->pf_xa = off; off += align256((size_t)s.blocks * 4);
    pl->pf_counts = off; off += align256((size_t)s.groups * 4);
    pl->pf_offsets = off; off += align256((size_t)(s.groups + 1) * 8);
    pl->pf_flag = off; off += 256;
    pl->pf_idx = off; off += align256((size_t)s.idx_capacity_max * 4);
    pl->pf_sel = off; off += s.select_ws_bytes;
    pl->pf_partq = pl->pf_partm = off;
    if (p->dtype == AA_FP32 && p->granularity == AA_STRIPE) {
        const size_t tiles = (size_t)s.blocks * (size_t)cdiv(p->block_q, 32);
        off += align256(tiles * p->d * 4);
        pl->pf_partm = off; off += align256(tiles * 4);
    }
    s.prefill_ws_bytes = off;
    return AA_OK;
}

bool misaligned(const void* ptr) { return ((uintptr_t)ptr & 15) != 0; }

// ---- workspace of stripe_select_noalloc: a device array that is part of the loaded library, one
// copy per GPU, held until the process ends.  Its name is a host-side handle, not a device
// address: host code uses the address hipGetSymbolAddress reports for the current device.
constexpr size_t kScratchBytes = (size_t)AA_NOALLOC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
__device__ __align__(256) static unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void** out) {
    int dev = -1;
    AA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return AA_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        AA_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return AA_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return AA_OK;
}

// kernels that ask for more dynamic LDS than the default limit: raised once per process
std::once_flag g_attr_once;
hipError_t g_attr_status = hipSuccess;
hipError_t raise_lds_limits() {
    std::call_once(g_attr_once, [] {
        g_attr_status = hipFuncSetAttribute((const void*)mask_block_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)kMaskBlockLdsMax);
    });
    return g_attr_status;
}

int engine_status(int rc, const char* name) {
    if (rc < 0) return AA_EUNSUPPORTED;
    return rc == (int)hipSuccess ? AA_OK : hip_fail((hipError_t)rc, name);
}

int launch_engine(const Plan& pl, const aa_params* prm, EngineArgs& ea, hipStream_t st) {
    const KParams& k = pl.kp;
    const unsigned grid = (unsigned)((long long)k.nblk_max * k.Hq * k.B);
    ea.groups_total = pl.sz.groups;
    ea.sel = 0;
    if (prm->dtype == AA_BF16) {
        // Two bf16 engines: 128 query rows per work-group (three work-groups per CU) and 256 rows
        // per work-group with the MFMA / softmax phases of the two waves of a SIMD alternating.
        // The second is faster on long tile loops and slower on short ones (its prologue and
        // epilogue overlap with nothing); it needs both blocks of a pair to share window and list.
        // Dense, 32 heads, 128 / 256 rows: 4096 tokens 130 / 133 us, 6000 273 / 280, 8192 481 / 474,
        // 32768 7214 / 6956.
        // Stage 3, where the line lies depends on heads, step and the spread of the lists; time of the 256-row engine over
        // the 128-row one: 32 / 8 heads, step 16, every column selected, mean list 14 tiles 1.09, 29 0.98, 45 1.02, 61 1.00,
        // 108 0.98; a part selected, 16 tiles 1.09, 25 1.00, 35 1.03, 50 (131072 tokens) 1.05; 8 / 8 heads 45 tiles 1.06, 61
        // 1.04, 108 0.93; 16 / 2 heads, step 4, 24 tiles 0.89, 56 0.83, 72 0.99.  48 tiles lie in the middle.
        const long long pp_entries = 48ll * kIdxPad * pl.sz.groups;
        const bool pair_ok = (ea.flags & kEngDense) || k.step % 2 == 0;
        int choice = prm->engine;                   // 0 auto, 1: 128 rows, 2: 256 rows
        if (!pair_ok) choice = AA_ENGINE_128;
        if (choice == AA_ENGINE_AUTO) {
            // stage 3: decided on the device from the list lengths, unless no outcome reaches the limit
            // (a launch that finds itself not selected still takes 4 us, 15 us at 128k)
            if (ea.flags & kEngList) choice = pl.sz.idx_capacity_max < pp_entries ? AA_ENGINE_128 : 3;
            else if (ea.flags & kEngDense) choice = k.N >= 8192 ? AA_ENGINE_256 : AA_ENGINE_128;
            else choice = AA_ENGINE_128;            // anchor region alone: at most step + 3 blocks of keys
        }
        const unsigned gridp = (unsigned)((long long)((k.nblk_max + 1) / 2) * k.Hq * k.B);
        int rc = AA_OK;
        if (choice == 3) {
            ea.sel_entries = pp_entries;
            ea.sel = 1;
            rc = engine_status(launch_engine_bf16(ea, grid, st), "engine_bf16_kernel");
            if (rc != AA_OK) return rc;
            ea.sel = 2;
            rc = engine_status(launch_engine_bf16_pp(ea, gridp, st), "engine_bf16_pp_kernel");
        } else if (choice == AA_ENGINE_256) {
            rc = engine_status(launch_engine_bf16_pp(ea, gridp, st), "engine_bf16_pp_kernel");
        } else {
            rc = engine_status(launch_engine_bf16(ea, grid, st), "engine_bf16_kernel");
        }
        return rc;
    }
    return engine_status(launch_engine_fp32(ea, st), "engine_fp32_kernel");
}

// no group of the call has candidates (the last group of the longest sequence has the most)
bool no_candidates(const KParams& k) {
    return (long long)(k.ngrp_max - 1) * k.step * k.bq - k.w <= k.n_init;
}

// Stage 1 of the fused prefill may finish the rows of groups without candidates itself.  The stage-wise path
// must give the same bits, so only where both take the same engine (the 256-row engine, when forced, does not).
bool direct_ok(const aa_params* p) { return p->dtype != AA_BF16 || p->engine != AA_ENGINE_256 || p->step % 2; }

// the 128-row engine's stage 1 also leaves the key norms of the stripe mask and its cleared counters
bool pooled_keys(const aa_params* p) { return p->granularity == AA_STRIPE && direct_ok(p); }

// Fused prefill without the cached state: stage 1 leaves the row maxima's means only, stage 3 attends the anchor region again, to
// the same bits.  At step 1 the region is (n_init + window) / 64 + 2 tiles of keys; finding its maxima costs half of
// attending it, the state's way through memory (128 KB per block and direction with M, L and Acc) three to four tiles.
// 32 / 8 heads, n_init = window = 128, cached / again: 4096 tokens (1024 blocks) 80.5 / 81.4 us, 8192 150 / 142, 16384
// 324 / 281, 30011 592 / 552, two sequences of 5000 198 / 171, every column selected 16384 1995 / 1990; with 8 / 8 heads,
// 9000 tokens (568 blocks) 67.7 / 68.3; 1000 tokens 36.0 / 37.3 (a chip that is not full pays for the longer chain of a block).
// 16384 tokens with n_init + window = 512: 367 / 348, 640: 393 / 392.  An even step could take the 256-row engine, a step of 3
// has two tiles more.
bool recompute_anchor(const Plan& pl, const aa_params* p) {
    const long long blocks = (pl.kp.total + p->block_q - 1) / p->block_q * p->Hq;
    return p->dtype == AA_BF16 && p->step == 1 && (long long)p->n_init + p->window <= 512 && blocks >= 1536 && direct_ok(p);
}

// Fused fp32 prefill: stage 1 leaves sums of every 32 rows, which the mask kernel turns into the pooled rows, instead of a pooling
// kernel.  That saves a launch and the kernel (4 us and more with the rows), but a mask wave, which meets every block of
// its keys' future, has d / 8 loads for each of the block's T tiles (1, 2 or 4 as compiled) in its chain: N d T / block is the
// measure.  Whole call, pooling kernel / sums, us (heads): 8192 (d = 64: 4096 tokens, block 64) 35.4 / 33.4 (1); 8000 (d = 64: 4000,
// block 128) 41.5 / 40.3 (4); 12000 (d = 128: 3000, block 128) 79.1 / 78.3 (8), (3000, block 32) 44.9 / 44.8 (1); 16000 (d =
// 128: 4000, block 128) 48.2 / 49.0 (1), (d = 64: 8000, block 64) 89.9 / 90.4 (8), (d = 32: 16000, block 64) 82.2 / 82.8 (2);
// 32000 (d = 128: 16000, block 64) 339 / 350 (8).  Blocks of at most 32 rows need no addition, and many heads
// make their pooling kernel long (d = 128, block 32, 8000 tokens: 100 / 103 (4), 167 / 164 (8), 297 / 275 (16)).
bool pools_from_parts(const KParams& k, const aa_params* p) {
    if (p->dtype != AA_FP32 || p->granularity != AA_STRIPE) return false;
    if (p->block_q <= 32 && k.total * p->Hq >= 8ll * p->N) return true;
    const long long tiles = p->block_q <= 32 ? 1 : p->block_q <= 64 ? 2 : 4;
    return (long long)p->N * p->d * tiles <= 12288ll * p->block_q;
}

// sel_ws (nullable): a stripe_select workspace (with the call's counts); the bf16 engines then also leave the pooled queries of
// stage 2 there, and the fp32 path leaves the pooled anchors to run_select (which is told so).
// out (nullable), lse, stats: see EngineArgs::direct; total, call_stats: the sums that the fill kernel adds to, cleared here;
// parts (nullable): the prefill workspace, where the fp32 path then leaves its sums per 32-row tile
int run_anchor(const Plan& pl, const aa_params* p, const void* q, const void* k, const void* v, float* M, float* L,
               float* Acc, float* xa, char* sel_ws, int32_t* counts, char* parts, long long* total, int64_t* call_stats,
               void* out, float* lse, int64_t* stats, hipStream_t st) {
    EngineArgs ea;
    memset(&ea, 0, sizeof(ea));
    ea.p = pl.kp;
    ea.flags = kEngAnchorRegion | kEngStoreState;
    ea.q = q; ea.k = k; ea.v = v;
    ea.Mout = M; ea.Lout = L; ea.Accout = Acc; ea.xa = xa;
    ea.direct = out != nullptr;
    ea.out = out; ea.lse = lse; ea.stats = (long long*)stats;
    if (sel_ws && p->dtype == AA_BF16) {
        ea.qp_hi = sel_ws + pl.sel_qhi; ea.qp_lo = sel_ws + pl.sel_qlo; ea.qlo_norm = (float*)(sel_ws + pl.sel_qln);
        if (pooled_keys(p)) {
            ea.kmax_blk = (float*)(sel_ws + pl.sel_kmax);
            ea.zero_counts = counts; ea.zero_seg = (int*)(sel_ws + pl.sel_segc); ea.nseg = (int)cdiv(pl.nwords, 64);
            if (total) { ea.zero_total = total; ea.zero_stats = (long long*)call_stats; }
        }
    }
    if (!M) {                                        // fused prefill that keeps no state (see recompute_anchor)
        ea.groups_total = pl.sz.groups;
        if (!pl.kp.use_anchor) ea.xa = nullptr;
        return engine_status(launch_anchor_max_bf16(ea, (unsigned)((long long)pl.kp.nblk_max * pl.kp.Hq * pl.kp.B), st),
                             "anchor_max_bf16_kernel");
    }
    if (parts) {                            // fp32 stripes in the fused call
        ea.flags |= kEngParts;
        ea.qp_hi = parts + pl.pf_partq; ea.qlo_norm = (float*)(parts + pl.pf_partm);
        ea.zero_counts = counts; ea.zero_seg = (int*)(sel_ws + pl.sel_segc); ea.nseg = (int)cdiv(pl.nwords, 64);
        ea.zero_total = total; ea.zero_stats = (long long*)call_stats;
    }
    const int rc = launch_engine(pl, p, ea, st);
    if (rc != AA_OK || p->dtype == AA_BF16 || sel_ws || !xa) return rc;
    SelectArgs sa;
    memset(&sa, 0, sizeof(sa));
    sa.p = pl.kp;
    sa.m_rows = M; sa.xa_out = xa;
    AA_LAUNCH(pool_fp32_kernel, dim3(pl.kp.nblk_max, pl.kp.Hq, pl.kp.B), dim3(256), 0, st, sa);
    return AA_OK;
}

// fused_M (nullable): the call follows run_anchor with this workspace, M is stage 1's; bf16: the pooled queries
// are in ws already; fp32: the pooled anchors are still to be computed, into xa
// total (nullable): the lists stand at places of their own (fused call), and their padded entries are summed up there
// stats (nullable): receives attended pairs and selected entries
int run_select(const Plan& pl, const aa_params* p, const void* q, const void* k, const float* xa, int32_t* counts,
               int64_t* offsets, int32_t* idx, int64_t cap, int32_t* flag, char* ws, const float* fused_M, float* xa_out,
               const char* parts, long long* total, int64_t* stats, hipStream_t st) {
    const KParams& kp = pl.kp;
    SelectArgs sa;
    memset(&sa, 0, sizeof(sa));
    sa.p = kp;
    sa.q = q; sa.k = k; sa.xa = xa;
    sa.qp_hi = ws + pl.sel_qhi; sa.qp_lo = ws + pl.sel_qlo; sa.qp_f32 = (float*)(ws + pl.sel_qhi);
    sa.bits = (unsigned*)(ws + pl.sel_bits);
    sa.kp_f32 = (float*)(ws + pl.sel_kp);
    sa.qlo_norm = (float*)(ws + pl.sel_qln);
    sa.segcount = (int*)(ws + pl.sel_segc);
    sa.nseg = (int)cdiv(pl.nwords, 64);
    sa.is_bf16 = p->dtype == AA_BF16;
    sa.nwords = pl.nwords;
    sa.counts = counts; sa.offsets = (long long*)offsets; sa.idx = idx;
    sa.idx_capacity = cap; sa.overflow = flag;
    sa.groups_total = pl.sz.groups;
    sa.stats = (long long*)stats;
    sa.total = total;
    if (total) sa.list_room = cap / ((long long)kp.Hq * (kp.packed ? 1 : kp.B));

    const dim3 gblk(kp.nblk_max, kp.Hq, kp.B), ggrp(kp.ngrp_max, kp.Hq, kp.B);
    if (p->granularity == AA_BLOCK) AA_HIP(raise_lds_limits());   // before anything is enqueued
    // A group's count is the sum of its segments'.  The scan takes it from there while that is little work for its one
    // work-group (64k segments: 16k tokens at step 1 32k; adding to the counts from every mask work-group cost 9 us
    // there); beyond, the mask kernels add to the counts as well.
    const long long segs = (long long)pl.sz.groups * sa.nseg;
    sa.sum_segs = sa.list_room || segs <= 65536;
    if (p->granularity == AA_BLOCK) {
        AA_LAUNCH(zero_i32_kernel, dim3((unsigned)cdiv(segs, 256)), dim3(256), 0, st, sa.segcount, segs, sa.total,
                  sa.total ? sa.stats : nullptr);
        if (!sa.sum_segs)
            AA_LAUNCH(zero_i32_kernel, dim3((unsigned)cdiv(pl.sz.groups, 256)), dim3(256), 0, st, counts,
                      (long long)pl.sz.groups, nullptr, nullptr);
    }
    const bool q_pooled = fused_M && p->dtype == AA_BF16;
    if (p->dtype != AA_BF16 && fused_M) {
        sa.m_rows = fused_M; sa.xa_out = xa_out;
        // first block of the first group with candidates (W_g > n_init); 32 bits: the call has such a group
        const long long span = (long long)kp.bq * kp.step;
        sa.first_block = (int)(((long long)kp.n_init + kp.w) / span + 1) * kp.step;
    }
    sa.pool_skip_q = q_pooled;
    if (p->granularity == AA_BLOCK) {
        if (p->dtype != AA_BF16)
            AA_LAUNCH(pool_fp32_kernel, gblk, dim3(256), 0, st, sa);
        else if (!q_pooled)
            AA_LAUNCH(pool_q_bf16_kernel, gblk, dim3(256), 0, st, sa);
        AA_LAUNCH(pool_k_kernel, dim3(kp.nblk_max, kp.Hkv, kp.B), dim3(256), 0, st, sa);
        AA_LAUNCH(mask_block_kernel, ggrp, dim3(256), mask_block_lds_bytes(kp.N, kp.d, kp.bq, kp.step), st, sa);
    } else if (p->dtype == AA_BF16) {
        sa.kmax_blk = (float*)(ws + pl.sel_kmax);
        if (!q_pooled || !pooled_keys(p))
            AA_LAUNCH(pool_q_bf16_kernel, dim3(kp.nblk_max, (q_pooled ? 0 : kp.Hq) + kp.Hkv, kp.B), dim3(256), 0, st, sa);
        // One work-group per (query head, row tile, key span with candidates); the longest sequence bounds
        // every other.  The span is halved until there are more than 1.5 work-groups per CU (three fit, but a span's
        // fixed cost, loading the pooled rows, is about three of its 64-key tiles).  All of stage 2 at 8k tokens: 54 us
        // with 96 work-groups of 2048 keys, 36 with 736 of 256 keys, 37 with 384 of 512; at 16k: 66 us with 224 of 2048,
        // 56 with 448 of 1024, 62 with 896 of 512.
        sa.mask_span = kSegKeys;
        for (;;) {
            sa.mask_items = mask_pair_items(kp.nblk_max, kp.step, kp.bq, kp.w, kp.n_init, sa.mask_span);
            if ((long long)sa.mask_items * kp.Hq * (kp.packed ? 1 : kp.B) > 384 || sa.mask_span == kMaskSpanMin) break;
            sa.mask_span /= 2;
        }
        const long long mask_per_xcd = cdiv((long long)sa.mask_items * kp.Hq * kp.B, 8);
        if (mask_per_xcd * 8 > 0x7fffffffll) return AA_EUNSUPPORTED;
        const dim3 gm((unsigned)(mask_per_xcd > 0 ? mask_per_xcd * 8 : 8));
        AA_LAUNCH(mask_bf16_kernel, gm, dim3(256), 0, st, sa);
    } else {
        if (parts) {
            sa.part_q = (const float*)(parts + pl.pf_partq); sa.part_m = (const float*)(parts + pl.pf_partm);
        } else {
            AA_LAUNCH(pool_fp32_kernel, gblk, dim3(256), 0, st, sa);
        }
        const int rc = engine_status(launch_mask_fp32(sa, st), "mask_fp32_kernel");
        if (rc != AA_OK) return rc;
    }
    if (p->granularity == AA_BLOCK) AA_LAUNCH(count_kernel, ggrp, dim3(256), 0, st, sa);
    if (sa.list_room) return engine_status(launch_fill(sa, kFillPlaces, st), "fill_kernel");
    // few groups: the fill kernel does the scan's work (a launch less, 5 us); every one of its work-groups then
    // reads up to all segments, 8 per thread at this limit
    const bool fill_scans = segs <= 2048;
    if (!fill_scans) AA_LAUNCH(scan_kernel, dim3(1), dim3(1024), 0, st, sa);
    return engine_status(launch_fill(sa, fill_scans ? kFillScan : kFillOffsets, st), "fill_kernel");
}

int run_sparse(const Plan& pl, const aa_params* p, const void* q, const void* k, const void* v, const float* M,
               const float* L, const float* Acc, const int32_t* counts, const int64_t* offsets, const int32_t* idx,
               int64_t idx_capacity, void* out, float* lse, bool direct, hipStream_t st) {
    EngineArgs ea;
    memset(&ea, 0, sizeof(ea));
    ea.p = pl.kp;
    ea.flags = kEngList | kEngStoreOut | (M ? kEngLoadState : kEngAnchorRegion);
    ea.q = q; ea.k = k; ea.v = v;
    ea.Min = M; ea.Lin = L; ea.Accin = Acc;
    ea.counts = counts; ea.offsets = (const long long*)offsets; ea.idx = idx;
    ea.idx_capacity = idx_capacity;
    ea.out = out; ea.lse = lse;
    ea.direct = direct;
    return launch_engine(pl, p, ea, st);
}

}  // namespace
}  // namespace aa

using namespace aa;

extern "C" {

int anchor_sizes(const aa_params* params, aa_sizes* out) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!out) return AA_EINVAL;
    *out = pl.sz;
    return AA_OK;
}

int anchor_workspace_bytes(const aa_params* params, size_t* bytes_out) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!bytes_out) return AA_EINVAL;
    *bytes_out = pl.sz.prefill_ws_bytes;
    return AA_OK;
}

int anchor_compute(const aa_params* params, const void* q, const void* k, const void* v, float* M, float* L,
                   float* Acc, float* xa_pooled, void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !v || !M || !L || !xa_pooled) return AA_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(Acc)) return AA_EINVAL;
    return run_anchor(pl, params, q, k, v, M, L, Acc, xa_pooled, nullptr, nullptr, nullptr, nullptr, nullptr,
                      nullptr, nullptr, nullptr, (hipStream_t)stream);
}

int stripe_select(const aa_params* params, const void* q, const void* k, const float* xa_pooled, int32_t* counts,
                  int64_t* offsets, int32_t* idx, int64_t idx_capacity, int32_t* overflow_flag, void* ws,
                  size_t ws_bytes, void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !xa_pooled || !counts || !offsets || !idx || !overflow_flag || !ws) return AA_EINVAL;
    if (idx_capacity < 0 || misaligned(q) || misaligned(k) || misaligned(idx) || misaligned(ws)) return AA_EINVAL;
    if (ws_bytes < pl.sz.select_ws_bytes) return AA_EWORKSPACE;
    return run_select(pl, params, q, k, xa_pooled, counts, offsets, idx, idx_capacity, overflow_flag, (char*)ws,
                      nullptr, nullptr, nullptr, nullptr, nullptr, (hipStream_t)stream);
}

int stripe_select_noalloc(const aa_params* params, const void* q, const void* k, const float* xa_pooled,
                          int32_t* counts, int64_t* offsets, int32_t* idx, int64_t idx_capacity,
                          int32_t* overflow_flag, void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !xa_pooled || !counts || !offsets || !idx || !overflow_flag) return AA_EINVAL;
    if (idx_capacity < 0 || misaligned(q) || misaligned(k) || misaligned(idx)) return AA_EINVAL;
    if (pl.sz.select_ws_bytes > kScratchBytes) return AA_EWORKSPACE;
    void* ws = nullptr;
    rc = scratch_of_current_device(&ws);
    if (rc != AA_OK) return rc;
    return run_select(pl, params, q, k, xa_pooled, counts, offsets, idx, idx_capacity, overflow_flag, (char*)ws,
                      nullptr, nullptr, nullptr, nullptr, nullptr, (hipStream_t)stream);
}

int sparse_attn(const aa_params* params, const void* q, const void* k, const void* v, const float* M, const float* L,
                const float* Acc, const int32_t* counts, const int64_t* offsets, const int32_t* idx,
                int64_t idx_capacity, void* out, float* lse, void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !v || !counts || !offsets || !idx || !out || idx_capacity < 0) return AA_EINVAL;
    const int nstate = (M != nullptr) + (L != nullptr) + (Acc != nullptr);
    if (nstate != 0 && nstate != 3) return AA_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || misaligned(idx) || misaligned(Acc))
        return AA_EINVAL;
    return run_sparse(pl, params, q, k, v, M, L, Acc, counts, offsets, idx, idx_capacity, out, lse, false,
                      (hipStream_t)stream);
}

int anchor_attention_prefill(const aa_params* params, const void* q, const void* k, const void* v, void* out,
                             float* lse, int64_t* stats, void* ws, size_t ws_bytes, void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !v || !out || !ws) return AA_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || misaligned(ws)) return AA_EINVAL;
    if (ws_bytes < pl.sz.prefill_ws_bytes) return AA_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    char* w = (char*)ws;
    float* M = (float*)(w + pl.pf_M);
    float* L = (float*)(w + pl.pf_L);
    float* Acc = (float*)(w + pl.pf_Acc);
    float* xa = (float*)(w + pl.pf_xa);
    int32_t* counts = (int32_t*)(w + pl.pf_counts);
    int64_t* offsets = (int64_t*)(w + pl.pf_offsets);
    int32_t* flag = (int32_t*)(w + pl.pf_flag);
    int32_t* idx = (int32_t*)(w + pl.pf_idx);
    // bf16: the block means of Q (first step of stage 2) come out of stage 1, which holds the block's
    // queries in registers; the stage-wise entry points compute the same bits in a kernel of their own
    // Rows of groups without candidates are complete after stage 1, which writes their output; if that is every
    // row (a prompt within its first group and window), it is the whole call: 53 -> 25 us at 1000 tokens, where
    // the other kernels' launches alone took 25 us.  At 8k tokens and step 16 it is a quarter of the rows.
    const bool direct = direct_ok(params);
    if (direct && no_candidates(pl.kp))
        return run_anchor(pl, params, q, k, v, M, L, Acc, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, out, lse, stats, st);
    // every list at a place of its own where the places can be computed (the index region holds every candidate)
    const bool places = (long long)params->block_q * params->step % kIdxPad == 0;
    long long* total = places ? (long long*)offsets + pl.sz.groups : nullptr;
    char* parts = pools_from_parts(pl.kp, params) ? w : nullptr;
    const bool again = recompute_anchor(pl, params);
    rc = run_anchor(pl, params, q, k, v, again ? nullptr : M, L, Acc, xa, w + pl.pf_sel, counts,
                    parts, total, places ? stats : nullptr, direct && !again ? out : nullptr, lse, nullptr, st);
    if (rc != AA_OK) return rc;
    rc = run_select(pl, params, q, k, xa, counts, offsets, idx, pl.sz.idx_capacity_max, flag, w + pl.pf_sel, M, xa,
                    parts, total, stats, st);
    if (rc != AA_OK) return rc;
    rc = run_sparse(pl, params, q, k, v, again ? nullptr : M, L, Acc, counts, offsets, idx, pl.sz.idx_capacity_max, out, lse,
                    direct && !again, st);
    if (rc != AA_OK) return rc;
    return AA_OK;
}

int dense_causal_flash(const aa_params* params, const void* q, const void* k, const void* v, void* out, float* lse,
                       void* stream) {
    Plan pl;
    int rc = make_plan(params, &pl);
    if (rc != AA_OK) return rc;
    if (!q || !k || !v || !out) return AA_EINVAL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out)) return AA_EINVAL;
    EngineArgs ea;
    memset(&ea, 0, sizeof(ea));
    ea.p = pl.kp;
    ea.flags = kEngAnchorRegion | kEngDense | kEngStoreOut;
    ea.q = q; ea.k = k; ea.v = v;
    ea.out = out; ea.lse = lse;
    return launch_engine(pl, params, ea, (hipStream_t)stream);
}

const char* anchor_strerror(int code) {
    switch (code) {
        case AA_OK: return "ok";
        case AA_EINVAL: return "invalid argument";
        case AA_EUNSUPPORTED: return "unsupported configuration";
        case AA_EWORKSPACE: return "workspace too small";
        case AA_EHIP: return "HIP error";
        default: return "unknown error code";
    }
}

const char* anchor_last_hip_error(void) { return g_hip_err; }

}  // extern "C"
