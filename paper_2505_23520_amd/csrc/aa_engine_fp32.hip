// fp32 tile engine: the same online-softmax walk as the bf16 engines (stage 1
// anchor computation, Algorithm 1; stage 3 gathered sparse attention, Algorithm 3;
// dense causal comparator -- arXiv 2505.23520) with fp32 inputs, fp32 products and
// fp32 probabilities, on the fp32 matrix instruction v_mfma_f32_32x32x2_f32.
//
// Fragments (the layout of the bf16 engines with k = 2 per instruction): lane (n, hf) = (lane % 32,
// lane / 32).  S^T = K Q^T: keys = M, query rows = N; k slot hf of step (j, e) is column
// 8 j + 4 hf + e, so one 16-byte piece of a K row feeds four instructions.  Score register v of lane
// (n, hf) belongs to query row n and key 8 (v / 4) + 4 hf + v % 4 -- which is exactly the B operand
// of O^T = V^T P^T if k slot hf of step v is that key: the probabilities never move between lanes.
// V^T rows are columns of V in any order: row c of column block db is column T c + db (T = d / 32),
// so a lane's T columns are one wide load and a wave reads two whole V rows at once.
//
// Shape: work-group = one tile of 32 query rows = 4 waves that share the rows and split the 32-key
// blocks among them (block b belongs to wave b % 4); each keeps its own (m, l, O) and they are merged
// once, through LDS, at the end.  At 64 matrix cycles per instruction 32 keys of K and V (32 KB at
// d = 128) feed 8192 cycles of a wave, 16 B/clk for a CU: K and V come straight from L2 into
// registers, the loop has no LDS stage and no barrier, and a gathered row costs what a contiguous one
// does.  32 rows per work-group keep the chip filled at small sizes, and splitting the keys
// shortens the chain of a short sequence.
// Bound: the fp32 matrix pipe (157 TFLOP/s nominal; the vector ALU without packed instructions
// reaches half of that), and on short sequences the chain of one wave's blocks.
// Measured against vector FMAs over LDS tiles (one work-group per query block, two lanes per row):
// prefill of 4000 tokens, 8 / 2 heads, d = 128, block 128: 918 -> 155 us; 1024 tokens, 1 head, d = 64: 201 -> 42 us
// (both with the matching stage-2 kernels); dense causal, 2313 tokens, 2 heads, d = 64: 858 -> 61 us.
#include "aa_common.h"
#include "aa_engine.h"

namespace aa {

namespace {
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr floatx16 kZero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
constexpr int KB = 32;   // keys per block
constexpr int RT = 32;   // query rows per work-group
constexpr int NW = 4;    // waves per work-group

// Work-groups per grid row: a launch takes fewer than 2^32 threads in x, and 256 threads per 32 rows (per 16 at a block of
// 16) reach that with 5e8 (2.7e8) rows times heads.  A multiple of 8, so that decode_work's XCD of a work-group holds.
constexpr unsigned kGridX = 1u << 23;

template <int T> struct vcols;
template <> struct vcols<1> { typedef float type; };
template <> struct vcols<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct vcols<4> { typedef float type __attribute__((ext_vector_type(4))); };
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float comp(float x, int) { return x; }
template <class V> __device__ __forceinline__ float comp(const V& x, int i) { return x[i]; }

template <int D>
__global__ __launch_bounds__(64 * NW, D == 128 ? 2 : 3) void engine_fp32_kernel(EngineArgs a) {
    constexpr int T = D / 32;                        // column blocks of O
    constexpr int NK = D / 8;                        // 16-byte pieces of a K / Q row per lane
    constexpr int VK = 16 / NK;                      // V rows per K piece
    constexpr int LAG = D == 128 ? NK / 2 : NK / 4;                      // K pieces (and their share of V rows) not yet in flight
    typedef typename vcols<T>::type vec;
    __shared__ float obuf[NW][T][16][64];            // every wave's O^T registers
    __shared__ float mbuf[NW][RT], lbuf[NW][RT];
    const KParams& p = a.p;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 31, hf = lane >> 5;

    if (a.flags & kEngStoreState) store_dense_stats(a);
    if (!engine_selected(a)) return;
    const int rts = (p.bq + RT - 1) / RT;            // row tiles of a query block
    const unsigned id = blockIdx.y * kGridX + blockIdx.x, tiles = (unsigned)(p.nblk_max * rts);
    if (id >= tiles * (unsigned)p.Hq * (unsigned)p.B) return;
    const Work wk = decode_work(p, (int)tiles, id);
    const Seq sq = seq_of(p, wk.b);
    const int blk = wk.i / rts;
    const int row0 = blk * p.bq + (wk.i % rts) * RT;             // first row of the tile
    const int rend = min(min(blk * p.bq + p.bq, row0 + RT), sq.len);
    if (row0 >= rend) return;
    const int hk = wk.h / p.grp;
    const int g = blk / p.step;
    const bool direct = a.direct && window_start(p, g) <= p.n_init;   // no candidates: stage 1 finishes the rows
    if ((a.flags & kEngLoadState) && direct) return;
    const int r = row0 + n;
    const bool rok = r < rend;
    const int rlast = rend - 1;

    // ---- block sequence: [initial tokens][window .. diagonal][list]
    int W = 0, ninit = 0, T1 = 0, t2s = 0, nA = 0;
    if (a.flags & kEngAnchorRegion) {
        if (!(a.flags & kEngDense)) { W = window_start(p, g); ninit = p.n_init; }
        const int e1 = min(ninit, rlast + 1);
        T1 = (e1 + KB - 1) / KB;
        t2s = max(T1, W / KB);
        nA = T1 + max(0, rlast / KB + 1 - t2s);
    }
    int cnt = 0;
    long long lbase = 0;
    if (a.flags & kEngList) {
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

    const float* kb_ = (const float*)a.k + tok_offset(p, p.ks, sq, wk.b, hk, 0) + 4 * hf;
    const float* vb_ = (const float*)a.v + tok_offset(p, p.vs, sq, wk.b, hk, 0) + T * n;

    int key = key_of(wave), key_next = key_of(wave + NW);
    floatx4 q[NK], kf[NK];
    vec vf[16];
    auto load_k = [&](int j, int kk) { kf[j] = *(const floatx4*)(kb_ + (long long)kk * p.ks[2] + 8 * j); };
    auto load_v = [&](int v, int kk) {
        int src = 16 * hf;                           // byte address of lane 4 hf, opaque: 16 sums are not kept in registers
        asm volatile("" : "+v"(src));
        const int row = __builtin_amdgcn_ds_bpermute(src + 4 * (8 * (v >> 2) + (v & 3)), kk);
        vf[v] = *(const vec*)(vb_ + (long long)row * p.vs[2]);
    };
    {
        const float* src = (const float*)a.q + tok_offset(p, p.qs, sq, wk.b, wk.h, rok ? r : row0) + 4 * hf;
#pragma unroll
        for (int j = 0; j < NK; ++j) q[j] = *(const floatx4*)(src + 8 * j);
    }
#pragma unroll
    for (int j = 0; j < NK - LAG; ++j) load_k(j, key);

    const float c2 = p.sigma * 1.4426950408889634f;  // exp(sigma*x) = exp2(c2*x)
    float m = -INFINITY, l = 0.f;                    // l: this lane's keys only
    floatx16 o[T];
#pragma unroll
    for (int db = 0; db < T; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;

    // K pieces and V rows go through the registers in one stream: K pieces of a block, its V rows, K pieces
    // of the wave's next block.  Each is requested NK - LAG pieces (half to three quarters of K's share) ahead of its use,
    // into registers whose contents the products have just used; the order is pinned with scheduling fences.
#pragma unroll 1
    for (int t = wave; t < nT; t += NW) {
        // two accumulation chains: half the rounding error of one (measured against 64 bits: d = 128 outputs
        // 1.5e-6 off with one chain), and no product waits for the one before it
        floatx16 s2[2] = {kZero16, kZero16};
#pragma unroll
        for (int j = 0; j < NK; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s2[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][e], q[j][e], s2[e & 1], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < VK; ++u)
                if (j >= LAG) load_v((j - LAG) * VK + u, key);
            if (j < LAG) load_k(j + NK - LAG, key);
            __builtin_amdgcn_sched_barrier(0);
        }
        floatx16 s = s2[0] + s2[1];
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
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
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
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
#pragma unroll
            for (int db = 0; db < T; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(comp(vf[v], db), s[v], o[db], 0, 0, 0);
            if (v + VK * (NK - LAG) < 16) load_v(v + VK * (NK - LAG), key);
            if (v == VK * LAG - 1) {
                key = key_next;
                key_next = key_of(t + 2 * NW);
            }
            if (v >= VK * LAG && v % VK == 0) load_k(v / VK - LAG, key);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- merge the four waves' states.  Wave w finishes O^T registers 4 w .. 4 w + 3 of every column
    // block: of row n the columns T (8 w + 4 hf) .. + 4 T - 1.
    l += __shfl_xor(l, 32, 64);
#pragma unroll
    for (int db = 0; db < T; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) obuf[wave][db][v][lane] = o[db][v];
    if (hf == 0) { mbuf[wave][n] = m; lbuf[wave][n] = l; }
    __syncthreads();

    const long long ri = row_index(p, sq, wk.b, wk.h, rok ? r : row0);
    float mall = -INFINITY, m0 = -INFINITY, l0 = 0.f;
    if (a.flags & kEngLoadState) {
        m0 = a.Min[ri] / p.sigma;
        l0 = a.Lin[ri];
        mall = m0;
    }
    float mw[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mw[w] = mbuf[w][n];
        mall = fmaxf(mall, mw[w]);
    }
    auto scale_of = [&](float x) -> float {          // a part that has seen no key counts for nothing
        return x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x - mall) * c2);
    };
    float lall = 0.f, res[4 * T];                    // res[T e + db]: column T (8 wave + 4 hf) + T e + db
    const long long col0 = T * (8 * wave + 4 * hf);
    if (a.flags & kEngLoadState) {
        const float f0 = scale_of(m0);
        lall = l0 * f0;
#pragma unroll
        for (int c = 0; c < 4 * T; c += 4) {
            const floatx4 x = *(const floatx4*)(a.Accin + ri * D + col0 + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) res[c + e] = x[e] * f0;
        }
    } else {
#pragma unroll
        for (int c = 0; c < 4 * T; ++c) res[c] = 0.f;
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = scale_of(mw[w]);
        lall = fmaf(lbuf[w][n], f, lall);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int db = 0; db < T; ++db) res[T * e + db] = fmaf(obuf[w][db][4 * wave + e][lane], f, res[T * e + db]);
    }

    float ms = mall * p.sigma;
    if (!rok) return;
    const bool first = wave == 0 && hf == 0;
    bool store_out = (a.flags & kEngStoreOut) != 0;
    if ((a.flags & kEngStoreState) && direct) {
        // what stage 3 makes of a cached state and an empty list, bit for bit
        ms = ms / p.sigma * p.sigma;
        store_out = true;
    } else if (a.flags & kEngStoreState) {
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
    switch (p.d) {
        case 32: return (int)launch_kernel(engine_fp32_kernel<32>, grid, dim3(64 * NW), 0, st, ea);
        case 64: return (int)launch_kernel(engine_fp32_kernel<64>, grid, dim3(64 * NW), 0, st, ea);
        case 128: return (int)launch_kernel(engine_fp32_kernel<128>, grid, dim3(64 * NW), 0, st, ea);
        default: return -1;
    }
}

}  // namespace aa
