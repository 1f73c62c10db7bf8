"""Performance cases of the AnchorAttention prefill library.

Every case is one pass through the public entry points of ``paper_2505_23520_amd.api`` on inputs
that are resident on the GPU: the fused sparse prefill, the same three stages called one by one, and
the dense causal kernel that a caller falls back to (or compares with).  The head layout (32 query /
8 KV heads, d = 128), block 128, step 16 and the planted-stripe input recipes are those of the
repository's workloads (``synth.py``), drawn on the GPU here because the host recipe takes minutes
at 128k tokens.

A case is a dict of plain values:
  kind    "prefill" (anchor_attention_prefill) | "stages" (anchor_compute, stripe_select,
          sparse_attn) | "dense" (dense_causal_flash)
  dtype   "bf16" | "fp32"
  lens    sequence lengths, comma separated; packed: one token axis with cu_seqlens, else a batch
  Hq, Hkv, d, block, n_init, window, step, theta, use_anchor, granularity ("stripe" | "block")
  signal  "literal": planted columns do not stand out (every column passes the threshold, the
          method's dense worst case); "logit": the threshold separates them; "peaked": they also
          hold most of the attention mass, with theta scaled alike
  planted stripe columns per sequence and KV head, of magnitude mag_lo .. mag_hi
  ar1     correlation of successive queries
  layout  "head" ([B, H, N, d]) | "token" ([B, N, H, d], as a projection leaves it)
"""
import math

import torch

from paper_2505_23520_amd import api

_SINKS, _SINK_MAG = 4, 4.0


def _case(name, kind, lens, **kw):
    c = dict(name=name, kind=kind, dtype="bf16", lens=lens, packed=False, Hq=32, Hkv=8, d=128, block=128,
             n_init=128, window=128, step=16, theta=math.log(32.0), use_anchor=True, granularity="stripe",
             signal="logit", planted=64, mag_lo=2.5, mag_hi=2.5, ar1=0.0, layout="head")
    c.update(kw)
    return c


def listed():
    return [
        # a short chat prompt: shorter than one group, latency and launches are what counts
        _case("prefill_short", "prefill", "1000"),
        # the 8k workload: an ordinary document
        _case("prefill_8k", "prefill", "8192"),
        # the 32k workload at a ragged length, correlated queries, K/V as the projections leave them
        _case("prefill_32k_odd", "prefill", "30011", planted=256, ar1=0.3, signal="peaked", layout="token"),
        # the headline workload where the threshold separates stripes from background (97 % sparsity)
        _case("prefill_128k", "prefill", "131072", planted=1024, mag_lo=1.5, mag_hi=3.5),
        # the same as literally worded: every candidate is selected, the largest amount of work
        _case("prefill_128k_literal", "prefill", "131072", planted=1024, mag_lo=1.5, mag_hi=3.5, signal="literal"),
        # a serving batch of prompts of mixed, odd lengths on one token axis
        _case("prefill_packed", "prefill", "911,4097,16384,30001", packed=True),
        # one list per query block (the method without the step rule)
        _case("prefill_step1", "prefill", "16384", planted=128, step=1),
        # a caller that runs the stages one by one and keeps the intermediate state
        _case("stages_16k", "stages", "16384", planted=128),
        # the tiny single-head fp32 workload
        _case("prefill_fp32_tiny", "prefill", "1024", dtype="fp32", Hq=1, Hkv=1, d=64, block=64, n_init=16, window=64,
              step=4, theta=math.log(16.0), planted=8, mag_lo=3.0, mag_hi=3.0, signal="peaked"),
        # fp32 at an ordinary prompt length and head dimension, a few heads (one tensor-parallel shard)
        _case("prefill_fp32_gqa", "prefill", "4000", dtype="fp32", Hq=8, Hkv=2, step=4, signal="peaked"),
        # dense causal attention: a batch of two odd-length prompts
        _case("dense_3k_b2", "dense", "3001,3001"),
        # dense causal attention at the length where the sparse path starts to pay
        _case("dense_32k", "dense", "32768", planted=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill"] * 5 + ["fp32"] * 2 + ["stages"] * 2 + ["dense"] * 2)
    if kind == "fp32":
        d, block = rng.choice([32, 64, 128]), rng.choice([32, 64, 128])
        Hkv = rng.choice([1, 2])
        n = _log_int(rng, 200, 6000)
        return _plain(_case("", rng.choice(["prefill", "prefill", "dense"]), str(n), dtype="fp32", Hq=Hkv * rng.choice([1, 2, 4]),
                            Hkv=Hkv, d=d, block=block, n_init=rng.choice([16, block]), window=rng.choice([block, 2 * block]),
                            step=rng.choice([1, 4, 16]), theta=math.log(16.0), planted=max(4, n // 128), signal="peaked"))
    heads = rng.choice([(32, 8), (32, 8), (16, 2), (8, 8)])
    kw = dict(Hq=heads[0], Hkv=heads[1], ar1=rng.choice([0.0, 0.3]), layout=rng.choice(["head", "head", "token"]))
    if kind == "dense":
        n = _log_int(rng, 200, 50000)
        lens = [n] * (2 if n < 8000 and rng.random() < 0.4 else 1)
        return _plain(_case("", "dense", ",".join(map(str, lens)), planted=max(4, n // 128), **kw))
    kw["step"] = rng.choice([16, 16, 16, 1, 4])
    if kind == "stages":
        n = 128 * _log_int(rng, 4, 300)
        return _plain(_case("", "stages", str(n), planted=max(4, n // 128), **kw))
    kw["signal"] = rng.choice(["logit", "logit", "peaked", "literal"])
    if rng.random() < 0.3:
        lens = [_log_int(rng, 100, 30000) for _ in range(rng.choice([2, 3, 5]))]
        kw.update(packed=True, layout="head")
    else:
        n = _log_int(rng, 300, 50000 if kw["signal"] == "literal" else 110000)
        lens = [n] * (2 if n < 8000 and rng.random() < 0.3 else 1)
    if rng.random() < 0.12:
        kw.update(granularity="block")
    elif rng.random() < 0.1 and max(lens) < 30000:
        kw.update(use_anchor=False)
    return _plain(_case("", "prefill", ",".join(map(str, lens)), planted=max(4, max(lens) // 128), **kw))


def _plain(c):
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _lens(c):
    return [int(x) for x in c["lens"].split(",")]


def _theta(c):
    return c["theta"] * (3.0 if c["signal"] == "peaked" else 1.0)


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _sequence(c, n, gen):
    """q [Hq, n, d], k, v [Hkv, n, d] of one sequence: N(0, 1) entries, per KV head a direction u that the
    queries lean to, stripe columns and sink keys planted along it."""
    d, grp, dt = c["d"], c["Hq"] // c["Hkv"], _dtype(c)
    amp = 1.0 if c["signal"] == "literal" else d ** 0.25
    gain = 3.0 if c["signal"] == "peaked" else 1.0
    rand = dict(device="cuda", generator=gen, dtype=torch.float32)
    q = torch.empty(c["Hq"], n, d, device="cuda", dtype=dt)
    k = torch.empty(c["Hkv"], n, d, device="cuda", dtype=dt)
    v = torch.empty(c["Hkv"], n, d, device="cuda", dtype=dt)
    for hk in range(c["Hkv"]):
        u = torch.randn(d, **rand)
        u = u / u.norm()
        kk = torch.randn(n, d, **rand)
        cols = torch.randperm(n, device="cuda", generator=gen)[:min(c["planted"], n)]
        mag = c["mag_lo"] + (c["mag_hi"] - c["mag_lo"]) * torch.rand(cols.numel(), **rand)
        kk[cols] += amp * gain * mag[:, None] * u
        kk[:_SINKS] += amp * gain * _SINK_MAG * u
        k[hk] = kk
        v[hk] = torch.randn(n, d, **rand)
        for h in range(hk * grp, (hk + 1) * grp):
            x = torch.randn(n, d, **rand)
            if c["ar1"]:
                rho, y = c["ar1"], x * math.sqrt(1.0 - c["ar1"] ** 2)
                x = y.clone()
                for lag in range(1, min(12, n)):
                    x[lag:] += rho ** lag * y[:-lag]
            q[h] = x + amp * u
    return q, k, v


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    parts = [_sequence(c, n, gen) for n in _lens(c)]
    if c["packed"]:
        return tuple(torch.cat([p[i] for p in parts], dim=1) for i in range(3))
    out = []
    for i in range(3):
        t = torch.stack([p[i] for p in parts])
        if c["layout"] == "token":
            t = t.transpose(1, 2).contiguous().transpose(1, 2)
        out.append(t)
    return tuple(out)


def _config(c):
    return api.Config(block=c["block"], n_init=c["n_init"], window=c["window"], step=c["step"], theta=_theta(c),
                      use_anchor=c["use_anchor"],
                      granularity=api.AA_BLOCK if c["granularity"] == "block" else api.AA_STRIPE)


def prepare(case, seed):
    c = case
    q, k, v = _inputs(c, seed)
    cu = None
    if c["packed"]:
        ends = [0]
        for n in _lens(c):
            ends.append(ends[-1] + n)
        cu = torch.tensor(ends, dtype=torch.int32, device="cuda")
    out = torch.empty_strided(q.shape, q.stride(), dtype=q.dtype, device="cuda")
    p = api.make_params(_config(c), q, k, v, out, cu_seqlens=cu, max_seqlen=max(_lens(c)))
    sizes = api.anchor_sizes(p)
    st = dict(kind=c["kind"], p=p, q=q, k=k, v=v, cu=cu, out=out)
    if c["kind"] == "stages":
        st["buf"] = api.alloc_stage_buffers(p)
        st["buf"]["idx"].zero_()
    else:
        st["lse"] = torch.empty(sizes.rows, dtype=torch.float32, device="cuda")
    if c["kind"] == "prefill":
        st["stats"] = torch.zeros(4, dtype=torch.int64, device="cuda")
        st["ws"] = torch.empty(sizes.prefill_ws_bytes, dtype=torch.uint8, device="cuda")
    return st


def run(state):
    s = state
    if s["kind"] == "prefill":
        api.anchor_attention_prefill(s["p"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["stats"], s["ws"])
        return dict(out=s["out"], lse=s["lse"], stats=s["stats"])
    if s["kind"] == "dense":
        api.dense_causal_flash(s["p"], s["q"], s["k"], s["v"], s["out"], s["lse"])
        return dict(out=s["out"], lse=s["lse"])
    b = s["buf"]
    api.anchor_compute(s["p"], s["q"], s["k"], s["v"], b["M"], b["L"], b["Acc"], b["xa"])
    api.stripe_select(s["p"], s["q"], s["k"], b["xa"], b["counts"], b["offsets"], b["idx"], b["flag"], b["ws"])
    api.sparse_attn(s["p"], s["q"], s["k"], s["v"], b["M"], b["L"], b["Acc"], b["counts"], b["offsets"], b["idx"],
                    s["out"], b["lse"])
    return dict(out=s["out"], lse=b["lse"], M=b["M"], L=b["L"], Acc=b["Acc"], xa=b["xa"], counts=b["counts"],
                offsets=b["offsets"], idx=b["idx"], flag=b["flag"])


# ------------------------------------------------------------------ what a pass cannot do without
def _pairs(c, n):
    """(anchor-region pairs, list pairs, (block, candidate) pairs) of one head of a sequence of n tokens"""
    span = c["block"] * c["step"]
    anchor = lists = cand = 0
    for g in range(-(-n // span)):
        r0, r1 = g * span, min(n, (g + 1) * span)
        w = max(c["n_init"], r0 - c["window"])
        tri = lambda m: m * (m + 1) // 2 if m > 0 else 0
        e = min(r1, c["n_init"])
        anchor += (tri(e) - tri(r0) if e > r0 else 0) + c["n_init"] * max(0, r1 - max(r0, c["n_init"]))
        anchor += tri(r1 - w) - tri(r0 - w)
        nc = w - c["n_init"]
        cand += -(-(r1 - r0) // c["block"]) * nc
        every = c["signal"] == "literal" or not c["use_anchor"]
        lists += (r1 - r0) * (nc if every else 0 if c["granularity"] == "block" else nc * min(c["planted"], n) // n)
    return anchor, lists, cand


def work(case):
    c = case
    item = 2 if c["dtype"] == "bf16" else 4
    tokens = sum(_lens(c))
    nbytes = tokens * c["d"] * item * (2 * c["Hq"] + 2 * c["Hkv"]) + tokens * c["Hq"] * 4
    if c["kind"] == "dense":
        return dict(bytes=nbytes, flops=c["Hq"] * sum(4 * c["d"] * n * (n + 1) // 2 for n in _lens(c)))
    anchor, lists, cand = (sum(x) for x in zip(*(_pairs(c, n) for n in _lens(c))))
    if c["kind"] == "stages":       # the state is the caller's: written by the first stage, read by the last
        nbytes += 2 * tokens * c["Hq"] * 4 * (c["d"] + 2)
    return dict(bytes=nbytes, flops=c["Hq"] * c["d"] * (4 * (anchor + lists) + 2 * cand))


def tolerance(case):
    """About four times the error against exact() that the kernels show over the listed cases: fp32 1.1e-6 (largest
    single difference 1.7e-5 of the root mean square), bf16 2.2e-3 (4.3e-2; probabilities and output in bf16)."""
    if case["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.0}


# ------------------------------------------------------------------ the same in 64 bits
_EXACT_PAIRS = 4e10     # (row, key) pairs that take about ten seconds


def exact(case, seed):
    c = case
    lens = _lens(c)
    per_head = sum(n * (n + 1) // 2 if c["kind"] == "dense" else sum(_pairs(c, n)[:2]) for n in lens)
    if per_head * c["Hq"] > _EXACT_PAIRS:
        return None
    q, k, v = _inputs(c, seed)
    d, block, n_init, grp = c["d"], c["block"], c["n_init"], c["Hq"] // c["Hkv"]
    dense, scale, theta = c["kind"] == "dense", 1.0 / math.sqrt(c["d"]), _theta(c)
    f64 = dict(dtype=torch.float64, device="cuda")
    out = torch.empty(q.shape, **f64)
    state = c["kind"] == "stages"
    acc_all = torch.empty(q.shape, **f64) if state else None
    rows = {"lse": [], "M": [], "L": [], "xa": []}       # per (head, sequence), joined below
    start = 0
    for b, n in enumerate(lens):
        span = 2048 if dense else block * c["step"]
        heads = {key: [] for key in rows}
        for h in range(c["Hq"]):
            sl = (h, slice(start, start + n)) if c["packed"] else (b, h)
            sk = (h // grp, slice(start, start + n)) if c["packed"] else (b, h // grp)
            Q, K, V = q[sl].double(), k[sk].double(), v[sk].double()
            O = out[sl]
            lse, M, L = torch.empty(n, **f64), torch.empty(n, **f64), torch.empty(n, **f64)
            xa = torch.empty(-(-n // block), **f64)
            for r0 in range(0, n, span):
                r1 = min(n, r0 + span)
                w = 0 if dense else max(n_init, r0 - c["window"])
                pos = torch.arange(0 if dense else min(w, r1), r1, device="cuda")
                if not dense:
                    pos = torch.cat([torch.arange(0, min(n_init, r1), device="cuda"), pos])
                r = torch.arange(r0, r1, device="cuda")
                s = (Q[r0:r1] @ K[pos].T) * scale
                s.masked_fill_(pos[None, :] > r[:, None], -math.inf)
                m = s.max(dim=1).values
                e = torch.exp(s - m[:, None])
                l, acc = e.sum(dim=1), e @ V[pos]
                if not dense:
                    M[r0:r1], L[r0:r1] = m, l
                    if state:
                        acc_all[sl][r0:r1] = acc
                    nb = -(-(r1 - r0) // block)
                    cut = torch.stack([m[i * block:(i + 1) * block].mean() for i in range(nb)])
                    xa[r0 // block:r0 // block + nb] = cut
                    if w > n_init:
                        if not c["use_anchor"]:
                            cut = torch.zeros_like(cut)
                        qbar = torch.stack([Q[r0 + i * block:min(r1, r0 + (i + 1) * block)].mean(dim=0) for i in range(nb)])
                        C = K[n_init:w]
                        if c["granularity"] == "block":
                            keep = (cut[:, None] - scale * (qbar @ C.view(-1, block, d).mean(dim=1).T) <= theta).any(dim=0)
                            keep = keep.repeat_interleave(block)
                        else:
                            keep = (cut[:, None] - scale * (qbar @ C.T) <= theta).any(dim=0)
                        sel = n_init + keep.nonzero()[:, 0]
                        if sel.numel():
                            s = (Q[r0:r1] @ K[sel].T) * scale
                            top = torch.maximum(m, s.max(dim=1).values)
                            e, down = torch.exp(s - top[:, None]), torch.exp(m - top)
                            l, acc, m = l * down + e.sum(dim=1), acc * down[:, None] + e @ V[sel], top
                O[r0:r1] = acc / l[:, None]
                lse[r0:r1] = m + torch.log(l)
            for key, x in (("lse", lse), ("M", M), ("L", L), ("xa", xa)):
                heads[key].append(x)
        for key in rows:
            rows[key].append(torch.stack(heads[key]))
        start += n
    if c["packed"]:
        flat = {key: torch.cat(x, dim=1).reshape(-1) for key, x in rows.items()}
    else:
        flat = {key: torch.stack(x).reshape(-1) for key, x in rows.items()}
    if c["kind"] == "dense":
        return dict(out=out, lse=flat["lse"])
    if c["kind"] == "prefill":
        return dict(out=out, lse=flat["lse"], stats=None)
    # Acc: per block four tiles of 32 rows, each in the order of the matrix cores' accumulators
    acc = acc_all.view(-1, 32, d // 32, 4, 2, 4).permute(0, 2, 3, 4, 1, 5).reshape(-1)
    return dict(out=out, lse=flat["lse"], M=flat["M"], L=flat["L"], Acc=acc, xa=flat["xa"], counts=None, offsets=None,
                idx=None, flag=None)
