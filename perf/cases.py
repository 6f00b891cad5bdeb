"""Timing cases of the quantized attention forward pass: what a user of this package has it do, through its public
entry points, from the smallest calls to the longest sequences.

A case is a plain dict; prepare() makes what the caller has in hand (tensors on the GPU, prefix sums, running
statistics, a workspace where a serving loop would keep one), run() is one call as a program makes it.

Kinds (case["kind"]):
  self      attention of a batch of equally long sequences on itself: the prefill of a language model (causal, grouped
            KV heads or not), or an encoder / diffusion model (full).  sage_attn_fwd_ex with its defaults: output and
            workspace come from torch's allocator.
  static    the same, small, from a latency-bound loop: output kept, sage_attn_fwd_static.
  chunk     a chunk of new queries against a longer KV cache in token-major layout, log-sum-exp wanted (chunked prefill,
            merging with other key sets).
  decode    one or a few new queries per sequence against a long cache, everything read as it is.
  serve     the decode step of a serving loop: output and workspace kept, mean(K) and delta_V supplied by the keeper of
            the cache (sage_attn_kv_stats / sage_attn_kv_stats_update).
  first     the first chunk of a growing cache: its running statistics are started from it
            (sage_attn_kv_stats_update) and its attention uses them.
  varlen    a packed batch of sequences of different lengths.
"""
import math

import torch

import paper_2411_10958_amd as sage

# B, H, H_kv, N, N_kv, d: batch, query heads, KV heads, queries, keys, head dimension; "lens": the sequence lengths of a
# packed batch.  spread > 1: token norms vary log-uniformly over [1, spread] (video); v_bias: channel-wise bias of V.
_BASE = dict(kind="self", B=1, H=32, H_kv=32, N=0, N_kv=0, d=128, dtype="bf16", causal=True, mode="int4_fp8", layout="HND",
             smooth_v=False, lens="", spread=1.0, v_bias=0.0)


def _case(name, **kw):
    c = dict(_BASE, **kw)
    c["N_kv"] = c["N_kv"] or c["N"]
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest configuration of workloads/: launches and host time are all there is
        _case("tiny", H=2, H_kv=2, N=256, d=64, dtype="fp16", causal=False),
        # one short prompt of a chat model (grouped KV heads, token-major as a fused QKV projection leaves it) in a
        # loop that may not allocate
        _case("short_prompt_static", kind="static", H_kv=8, N=300, layout="NHD"),
        # a batch of short prompts (the short end of the speed-over-length table)
        _case("causal1k", B=4, N=1024),
        # language-model prefill, the paper's kernel-benchmark shape and bench.py's workload
        _case("prefill4k", B=4, N=4096, causal=False),
        # the causal sweep of bench.py, 8-bit mode
        _case("causal8k_int8", N=8192, mode="int8_fp8"),
        # the 256-wide heads of workloads/
        _case("causal8k_d256", H=16, H_kv=16, N=8192, d=256),
        # video diffusion: ragged length, d = 64, varying token norms, biased V channels with the smooth-V option
        _case("video17k_vbias", B=2, H=48, H_kv=48, N=17776, d=64, causal=False, smooth_v=True, spread=8.0, v_bias=8.5),
        # the longest configuration: long-context prefill with grouped KV heads
        _case("long128k", H_kv=8, N=131072),
        # a chunk of 512 new tokens against a 16k cache
        _case("chunk512_16k", kind="chunk", B=2, H_kv=8, N=512, N_kv=16384, layout="NHD"),
        # one decode step against a 32k cache, everything read as it is
        _case("decode32k", kind="decode", B=4, H_kv=8, N=1, N_kv=32768),
        # the decode step of a serving loop with odd cache length, fp16, 8-bit mode, statistics kept
        _case("serve_decode5k_int8", kind="serve", B=16, H_kv=8, N=1, N_kv=5003, dtype="fp16", mode="int8_fp8", layout="NHD"),
        # a packed batch of prompts of mixed lengths
        _case("varlen_fp16", kind="varlen", B=8, H_kv=8, dtype="fp16", lens="2048,37,1501,4096,777,128,3333,1"),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], even over the logarithm; two times in three as it comes (odd and ragged sizes), else a
    multiple of 64 where there is one."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if n >= 128 and rng.random() < 1 / 3:
        n = n // 64 * 64
    return max(lo, min(hi, n))


def draw(rng):
    kind = rng.choice(["self", "self", "self", "static", "chunk", "decode", "serve", "first", "varlen"])
    d = rng.choice([64, 128, 128, 128, 256])
    G = rng.choice([1, 1, 2, 4, 8])
    H = G * rng.choice([2, 4, 5, 8] if kind == "static" else [1, 2, 4, 6, 8])
    c = dict(kind=kind, H=H, H_kv=H // G, d=d, dtype=rng.choice(["bf16", "bf16", "fp16"]),
             mode=rng.choice(["int4_fp8", "int4_fp8", "int8_fp8"]), layout=rng.choice(["HND", "NHD"]))
    if kind == "static":                    # what fits the built-in workspace
        c.update(N=_log_int(rng, 16, 640), causal=rng.random() < 0.7)
    elif kind in ("self", "first"):
        c.update(N=_log_int(rng, 100, 40000), B=rng.randint(1, 4), causal=kind == "first" or rng.random() < 0.6)
        if kind == "self" and not c["causal"] and rng.random() < 0.4:
            c.update(smooth_v=True, spread=8.0, v_bias=8.5)
    elif kind == "chunk":
        c.update(N=_log_int(rng, 64, 2048), B=rng.randint(1, 2))
        c.update(N_kv=c["N"] + _log_int(rng, 256, 40000))
    elif kind in ("decode", "serve"):
        c.update(N=rng.choice([1, 1, 1, 2, 4]), B=_log_int(rng, 1, 32))
        c.update(N_kv=_log_int(rng, 200, 65536))
        while c["B"] > 1 and c["B"] * c["N_kv"] * c["H_kv"] * d > 1 << 30:
            c["B"] //= 2
    else:
        lens = [_log_int(rng, 1, 6000) for _ in range(rng.randint(2, 12))]
        c.update(B=len(lens), lens=",".join(map(str, lens)))
    c = _case("", **c)
    while work(c)["flops"] > 4e13:          # well below the largest listed case
        c["B"], c["N"], c["N_kv"] = 1, c["N"] * 3 // 4, c["N_kv"] * 3 // 4
    return c


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _qk(g, shape, case, dt, tok, chan):
    """Token noise (times a token norm for the video recipe) plus a per-channel offset that all tokens of a head
    share, ten times larger in four channels: the channel-wise outliers that the smoothing is for (the recipe of
    workloads/inputs.py).  tok, chan: the shapes that broadcast over everything but tokens / but heads and channels."""
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    std = 3.0
    if case["spread"] > 1.0:
        x *= torch.exp(torch.rand(tok, generator=g, device="cuda") * math.log(case["spread"]))
        std = 4.0
    off = torch.randn(chan, generator=g, device="cuda") * std
    if case["spread"] == 1.0:
        pick = torch.rand(chan, generator=g, device="cuda").argsort(dim=-1) < 4
        off = torch.where(pick, off * 10.0, off)
    return x.add_(off).to(dt)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float16
    B, H, Hkv, N, Nk, d = (case[n] for n in ("B", "H", "H_kv", "N", "N_kv", "d"))
    if case["kind"] == "varlen":
        lens = _lens(case)
        total = sum(lens)
        def shapes(h, n):
            return (total, h, d), (total, h, 1), (1, h, d)
    elif case["layout"] == "NHD":
        def shapes(h, n):
            return (B, n, h, d), (B, n, h, 1), (B, 1, h, d)
    else:
        def shapes(h, n):
            return (B, h, n, d), (B, h, n, 1), (B, h, 1, d)
    q = _qk(g, shapes(H, N)[0], case, dt, *shapes(H, N)[1:])
    k = _qk(g, shapes(Hkv, Nk)[0], case, dt, *shapes(Hkv, Nk)[1:])
    v = torch.randn(shapes(Hkv, Nk)[0], generator=g, device="cuda", dtype=torch.float32)
    if case["v_bias"] > 0:
        chan = shapes(Hkv, Nk)[2]
        sign = torch.where(torch.rand(chan, generator=g, device="cuda") < 0.5, -1.0, 1.0)
        v += sign * (case["v_bias"] - 0.5 + torch.rand(chan, generator=g, device="cuda"))
    s = dict(q=q, k=k, v=v.to(dt), kind=case["kind"],
             kw=dict(causal=case["causal"], mode=case["mode"], smooth_v=case["smooth_v"], layout=case["layout"]))
    if case["kind"] == "varlen":
        cu = torch.zeros(len(lens) + 1, dtype=torch.int32)
        cu[1:] = torch.tensor(lens, dtype=torch.int32).cumsum(0)
        s["kw"].pop("layout")
        s["kw"].update(cu_seqlens_q=cu.cuda(), max_seqlen_q=max(lens), max_seqlen_k=max(lens))
    if case["kind"] in ("static", "serve"):
        s["out"] = torch.empty_like(q)
    if case["kind"] == "serve":
        s["kw"]["kv_stats"] = sage.sage_attn_kv_stats(k, s["v"], layout=case["layout"])
        a = sage.make_args(q, k, s["v"], s["out"], **s["kw"])
        s["kw"]["workspace"] = torch.empty(sage.sage_attn_workspace_bytes(a), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    q, k, v, kw = s["q"], s["k"], s["v"], s["kw"]
    if s["kind"] == "static":
        return sage.sage_attn_fwd_static(q, k, v, s["out"], **kw)
    if s["kind"] == "serve":
        return sage.sage_attn_fwd_ex(q, k, v, out=s["out"], **kw)
    if s["kind"] == "first":
        k_mean, v_scale, state = sage.sage_attn_kv_stats_update(k, v, None, layout=kw["layout"])
        out = sage.sage_attn_fwd_ex(q, k, v, kv_stats=(k_mean, v_scale), **kw)
        return out, k_mean, v_scale, state[0], state[1]
    if s["kind"] in ("chunk", "varlen", "decode"):
        return sage.sage_attn_fwd_ex(q, k, v, return_lse=True, **kw)
    return sage.sage_attn_fwd_ex(q, k, v, **kw)


def _pairs(n, nk, causal):
    """Visible (query, key) pairs of one head."""
    return n * (2 * nk - n + 1) / 2 if causal else n * nk


def work(case):
    """Inputs read once, outputs written once; two products of 2 d operations per visible (query, key) pair."""
    H, Hkv, d = case["H"], case["H_kv"], case["d"]
    if case["kind"] == "varlen":
        tq = tk = sum(_lens(case))
        pairs = sum(_pairs(n, n, case["causal"]) for n in _lens(case))
    else:
        tq, tk = case["B"] * case["N"], case["B"] * case["N_kv"]
        pairs = case["B"] * _pairs(case["N"], case["N_kv"], case["causal"])
    nbytes = 2 * d * (2 * tq * H + 2 * tk * Hkv)
    if case["kind"] in ("chunk", "varlen", "decode"):
        nbytes += 4 * tq * H                                    # the log-sum-exp
    if case["kind"] == "first":
        nbytes += case["B"] * Hkv * d * (4 + 4 + 8 + 4)         # statistics and their state
    if case["kind"] == "serve":
        nbytes += case["B"] * Hkv * d * 8
    return {"bytes": nbytes, "flops": 4.0 * H * d * pairs}


def tolerance(case):
    """P~ is quantized to 8 bits under the running maximum of the keys it is summed with, so the same call with its key
    range summed in another order - whole, or in 3 or 8 chunks (kv_splits) that are merged - gives other codes of P~:
    measured on these cases, up to 7.3e-3 of the output's norm and 0.13 of its root mean square (bf16 and fp16, both
    modes, self attention to decode).  About three times that is allowed.  (Delta-S summed in FP32 instead of exactly
    moves less: 2.2e-4 and 0.09.)"""
    return {"rel": 0.02, "max": 0.4}


def _attend64(q, k, v, scale, causal):
    """Plain attention of one head in float64, and its log-sum-exp; 2048 queries at a time."""
    n, nk = q.shape[0], k.shape[0]
    out, lse = torch.empty_like(q), torch.empty(n, dtype=torch.float64, device=q.device)
    kt = k.t().contiguous()
    for i in range(0, n, 2048):
        s = torch.matmul(q[i:i + 2048], kt).mul_(scale)
        if causal:
            row = torch.arange(i, i + s.shape[0], device=q.device)[:, None]
            s.masked_fill_(torch.arange(nk, device=q.device)[None, :] > row + (nk - n), -math.inf)
        lse[i:i + 2048] = torch.logsumexp(s, 1)
        out[i:i + 2048] = torch.matmul(s.sub_(lse[i:i + 2048, None]).exp_(), v)
    return out, lse


def exact(case, seed):
    """What run() returns if nothing is quantized: attention, log-sum-exp and running statistics in float64.  The 4-bit
    codes alone are 0.07 to 0.11 off that (measured: 0.098 on prefill4k, 0.11 on causal8k_d256); where they may pass a
    tenth - long rows, wide heads - the attention output has no value to be held to."""
    if work(case)["flops"] > 3e13:
        return None
    noisy = case["mode"] == "int4_fp8" and case["kind"] != "decode" and (case["d"] == 256 or case["N_kv"] > 4096)
    s = prepare(case, seed)
    q, k, v = (s[n].double() for n in ("q", "k", "v"))
    H, G, scale = case["H"], case["H"] // case["H_kv"], 1 / math.sqrt(case["d"])
    out = torch.empty_like(q)
    if case["kind"] == "varlen":
        lse = torch.empty(H, q.shape[0], dtype=torch.float64, device="cuda")
        a = 0
        for n in _lens(case):
            for h in range(H):
                t = slice(a, a + n)
                out[t, h], lse[h, t] = _attend64(q[t, h], k[t, h // G], v[t, h // G], scale, case["causal"])
            a += n
        return None if noisy else out, lse
    if case["layout"] == "NHD":
        q, k, v = (x.transpose(1, 2) for x in (q, k, v))
    o = out.transpose(1, 2) if case["layout"] == "NHD" else out
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device="cuda")
    for b in range(case["B"]):
        for h in range(H):
            o[b, h], lse[b, h] = _attend64(q[b, h], k[b, h // G], v[b, h // G], scale, case["causal"])
    if case["kind"] in ("chunk", "decode"):
        return None if noisy else out, lse
    if case["kind"] == "first":
        vmax = v.abs().amax(2)
        return None if noisy else out, k.mean(2), vmax / 448, k.sum(2), vmax
    return None if noisy else out
