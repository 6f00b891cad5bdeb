"""Calls whose queries of a KV head fit 32 columns are served by a kernel that quantizes K and V itself, by the rule of
attention_raw_ok (csrc/sage_attn_raw.hip).  sage_attn_prologue + sage_attn_core always take the general path, so
the two can be compared on the same arguments: same codes, scales, chunks and order of every sum, so the same bits."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import parity

pytestmark = pytest.mark.gpu


def _pa():
    import paper_2411_10958_amd as pa
    pa.load_library()
    return pa


def _inputs(B, N, Nk, d, H, Hkv, dtype, layout, seed=0):
    spec = wl.WorkloadSpec("raw", B, H, Hkv, N, d, dtype, True, 3.0, 1.5, 2, 10.0, 1.0, 77, 0.0, Nk)
    data = wl.make_inputs(spec, seed)
    q, k, v = (wl.to_torch(data[n], dtype, torch.device("cuda:0")) for n in "qkv")
    if layout == "NHD":
        q, k, v = (x.transpose(1, 2).contiguous() for x in (q, k, v))
    return q, k, v


def _both(pa, q, k, v, args):
    """(out, lse) of the call as a whole and of its two halves (the general path)."""
    lib, res = pa.load_library(), []
    ws = torch.empty(pa.sage_attn_workspace_bytes(args), dtype=torch.uint8, device="cuda")
    for whole in (True, False):
        out = torch.full_like(q, 3.0)
        lse = torch.full((args.B * args.H * args.N,), 5.0, dtype=torch.float32, device="cuda")
        args.out, args.lse, args.workspace, args.workspace_bytes = out.data_ptr(), lse.data_ptr(), ws.data_ptr(), ws.numel()
        if whole:
            assert lib.sage_attn_fwd_ex(ctypes.byref(args)) == 0
        else:
            assert lib.sage_attn_prologue(ctypes.byref(args)) == 0 and lib.sage_attn_core(ctypes.byref(args)) == 0
        torch.cuda.synchronize()
        res.append((out, lse))
    return res


def _compare(res):
    (a, la), (b, lb) = res
    assert torch.isfinite(a).all()
    assert torch.equal(a, b), f"{int((a != b).sum())} of {a.numel()} outputs differ"
    assert torch.equal(la, lb), f"{int((la != lb).sum())} of {la.numel()} log-sum-exps differ"


# B, N, N_kv, d, dtype, H, Hkv, causal, layout, kv_splits: the fewest keys; block and group edges (63, 64, 65, 16 n + 1); one
# to eight heads in a group (four at a time in the Delta-S product); all 32 columns; split and unsplit, asked for and not
CASES = [
    (96, 1, 1, 128, "bf16", 1, 1, True, "HND", 0),
    (48, 1, 63, 64, "fp16", 4, 2, True, "NHD", 0),
    (100, 2, 64, 128, "bf16", 5, 1, True, "HND", 0),
    (96, 4, 65, 256, "bf16", 8, 1, True, "NHD", 0),
    (48, 32, 145, 128, "fp16", 2, 2, True, "NHD", 0),
    (96, 32, 300, 64, "bf16", 1, 1, False, "HND", 1),
    (24, 1, 1041, 128, "bf16", 8, 2, True, "HND", 0),
    (16, 3, 2000, 256, "fp16", 6, 2, False, "NHD", 3),
    (48, 5, 1500, 64, "bf16", 6, 1, True, "NHD", 2),
    (11, 1, 1999, 128, "fp16", 3, 3, True, "NHD", 0),
    (24, 2, 1300, 128, "bf16", 8, 4, False, "HND", 0),
    (96, 1, 777, 128, "fp16", 3, 1, False, "NHD", 1),
    (50, 4, 520, 256, "fp16", 4, 2, True, "HND", 1),
]


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,dtype,H,Hkv,causal,layout,splits", CASES)
def test_equals_the_general_path(B, N, Nk, d, dtype, H, Hkv, causal, layout, splits, mode):
    pa = _pa()
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, dtype, layout)
    if Nk > 300:
        v[..., 3] = 0.0                       # an all-zero channel: scale 0
        k.view(-1)[: 16 * d * (Hkv if layout == "NHD" else 1)] *= 64.0      # one loud group of keys
    a = pa.make_args(q, k, v, None, causal=causal, mode=mode, layout=layout, kv_splits=splits)
    print(f"raw K, V: B={B} N={N} N_kv={Nk} d={d} {dtype} H={H}/{Hkv} causal={causal} {layout} {mode} "
          f"splits={pa.sage_attn_kv_splits(a)}", flush=True)
    assert B * Hkv * pa.sage_attn_kv_splits(a) >= 96
    _compare(_both(pa, q, k, v, a))


@pytest.mark.parametrize("special", ["", "nan key", "zero query", "loud query"])
@pytest.mark.parametrize("B,Nk,d,dtype,H,Hkv,causal,layout,splits", [(40, 129, 64, "bf16", 8, 2, True, "NHD", 0), (100, 640, 128, "fp16", 4, 1, False, "HND", 1),
                                                                     (20, 1999, 128, "bf16", 10, 2, True, "HND", 0), (64, 65, 256, "fp16", 8, 1, True, "NHD", 0),
                                                                     (24, 1000, 256, "bf16", 4, 4, False, "HND", 2)])
def test_one_query_in_the_4_bit_mode_equals_the_general_path(B, Nk, d, dtype, H, Hkv, causal, layout, splits, special):
    """A single query's codes are all zero, and the kernel for it forms neither them nor K's."""
    pa = _pa()
    q, k, v = _inputs(B, 1, Nk, d, H, Hkv, dtype, layout, 3)
    print(f"raw K, V, one query: B={B} N_kv={Nk} d={d} {dtype} H={H}/{Hkv} causal={causal} {layout} {special}", flush=True)
    if special == "nan key":
        k.view(-1)[(Nk // 2) * d * (Hkv if layout == "NHD" else 1) + 5] = float("nan")
    elif special:
        q *= 0.0 if special == "zero query" else 64.0
    a = pa.make_args(q, k, v, None, causal=causal, mode="int4_fp8", layout=layout, kv_splits=splits)
    assert B * Hkv * pa.sage_attn_kv_splits(a) >= 64
    (x, lx), (y, ly) = _both(pa, q, k, v, a)
    assert torch.equal(x.isnan(), y.isnan()) and bool(x.isnan().any()) == (special == "nan key")
    assert torch.equal(x.nan_to_num(0.5), y.nan_to_num(0.5)) and torch.equal(lx.nan_to_num(0.5), ly.nan_to_num(0.5))


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("B,Nk,d,dtype,H,Hkv,layout,splits", [(40, 129, 64, "bf16", 8, 2, "NHD", 0), (100, 640, 128, "fp16", 4, 1, "HND", 1),
                                                              (24, 1000, 256, "bf16", 4, 4, "HND", 2)])
def test_one_query_and_a_key_that_is_not_finite(B, Nk, d, dtype, H, Hkv, layout, splits, value):
    """With the statistics supplied an infinite key leaves mean(K) finite: the general path's scale of the key's group is infinite and its
    rows NaN, and so they are where no codes are formed."""
    pa = _pa()
    q, k, v = _inputs(B, 1, Nk, d, H, Hkv, dtype, layout, 3)
    print(f"raw K, V, one query, a key of {value}: B={B} N_kv={Nk} d={d} {dtype} H={H}/{Hkv} {layout}", flush=True)
    stats = pa.sage_attn_kv_stats(k, v, layout=layout)
    (k if layout == "HND" else k.transpose(1, 2))[1, 0, Nk // 2, 5] = value
    (x, lx), (y, ly) = _both(pa, q, k, v, pa.make_args(q, k, v, None, mode="int4_fp8", layout=layout, kv_splits=splits, kv_stats=stats))
    hit = (x if layout == "HND" else x.transpose(1, 2))[1, :H // Hkv]
    assert bool(hit.isnan().all()) and int(x.isnan().sum()) == hit.numel() and int(lx.isnan().sum()) == H // Hkv
    assert torch.equal(x.isnan(), y.isnan()) and torch.equal(lx.isnan(), ly.isnan())
    assert torch.equal(x.nan_to_num(0.5), y.nan_to_num(0.5)) and torch.equal(lx.nan_to_num(0.5), ly.nan_to_num(0.5))


# the lines of raw_reduces: chunks of 256 keys times channels, bytes of K and V; last: whether the kernel reduces the statistics itself
REDUCE_CASES = [(1, 65536, 64, 2, 2, True), (1, 65537, 64, 2, 2, False), (1, 32768, 128, 4, 1, True), (1, 32769, 128, 4, 1, False), (2, 8192, 256, 1, 1, True),
                (2, 8193, 256, 1, 1, False), (32, 4096, 128, 4, 4, True), (32, 4097, 128, 4, 4, False), (64, 2, 128, 4, 1, True), (64, 257, 256, 2, 2, True)]


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,Nk,d,H,Hkv,reduces", REDUCE_CASES)
def test_statistics_reduced_in_the_kernel_or_before(B, Nk, d, H, Hkv, reduces, mode):
    pa = _pa()
    print(f"raw K, V, statistics: B={B} N_kv={Nk} d={d} H={H}/{Hkv} {mode}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(Nk + d)
    q, k, v = (torch.randn(B, h, n, d, generator=gen, device="cuda").add_(0.5).half() for h, n in ((H, 2), (Hkv, Nk), (Hkv, Nk)))
    for splits in ((0, 1) if B * Hkv >= 64 else (0,)):           # (in several chunks, and in one)
        _compare(_both(pa, q, k, v, pa.make_args(q, k, v, None, causal=True, mode=mode, kv_splits=splits)))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
def test_packed_batch_equals_the_general_path(mode):
    """Sequences without queries, without keys, with fewer keys than queries, and of very different lengths."""
    pa = _pa()
    lens_q, lens_k, d, H, Hkv = [1, 0, 8, 3, 2] * 10, [700, 90, 5, 0, 1300] * 10, 128, 8, 2
    cu = [torch.tensor([0] + list(torch.tensor(x).cumsum(0)), dtype=torch.int32, device="cuda") for x in (lens_q, lens_k)]
    q, _, _ = _inputs(1, sum(lens_q), sum(lens_q), d, H, Hkv, "bf16", "NHD")
    _, k, v = _inputs(1, 1, sum(lens_k), d, H, Hkv, "bf16", "NHD", 1)
    q, k, v = q[0], k[0], v[0]
    a = pa.make_varlen_args(q, k, v, None, *cu, max(lens_q), max(lens_k), causal=True, mode=mode)
    print(f"raw K, V: packed batch {lens_q[:5]} / {lens_k[:5]}, ten times, {mode}", flush=True)
    _compare(_both(pa, q, k, v, a))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,causal,layout", [(128, True, "NHD"), (128, False, "HND"), (256, True, "HND"), (64, False, "NHD")])
def test_long_chunks_equal_the_general_path(d, causal, layout, mode):
    """One chunk of thousands of keys per workgroup: 79 blocks through the double buffer and the rescaled accumulator."""
    pa = _pa()
    B, H, Hkv, Nk = 24, 8, 4, 5003
    gen = torch.Generator(device="cuda").manual_seed(d + causal)
    def tensor(heads, n, std, offset):
        shape = (B, heads, n, d) if layout == "HND" else (B, n, heads, d)
        chan = (1, heads, 1, d) if layout == "HND" else (1, 1, heads, d)
        x = std * torch.randn(shape, generator=gen, device="cuda") + offset * torch.randn(chan, generator=gen, device="cuda")
        return x.to(torch.bfloat16)
    q, k, v = tensor(H, 1, 3.0, 1.5), tensor(Hkv, Nk, 3.0, 3.0), tensor(Hkv, Nk, 1.0, 0.0)
    a = pa.make_args(q, k, v, None, causal=causal, mode=mode, layout=layout, kv_splits=1)
    print(f"raw K, V, one chunk of {Nk} keys: d={d} causal={causal} {layout} {mode}", flush=True)
    _compare(_both(pa, q, k, v, a))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
def test_scales_at_the_ends_of_the_range(mode):
    """Scales outside the range of the quick division (subnormal ones too): the exact division takes over, for eight channels of
    V together (a thread's), for a wavefront's 16 keys and for a wavefront's queries."""
    pa = _pa()
    q, k, v = _inputs(96, 1, 200, 128, 2, 1, "bf16", "HND")
    for i, e in enumerate((-70, 60, 100, -125)):
        v[..., 8 * i: 8 * i + 8] *= 2.0 ** e
    v[..., 32] *= 2.0 ** -90                  # one channel of eight
    k[::3] *= 2.0 ** -70
    q[1::3] *= 2.0 ** -70
    _compare(_both(pa, q, k, v, pa.make_args(q, k, v, None, causal=True, mode=mode)))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,dtype,H,Hkv,causal,layout,splits", [
    (48, 1, 1100, 128, "bf16", 8, 2, False, "HND", 2), (96, 2, 300, 128, "fp16", 4, 1, True, "NHD", 1),
    (48, 4, 600, 256, "bf16", 4, 2, True, "HND", 1), (50, 16, 1041, 64, "fp16", 2, 1, False, "NHD", 0),
])
def test_matches_the_oracle(B, N, Nk, d, dtype, H, Hkv, causal, layout, splits, mode):
    """The first and the last sequence of a batch against Algorithm 1 walking the same key chunks."""
    pa = _pa()
    spec = wl.WorkloadSpec("raw", B, H, Hkv, N, d, dtype, causal, 3.0, 1.5, 2, 10.0, 1.0, 77, 0.0, Nk)
    data = wl.make_inputs(spec, 3)
    q, k, v = (wl.to_torch(data[n], dtype, torch.device("cuda:0")) for n in "qkv")
    if layout == "NHD":
        q, k, v = (x.transpose(1, 2).contiguous() for x in (q, k, v))
    kw = dict(causal=causal, mode=mode, layout=layout, kv_splits=splits)
    S = pa.sage_attn_kv_splits(pa.make_args(q, k, v, None, **kw))
    print(f"raw K, V against the oracle: B={B} N={N} N_kv={Nk} d={d} {dtype} H={H}/{Hkv} causal={causal} {layout} {mode} splits={S}", flush=True)
    assert B * Hkv * S >= 96
    out, lse = pa.sage_attn_fwd_ex(q, k, v, return_lse=True, **kw)
    torch.cuda.synchronize()
    ends = [0, B - 1]
    got = wl.from_torch((out.transpose(1, 2) if layout == "NHD" else out)[ends].contiguous())
    pros = parity.check_heads(got, {n: data[n][ends] for n in "qkv"}, causal, mode, dtype, want_lse=True, splits=S)
    for i, b in enumerate(ends):
        for h in range(H):
            # (the bar of the log-sum-exp elsewhere: a few FP32 operations on its largest term)
            pro, ref = pros[i][h], pros[i][h]["lse"].astype(np.float64)
            corr = np.log(2.0) * float(pro["kappa"]) * (pro["Q"].astype(np.float64) @ pro["kbar"].astype(np.float64))
            big = np.maximum(np.maximum(np.abs(ref), np.abs(corr)), np.maximum(np.abs(ref - corr), 1.0))
            assert (np.abs(lse[b, h].cpu().numpy() - ref) <= 1e-5 * big + 1e-5).all()


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,H,Hkv", [(64, 2, 2), (128, 2, 1), (128, 8, 1), (256, 2, 1)])
def test_sequence_of_a_packed_batch_equals_the_sequence_alone(d, H, Hkv, mode):
    """Bit for bit at the same kv_splits, whichever kernel the number of sequences leads to: 100 decode steps together are
    served from raw K and V, one of them alone is not.  The inputs make the order of float64 sums visible: <q, k> is 2^14,
    plus half a unit of its last FP32 place, plus terms that a float64 sum of 2^14 keeps only if they meet each other first, at
    random channels.  Even sequences carry them in Delta-S (keys 1 and -1, so mean(K) = 0), odd ones in the row constant of
    the log-sum-exp (all keys 1, so mean(K) = 1).  sm_scale = ln 2 makes kappa 1."""
    pa = _pa()
    B, nk = 100, 8
    gen = torch.Generator().manual_seed(d + H)
    q = torch.zeros(B, H, d, dtype=torch.float64)
    for b in range(B):
        for h in range(H):
            c = torch.randperm(d, generator=gen)
            q[b, h, c[0]], q[b, h, c[1]] = 2.0 ** 14, 2.0 ** -10
            n_tiny = int(torch.randint(d // 8, d - 1, (1,), generator=gen))
            q[b, h, c[2: 2 + n_tiny]] = 2.0 ** -torch.randint(41, 46, (n_tiny,), generator=gen).double()
    k = torch.ones(B, nk, Hkv, d)
    k[::2, 1::2] = -1.0
    v = torch.randn(B, nk, Hkv, d, generator=gen)
    q, k, v = (x.to(torch.bfloat16).cuda() for x in (q, k, v))
    cu_q = torch.arange(B + 1, dtype=torch.int32, device="cuda")
    kw = dict(causal=True, mode=mode, sm_scale=0.69314718, kv_splits=1, return_lse=True)
    print(f"packed batch and its sequences: d={d} H={H}/{Hkv} {mode}", flush=True)
    out, lse = pa.sage_attn_fwd_ex(q, k.reshape(-1, Hkv, d), v.reshape(-1, Hkv, d), cu_seqlens_q=cu_q, cu_seqlens_k=cu_q * nk,
                                   max_seqlen_q=1, max_seqlen_k=nk, **kw)
    for b in range(B):
        one, one_lse = pa.sage_attn_fwd_ex(q[b][None, None], k[b][None], v[b][None], layout="NHD", **kw)
        torch.cuda.synchronize()
        assert torch.equal(one[0], out[b:b + 1]), f"sequence {b}"
        assert torch.equal(one_lse[0, :, 0], lse[:, b]), f"sequence {b}: {(one_lse[0, :, 0] - lse[:, b]).tolist()}"
