"""The Q quantizers' codes, scales, block means and row constants where their maps can go wrong: numbers of queries around the rows of a
pass (8, 16, 32), of a wavefront and of a block, every width and both modes, against the CPU oracle byte for byte; and a value that is not a number, in Q and in K."""
import numpy as np
import pytest
import torch

from oracle import sage_oracle as so
from test_gpu_attention_from_raw_kv import _both, _inputs
from test_gpu_parity import _pa
from test_gpu_prologue_fuzz import GMAPS

pytestmark = pytest.mark.gpu
WANT = ("q_codes", "q_scale", "q_mean")


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("N", [1, 2, 7, 9, 15, 17, 32, 33, 127, 128, 131])
@pytest.mark.parametrize("d,dtype,group_map", [(64, "bf16", "lane"), (64, "fp16", "block"), (128, "fp16", "token"), (128, "bf16", "lane"), (256, "bf16", "block"), (256, "fp16", "lane")])
def test_q_codes(d, dtype, group_map, N, mode):
    pa = _pa()
    print(f"Q codes: d={d} {dtype} N={N} {group_map} {mode}", flush=True)
    q, k, v = _inputs(1, N, 70, d, 3, 1, dtype, "HND", seed=N)
    got, _, _ = pa.sage_attn_quant(q, k, v, mode=mode, group_map=group_map, want=WANT)
    torch.cuda.synchronize()
    for h in range(3):
        pro = so.quantize_head(q[0, h].float().cpu().numpy(), k[0, 0].float().cpu().numpy(), v[0, 0].float().cpu().numpy(), mode=mode, gmap=GMAPS[group_map])
        assert np.array_equal(got["q_codes"][0, h].cpu().numpy(), pro["q_codes"])
        assert np.array_equal(got["q_scale"][0, h].cpu().numpy(), pro["q_scale"][pro["q_groups"][::1 if group_map == "token" else 2]])
        if mode == "int4_fp8":
            assert np.array_equal(got["q_mean"][0, h].cpu().numpy(), pro["qbar"])


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,dtype,group_map", [(64, "bf16", "tensor"), (128, "fp16", "tensor"), (256, "bf16", "tensor"), (128, "bf16", "block"), (256, "fp16", "token"), (64, "fp16", "token")])
@pytest.mark.parametrize("N", [1, 16, 129, 300])
def test_q_codes_of_other_groups(d, dtype, group_map, N, mode):
    test_q_codes(d, dtype, group_map, N, mode)


# (token-major rows of 4096 values and 512 blocks: eight lanes a row in the 8-bit mode; a block less, and one that is all there is of a sequence)
@pytest.mark.parametrize("mode", ["int8_fp8", "int4_fp8"])
@pytest.mark.parametrize("group_map,lse", [("lane", True), ("token", False), ("block", True), ("tensor", False)])
@pytest.mark.parametrize("B,N", [(8, 3), (8, 128), (7, 128), (4, 131), (3, 300)])
def test_64_wide_heads_of_long_token_major_rows(B, N, group_map, lse, mode):
    """The bits of the same heads one after the other in memory."""
    pa = _pa()
    print(f"Q, long rows: B={B} N={N} {group_map} {mode}", flush=True)
    q, k, v = _inputs(B, N, 70, 64, 64, 4, "bf16", "HND")
    kw = dict(mode=mode, group_map=group_map, return_lse=True) if lse else dict(mode=mode, group_map=group_map)
    a = pa.sage_attn_fwd_ex(q, k, v, **kw)
    b = pa.sage_attn_fwd_ex(*(x.transpose(1, 2).contiguous() for x in (q, k, v)), layout="NHD", **kw)
    if lse:
        assert torch.equal(a[1], b[1])
        a, b = a[0], b[0]
    assert torch.isfinite(a).all() and torch.equal(a, b.transpose(1, 2))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("N", [1, 2, 7, 9, 15, 17, 32, 33, 127, 128, 131])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "fp16"), (256, "bf16")])
def test_row_constants(d, dtype, N, mode):
    """Where all keys are alike, smoothing leaves zeros: every score is 0, and the log-sum-exp of a row is ln N_kv plus its row constant, sm_scale <q, k>.
    The row constant is rounded to FP32 once, from float64 and an FP32 kappa, and then goes with a base-2 logarithm (20 at most, its offset included, of an
    instruction good to 2^-22) and 448 N_kv, a sum in FP32 of 70 terms, through a sum and a product in FP32: errors of 2^-24 of kappa <q, k> / ln 2 and
    20 each, together below 2^-20 of the two."""
    pa = _pa()
    print(f"row constants: d={d} {dtype} N={N} {mode}", flush=True)
    q, k, v = _inputs(1, N, 70, d, 3, 1, dtype, "HND", seed=N)
    k = k[:, :, :1].expand_as(k).contiguous()
    (_, whole), (_, general) = _both(pa, q, k, v, pa.make_args(q, k, v, mode=mode))         # (the whole call of few queries quantizes Q elsewhere)
    dot = (q[0].double() @ k[0, 0, 0].double()).flatten().cpu().numpy() / np.sqrt(d)
    for lse in (whole, general):
        assert (np.abs(lse.cpu().numpy() - (np.log(70.0) + dot)) <= 2.0**-20 * (np.abs(dot) + 20.0)).all()


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,N", [(64, 40), (128, 17), (256, 130)])
def test_a_value_that_is_not_a_number(d, N, mode):
    """Its code is 0, and in the 4-bit mode those of its channel (whose mean it makes NaN); all others are what they are beside a zero."""
    pa = _pa()
    print(f"Q codes, NaN: d={d} N={N} {mode}", flush=True)
    q, k, v = _inputs(1, N, 70, d, 2, 2, "bf16", "HND")
    c = d // 2 + 3
    bad = q.clone()
    bad[0, 1, N // 2, c] = float("nan")
    if mode == "int4_fp8":
        q[0, 1, :128, c] = 0.0                 # (its block of queries)
    else:
        q[0, 1, N // 2, c] = 0.0
    (a, _, _), (b, _, _) = (pa.sage_attn_quant(x, k, v, mode=mode, want=WANT) for x in (q, bad))
    torch.cuda.synchronize()
    assert torch.equal(a["q_codes"], b["q_codes"]) and torch.equal(a["q_scale"], b["q_scale"])


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("kw", [dict(), dict(delta_s="digits"), dict(group_map="token"), dict(group_map="block"), dict(group_map="tensor"), dict(smooth_k=False), dict(smooth_v=True)])
@pytest.mark.parametrize("d,Nk", [(64, 70), (128, 300), (256, 130)])
def test_a_key_that_is_not_a_number(d, Nk, kw, mode):
    """Its code is 0, and smoothed, those of its channel are; all other codes and scales are what they are beside a zero."""
    pa = _pa()
    print(f"K codes, NaN: d={d} N_kv={Nk} {kw} {mode}", flush=True)
    q, k, v = _inputs(1, 40, Nk, d, 2, 2, "bf16", "HND")
    c = d // 2 + 3
    bad = k.clone()
    bad[0, 1, Nk // 2, c] = float("nan")
    if kw.get("smooth_k", True):
        k[0, 1, :, c] = 0.0
    else:
        k[0, 1, Nk // 2, c] = 0.0
    (a, _, _), (b, _, _) = (pa.sage_attn_quant(q, x, v, mode=mode, want=("k_codes", "k_scale"), **kw) for x in (k, bad))
    torch.cuda.synchronize()
    assert int(b["k_codes"].abs().max()) <= (7 if mode == "int4_fp8" else 127)
    assert torch.equal(a["k_codes"], b["k_codes"]) and torch.equal(a["k_scale"], b["k_scale"])


@pytest.mark.parametrize("d", [64, 128, 256])
def test_a_key_that_is_not_a_number_beside_supplied_statistics(d):
    """mean(K) is finite then, and only the value itself has code 0."""
    pa = _pa()
    print(f"K codes, NaN beside supplied statistics: d={d}", flush=True)
    q, k, v = _inputs(1, 40, 200, d, 2, 2, "bf16", "HND")
    stats = pa.sage_attn_kv_stats(k, v)
    bad = k.clone()
    bad[0, 1, 77, 5] = float("nan")
    k[0, 1, 77, 5] = 0.0
    stats[0][0, 1, 5] = 0.0                       # (a zero less this mean has code 0 too)
    (a, _, _), (b, _, _) = (pa.sage_attn_quant(q, x, v, kv_stats=stats, want=("k_codes", "k_scale")) for x in (k, bad))
    torch.cuda.synchronize()
    assert torch.equal(a["k_codes"], b["k_codes"]) and torch.equal(a["k_scale"], b["k_scale"])
