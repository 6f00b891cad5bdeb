"""The Delta-S product of few key blocks and many block means, shared between several workgroups per key block (k_parts in csrc/sage_prologue.hip): a value
does not depend on the step it is formed in, so every query head of a KV head has the bits it has in a call of its own (one step, one workgroup)."""
import numpy as np
import pytest
import torch

from launch_recorder import launches
from paper_2411_10958_amd.binding import _GROUPS
from test_gpu_attention_from_raw_kv import _inputs
from test_gpu_parity import _pa

# N, N_kv, d, H, Hkv, dtype, causal, layout, workgroups per key block: parts that end within a head and at one, heads shorter than a step, a ragged
# end of both, keys that few or no query blocks see, the short sequence of launches and the long one
CASES = [(2000, 2000, 128, 8, 1, "bf16", True, "HND", 2), (2049, 2049, 64, 16, 2, "fp16", True, "NHD", 2), (130, 900, 128, 64, 1, "bf16", False, "HND", 2), (1000, 1000, 64, 64, 1, "bf16", True, "HND", 8),
         (1281, 5000, 128, 48, 3, "bf16", True, "HND", 2), (4100, 4100, 256, 8, 1, "bf16", True, "HND", 4), (700, 5000, 256, 64, 2, "fp16", False, "NHD", 3)]


@pytest.mark.parametrize("N,Nk,d,H,Hkv,dtype,causal,layout,parts", CASES)
def test_the_launch_has_them(N, Nk, d, H, Hkv, dtype, causal, layout, parts):
    (status, seq), = launches([("sage_attn_fwd_ex", dict(B=1, H=H, H_kv=Hkv, N=N, N_kv=Nk, d=d, dtype=1, mode=0, layout=int(layout == "NHD"), causal=int(causal), kv_splits=1))])
    assert status == 0
    assert [x.grid[2] for x in seq if x.kernel in ("k_quant_kv", "k_quant_k")] == [parts]


@pytest.mark.gpu
@pytest.mark.parametrize("N,Nk,d,H,Hkv,dtype,causal,layout,parts", CASES)
def test_every_head_has_the_bits_of_a_call_of_its_own(N, Nk, d, H, Hkv, dtype, causal, layout, parts):
    pa = _pa()
    print(f"parts of Delta-S: N={N} N_kv={Nk} d={d} H={H}/{Hkv} {dtype} causal={causal} {layout} parts={parts}", flush=True)
    q, k, v = _inputs(1, N, Nk, d, H, Hkv, dtype, layout)
    kw = dict(causal=causal, layout=layout, kv_splits=1, delta_s="digits", return_lse=True)
    hd = 2 if layout == "NHD" else 1
    out, lse = pa.sage_attn_fwd_ex(q, k, v, **kw)
    short, _ = pa.sage_attn_fwd_ex(q, k, v, **dict(kw, return_lse=False)), None
    assert torch.isfinite(out).all() and torch.equal(out, short)
    for h in sorted({0, 1, H // 2, H - 2, H - 1}):
        g = h // (H // Hkv)
        o, l = pa.sage_attn_fwd_ex(q.narrow(hd, h, 1).contiguous(), k.narrow(hd, g, 1).contiguous(), v.narrow(hd, g, 1).contiguous(), **kw)
        assert torch.equal(o, out.narrow(hd, h, 1)) and torch.equal(l, lse.narrow(1, h, 1)), h


# B, then as above, and the groups of scales: more than one sequence, workgroups numbered heads first (token-major rows of 4096 values), a scale per key and per block
MORE = [(3, 1100, 1100, 128, 16, 1, "bf16", True, "HND", "lane", 2), (2, 1500, 2100, 64, 32, 2, "fp16", False, "NHD", "token", 3), (2, 2049, 2049, 128, 16, 2, "bf16", True, "NHD", "block", 2),
        (1, 1540, 300, 128, 512, 32, "bf16", False, "NHD", "lane", 3), (1, 2100, 2100, 256, 256, 16, "fp16", True, "NHD", "token", 2), (2, 2000, 2000, 256, 16, 1, "bf16", True, "HND", "token", 4)]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,dtype,causal,layout,group_map,parts", MORE)
def test_the_launch_has_them_too(B, N, Nk, d, H, Hkv, dtype, causal, layout, group_map, parts):
    (status, seq), = launches([("sage_attn_fwd_ex", dict(B=B, H=H, H_kv=Hkv, N=N, N_kv=Nk, d=d, dtype=1, mode=0, layout=int(layout == "NHD"), causal=int(causal), kv_splits=1,
                                                         group_map=_GROUPS[group_map]))])
    assert status == 0
    assert [x.grid[2] for x in seq if x.kernel in ("k_quant_kv", "k_quant_k")] == [parts]


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,dtype,causal,layout,group_map,parts", MORE)
def test_every_sequence_and_head_has_the_bits_of_a_call_of_its_own(B, N, Nk, d, H, Hkv, dtype, causal, layout, group_map, parts):
    pa = _pa()
    print(f"parts of Delta-S: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {dtype} causal={causal} {layout} {group_map} parts={parts}", flush=True)
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, dtype, layout)
    kw = dict(causal=causal, layout=layout, kv_splits=1, delta_s="digits", return_lse=True, group_map=group_map)
    hd = 2 if layout == "NHD" else 1
    out, lse = pa.sage_attn_fwd_ex(q, k, v, **kw)
    for b in range(B):
        for h in sorted({0, 1, H // 2, H - 1}):
            g = h // (H // Hkv)
            o, l = pa.sage_attn_fwd_ex(*(x[b:b + 1].narrow(hd, i, 1).contiguous() for x, i in ((q, h), (k, g), (v, g))), **kw)
            assert torch.equal(o[0], out[b].narrow(hd - 1, h, 1)) and torch.equal(l[0], lse[b].narrow(0, h, 1)), (b, h)


# 256 channels: without a mask only where they level out the workgroups per CU, under one fewer where the chip is full without; packed batches by the rule of the other widths
@pytest.mark.parametrize("B,N,H,Hkv,causal,packed,parts", [(1, 4000, 64, 4, 0, 0, 1), (1, 8000, 32, 2, 0, 0, 1), (1, 16000, 4, 1, 0, 0, 1), (8, 1830, 16, 1, 0, 0, 1), (1, 8000, 8, 1, 0, 0, 2), (1, 4000, 24, 3, 0, 0, 2), (1, 8000, 48, 3, 0, 0, 4),
                                                           (1, 8000, 64, 4, 0, 0, 1), (1, 16000, 32, 4, 0, 0, 2), (1, 16000, 8, 1, 1, 0, 2), (1, 8000, 8, 1, 1, 0, 3), (1, 16000, 16, 2, 1, 0, 4), (1, 30000, 2, 2, 1, 0, 1), (1, 17627, 2, 1, 1, 0, 2),
                                                           (4, 4000, 16, 2, 0, 1, 2), (8, 3000, 32, 4, 0, 1, 2), (16, 4000, 64, 4, 1, 1, 1), (3, 5344, 4, 1, 1, 1, 2), (2, 4807, 8, 1, 1, 1, 4)])
def test_parts_of_256_channels(B, N, H, Hkv, causal, packed, parts):
    extra = dict(layout=1, cu_seqlens_q=4096, cu_seqlens_k=4096) if packed else {}
    (status, seq), = launches([("sage_attn_fwd_ex", dict(B=B, H=H, H_kv=Hkv, N=N, N_kv=N, d=256, dtype=1, mode=0, causal=causal, kv_splits=1, **extra))])
    assert status == 0
    assert [x.grid[2] for x in seq if x.kernel in ("k_quant_kv", "k_quant_k")] == [parts]


# packed batches: the parts are counted by the longest sequence, so a short one has fewer steps than parts, or no queries, or no keys
PACKED = [([1500, 700, 0, 130, 5], [1500, 700, 64, 200, 5], 128, 16, 1, "bf16", True, 3), ([1700, 300, 1, 90], [900, 0, 70, 1], 64, 32, 2, "fp16", False, 3), ([1300, 40], [400, 130], 128, 512, 32, "bf16", False, 2)]


@pytest.mark.parametrize("lens_q,lens_k,d,H,Hkv,dtype,causal,parts", PACKED)
def test_the_launch_of_a_packed_batch_has_them(lens_q, lens_k, d, H, Hkv, dtype, causal, parts):
    (status, seq), = launches([("sage_attn_fwd_ex", dict(B=len(lens_q), H=H, H_kv=Hkv, N=max(lens_q), N_kv=max(lens_k), d=d, dtype=1, mode=0, layout=1, causal=int(causal), kv_splits=1,
                                                         cu_seqlens_q=4096, cu_seqlens_k=4096))])
    assert status == 0
    assert [x.grid[2] for x in seq if x.kernel in ("k_quant_kv", "k_quant_k")] == [parts]


@pytest.mark.gpu
@pytest.mark.parametrize("lens_q,lens_k,d,H,Hkv,dtype,causal,parts", PACKED)
def test_every_packed_sequence_has_the_bits_of_a_call_of_its_own(lens_q, lens_k, d, H, Hkv, dtype, causal, parts):
    pa = _pa()
    print(f"parts of Delta-S: packed q={lens_q} k={lens_k} d={d} H={H}/{Hkv} {dtype} causal={causal} parts={parts}", flush=True)
    (q, _, _), (_, k, v) = _inputs(1, sum(lens_q), sum(lens_q), d, H, Hkv, dtype, "NHD"), _inputs(1, sum(lens_k), sum(lens_k), d, Hkv, Hkv, dtype, "NHD")
    q, k, v = q[0], k[0], v[0]
    oq, ok = (np.concatenate([[0], np.cumsum(x)]).tolist() for x in (lens_q, lens_k))
    cu_q, cu_k = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in (oq, ok))
    kw = dict(causal=causal, kv_splits=1, delta_s="digits", return_lse=True)
    out, lse = pa.sage_attn_fwd_ex(q, k, v, cu_seqlens_q=cu_q, cu_seqlens_k=cu_k, **kw)
    for b, (n, nk) in enumerate(zip(lens_q, lens_k)):
        part = out[oq[b]:oq[b + 1]]
        if nk == 0:
            assert torch.count_nonzero(part) == 0
        if n == 0 or nk == 0:
            continue
        for h in sorted({0, H // 2, H - 1}):
            g = h // (H // Hkv)
            o, l = pa.sage_attn_fwd_ex(*(x[i0:i1, i:i + 1].unsqueeze(0).contiguous() for x, i0, i1, i in ((q, oq[b], oq[b + 1], h), (k, ok[b], ok[b + 1], g), (v, ok[b], ok[b + 1], g))), layout="NHD", **kw)
            assert torch.equal(o[0], part[:, h:h + 1]) and torch.equal(l[0, 0], lse[h, oq[b]:oq[b + 1]]), (b, h)
