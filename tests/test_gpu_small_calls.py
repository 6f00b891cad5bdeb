"""Small calls run the preprocessing as two launches (Q beside the statistics, K beside V with the statistics reduced in
each workgroup).  The same call with the log-sum-exp asked for takes the general sequence - the arithmetic is the same, so
the outputs must be the same bits - and so does one with the statistics supplied, up to the pass that is left out."""
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def _inputs(B, N, Nk, d, H, Hkv, dtype, layout):
    spec = wl.WorkloadSpec("small", B, H, Hkv, N, d, dtype, True, 3.0, 1.5, 2, 10.0, 1.0, 77, 0.0, Nk)
    data = wl.make_inputs(spec, 0)
    q, k, v = (wl.to_torch(data[n], dtype, torch.device("cuda:0")) for n in "qkv")
    if layout == "NHD":
        q, k, v = (x.transpose(1, 2).contiguous() for x in (q, k, v))
    return q, k, v


# one key; block and chunk edges (64, 256 keys); the longest (8 chunks) and one past it; the most workgroups (512) and more
@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,dtype,H,Hkv,causal,layout", [
    (1, 1, 1, 128, "bf16", 2, 1, True, "HND"), (2, 64, 65, 64, "fp16", 4, 2, True, "NHD"),
    (1, 129, 256, 256, "bf16", 2, 2, False, "HND"), (3, 300, 513, 128, "fp16", 4, 4, True, "HND"),
    (1, 257, 257, 128, "bf16", 32, 8, True, "NHD"), (2, 100, 2048, 64, "bf16", 3, 1, True, "HND"),
    (1, 2049, 2049, 64, "fp16", 2, 1, True, "NHD"), (4, 128, 1024, 128, "bf16", 8, 8, False, "HND"),
    (4, 128, 1025, 64, "bf16", 8, 8, False, "HND"),
])
def test_small_call_equals_the_general_sequence(B, N, Nk, d, dtype, H, Hkv, causal, layout, mode):
    import paper_2411_10958_amd as pa
    print(f"small call: B={B} N={N} N_kv={Nk} d={d} {dtype} H={H}/{Hkv} causal={causal} {layout} {mode}", flush=True)
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, dtype, layout)
    kw = dict(causal=causal, mode=mode, layout=layout)
    for group_map in ("lane", "block", "token"):
        out = pa.sage_attn_fwd_ex(q, k, v, group_map=group_map, **kw)
        general, _ = pa.sage_attn_fwd_ex(q, k, v, group_map=group_map, return_lse=True, **kw)
        given = pa.sage_attn_fwd_ex(q, k, v, group_map=group_map, kv_stats=pa.sage_attn_kv_stats(k, v, layout=layout), **kw)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all()
        assert torch.equal(out, general) and torch.equal(out, given)
