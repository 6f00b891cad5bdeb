"""The Delta-S product of few key blocks and many block means, shared between several workgroups per key block (k_parts in csrc/sage_prologue.hip): a value
does not depend on the step it is formed in, so every query head of a KV head has the bits it has in a call of its own (one step, one workgroup)."""
import pytest
import torch

from launch_recorder import launches
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
