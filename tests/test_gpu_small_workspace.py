"""Workspaces too small for the automatic key chunks: fewer chunks, the bits of a call that asks for that many, and nothing written past the end."""
import pytest
import torch

from test_gpu_attention_from_raw_kv import _inputs
from test_gpu_parity import _pa

pytestmark = pytest.mark.gpu


# general and raw kernel, packed and unpacked tiles, several chunks and one; the last packs its short queries and has to give that up
@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,chunks", [(1, 300, 3000, 128, 8, 8, "int4_fp8", 3), (1, 200, 2500, 64, 20, 4, "int8_fp8", 1), (2, 1, 5000, 128, 32, 8, "int4_fp8", 5),
                                                       (9, 2, 2100, 256, 16, 16, "int8_fp8", 2), (3, 40, 2000, 128, 12, 4, "int4_fp8", 2), (3, 40, 500, 128, 12, 4, "int4_fp8", 1)])
def test_fewer_chunks(B, N, Nk, d, H, Hkv, mode, chunks):
    pa = _pa()
    print(f"small workspace: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode} chunks={chunks}", flush=True)
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, "bf16", "HND")
    asked = pa.make_args(q, k, v, causal=True, mode=mode, kv_splits=chunks)
    need, auto = pa.sage_attn_workspace_bytes(asked), pa.make_args(q, k, v, causal=True, mode=mode)
    assert pa.sage_attn_workspace_bytes(auto) > need
    ws = torch.full((need + 65536,), 0x5a, dtype=torch.uint8, device="cuda")
    auto.workspace_bytes = need
    assert pa.sage_attn_kv_splits(auto) == chunks
    out, lse = pa.sage_attn_fwd_ex(q, k, v, causal=True, mode=mode, workspace=ws[:need], return_lse=True)
    want, wlse = pa.sage_attn_fwd_ex(q, k, v, causal=True, mode=mode, kv_splits=chunks, return_lse=True)
    assert torch.equal(out, want) and torch.equal(lse, wlse)
    assert bool((ws[need:] == 0x5a).all())
    with pytest.raises(pa.SageError):
        pa.sage_attn_fwd_ex(q, k, v, causal=True, mode=mode, workspace=ws[:pa.sage_attn_workspace_bytes(pa.make_args(q, k, v, causal=True, mode=mode, kv_splits=1)) - 1])
