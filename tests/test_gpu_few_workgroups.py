"""Decode-shaped calls of few workgroups: whether the kernel that quantizes K and V itself serves them depends on the length of
their chunks (attention_raw_ok in csrc/sage_attn_raw.hip); on both sides of every line the bits are those of the general path.
tests/test_launch_routes.py holds each case to the side it is meant for."""
import pytest
import torch

from test_gpu_attention_from_raw_kv import _both, _compare, _inputs, _pa

pytestmark = pytest.mark.gpu

# B, N, N_kv, d, H, Hkv, kv_splits, served by the kernel in the 4-bit / 8-bit mode (log-sum-exp wanted): one workgroup of one key; chunks at
# a line and one block past it (4-bit: 20 / 12 / 8 blocks of 64 / 128 / 256 channels, with more than four heads per KV head 16 / 8 / 4; 8-bit: 32 /
# 20 / 14; from 16 workgroups on half as long again; any length from 64 on); the library's own chunks
CASES = [(1, 1, 1, 128, 1, 1, 0, 1, 1), (1, 3, 64 * 20, 64, 4, 1, 1, 1, 1), (1, 1, 64 * 20 + 1, 64, 2, 2, 1, 0, 1), (1, 1, 64 * 16 + 1, 64, 8, 1, 1, 0, 1),
         (1, 4, 64 * 12, 128, 4, 2, 1, 1, 1), (1, 1, 64 * 12 + 1, 128, 3, 3, 1, 0, 1), (2, 1, 64 * 8 - 1, 256, 4, 4, 1, 1, 1), (1, 2, 64 * 8 + 1, 256, 2, 1, 1, 0, 1),
         (1, 1, 64 * 8, 128, 8, 1, 1, 1, 1), (1, 1, 64 * 8 + 1, 128, 8, 1, 1, 0, 1), (1, 4, 64 * 4, 256, 8, 1, 1, 1, 1), (1, 1, 64 * 4 + 1, 256, 6, 1, 1, 0, 1),
         (1, 1, 64 * 32, 64, 1, 1, 1, 0, 1), (1, 1, 64 * 32 + 1, 64, 1, 1, 1, 0, 0), (1, 5, 64 * 20, 128, 2, 1, 1, 0, 1), (1, 5, 64 * 20 + 1, 128, 2, 1, 1, 0, 0),
         (1, 1, 64 * 14, 256, 1, 1, 1, 0, 1), (1, 1, 64 * 14 + 1, 256, 1, 1, 1, 0, 0), (1, 1, 3000, 128, 8, 2, 0, 1, 1), (1, 32, 1500, 64, 1, 1, 0, 1, 1),
         (15, 1, 64 * 21, 64, 2, 1, 1, 0, 1), (16, 1, 64 * 30, 64, 2, 1, 1, 1, 1), (16, 1, 64 * 30 + 1, 64, 2, 1, 1, 0, 1), (15, 1, 64 * 21, 256, 1, 1, 1, 0, 0),
         (16, 1, 64 * 21, 256, 1, 1, 1, 0, 1), (63, 1, 64 * 49, 64, 1, 1, 1, 0, 0), (64, 1, 64 * 49, 64, 1, 1, 1, 1, 1)]
# B, N, N_kv, d, H, Hkv, mode, served by the kernel (no log-sum-exp, one chunk): the general path is three launches
THREE_LAUNCHES = [(1, 2, 128, 128, 2, 1, "int4_fp8", 1), (1, 2, 129, 128, 2, 1, "int4_fp8", 0), (3, 1, 192, 256, 4, 4, "int4_fp8", 1), (3, 1, 193, 256, 4, 4, "int4_fp8", 0),
                  (2, 4, 256, 64, 8, 1, "int4_fp8", 1), (2, 4, 257, 64, 8, 1, "int4_fp8", 0), (47, 1, 300, 128, 4, 1, "int4_fp8", 0), (48, 1, 300, 128, 4, 1, "int4_fp8", 1),
                  (47, 2, 700, 64, 2, 1, "int4_fp8", 0), (48, 2, 700, 64, 2, 1, "int4_fp8", 1), (1, 1, 384, 64, 3, 3, "int8_fp8", 1), (1, 1, 385, 64, 3, 3, "int8_fp8", 0),
                  (2, 8, 256, 128, 2, 1, "int8_fp8", 1), (2, 8, 257, 128, 2, 1, "int8_fp8", 0), (1, 4, 192, 256, 8, 1, "int8_fp8", 1), (1, 4, 193, 256, 8, 1, "int8_fp8", 0),
                  (95, 9, 100, 64, 2, 1, "int4_fp8", 0), (96, 9, 100, 64, 2, 1, "int4_fp8", 1), (2, 30, 128, 256, 2, 2, "int4_fp8", 1), (2, 30, 129, 256, 2, 2, "int4_fp8", 0),
                  (15, 1, 384, 128, 2, 1, "int8_fp8", 0), (16, 1, 384, 128, 2, 1, "int8_fp8", 1), (16, 1, 385, 128, 2, 1, "int8_fp8", 0), (31, 1, 900, 128, 2, 1, "int8_fp8", 0), (32, 1, 900, 128, 2, 1, "int8_fp8", 1)]


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,splits,raw4,raw8", CASES)
def test_equals_the_general_path(B, N, Nk, d, H, Hkv, splits, raw4, raw8, mode):
    pa = _pa()
    layout, causal = ("HND", "NHD")[Nk % 2], Nk >= N and H % 2 == 0
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, ("fp16", "bf16")[d % 128 == 0], layout)
    print(f"few workgroups: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} causal={causal} {layout} {mode} splits={splits}", flush=True)
    _compare(_both(pa, q, k, v, pa.make_args(q, k, v, None, causal=causal, mode=mode, layout=layout, kv_splits=splits)))


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,raw", THREE_LAUNCHES)
def test_equals_the_three_launches(B, N, Nk, d, H, Hkv, mode, raw):
    pa = _pa()
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, "bf16", "HND")
    print(f"few workgroups, three launches: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode}", flush=True)
    args = pa.make_args(q, k, v, torch.empty_like(q), causal=True, mode=mode, kv_splits=1)
    ws = torch.empty(pa.sage_attn_workspace_bytes(args), dtype=torch.uint8, device="cuda")
    out = pa.sage_attn_fwd_ex(q, k, v, causal=True, mode=mode, kv_splits=1, workspace=ws)
    halves = torch.full_like(q, 3.0)
    args.out, args.workspace, args.workspace_bytes = halves.data_ptr(), ws.data_ptr(), ws.numel()
    pa.sage_attn_prologue(args)
    pa.sage_attn_core(args)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.equal(out, halves)
