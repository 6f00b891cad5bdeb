"""Decode-shaped calls of few workgroups: whether the kernel that quantizes K and V itself serves them depends on the length of
their chunks (attention_raw_ok in csrc/sage_attn_raw.hip); on both sides of every line the bits are those of the general path."""
import pytest

from test_gpu_attention_from_raw_kv import _both, _compare, _inputs, _pa

pytestmark = pytest.mark.gpu

# B, N, N_kv, d, H, Hkv, kv_splits: one workgroup of one key; chunks at a line and one block past it (4-bit: 20 / 12 / 8 blocks, with
# more than four heads per KV head 16 / 8 / 4; 8-bit: 32 / 20 / 14); the library's own chunks
CASES = [(1, 1, 1, 128, 1, 1, 0), (1, 3, 64 * 20, 64, 4, 1, 1), (1, 1, 64 * 20 + 1, 64, 2, 2, 1), (1, 4, 64 * 12, 128, 8, 2, 1), (1, 1, 64 * 12 + 1, 128, 3, 3, 1),
         (2, 1, 64 * 8 - 1, 256, 4, 4, 1), (1, 2, 64 * 8 + 1, 256, 2, 1, 1), (1, 1, 64 * 8, 128, 8, 1, 1), (1, 4, 64 * 4, 256, 8, 1, 1), (1, 1, 64 * 4 + 1, 256, 6, 1, 1),
         (1, 1, 64 * 32, 64, 1, 1, 1), (1, 5, 64 * 20, 128, 2, 1, 1), (1, 1, 64 * 14 + 1, 256, 1, 1, 1), (1, 1, 3000, 128, 8, 2, 0), (1, 32, 1500, 64, 1, 1, 0),
         (63, 1, 64 * 21, 64, 4, 1, 1), (64, 1, 64 * 21, 64, 4, 1, 1)]


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,splits", CASES)
def test_equals_the_general_path(B, N, Nk, d, H, Hkv, splits, mode):
    pa = _pa()
    layout, causal = ("HND", "NHD")[Nk % 2], Nk >= N and H % 2 == 0
    q, k, v = _inputs(B, N, Nk, d, H, Hkv, ("fp16", "bf16")[d % 128 == 0], layout)
    print(f"few workgroups: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} causal={causal} {layout} {mode} splits={splits}", flush=True)
    _compare(_both(pa, q, k, v, pa.make_args(q, k, v, None, causal=causal, mode=mode, layout=layout, kv_splits=splits)))
