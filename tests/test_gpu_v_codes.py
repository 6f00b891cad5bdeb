"""The V quantizer's codes byte for byte against the CPU oracle, where its rows, its transposition in LDS and its two forms of the
quotient can go wrong: lengths around the 64 keys of a block and the rows of a thread, every width, channels of zeros (scale 0:
the dividing form), values of either zero and far below the channel's scale."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import sage_oracle as so
from test_gpu_parity import _pa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pv", ["e4m3", "e5m2", "int8"])
@pytest.mark.parametrize("zeros", [False, True])
@pytest.mark.parametrize("nk", [1, 3, 4, 5, 63, 64, 65, 131])
@pytest.mark.parametrize("d,dtype,smooth_v", [(64, "bf16", False), (64, "fp16", True), (128, "fp16", False), (128, "bf16", True), (256, "bf16", False),
                                              (256, "fp16", True)])
def test_v_codes(d, dtype, smooth_v, nk, zeros, pv):
    pa = _pa()
    print(f"V codes: d={d} {dtype} N_kv={nk} smooth_v={smooth_v} zeros={zeros} {pv}", flush=True)
    rng = np.random.default_rng(d + nk)
    x = (rng.standard_normal((2, nk, d)) * 2.0 ** rng.integers(-6, 7, (2, 1, d))).astype(np.float32)
    x[rng.random(x.shape) < 0.05] = -0.0
    x[rng.random(x.shape) < 0.05] *= np.float32(2.0 ** -14)
    if zeros:
        x[:, :, rng.integers(d, size=3)] = 0.0
    dev = torch.device("cuda:0")
    tt = torch.bfloat16 if dtype == "bf16" else torch.float16
    v = torch.from_numpy(x[None]).to(tt).to(dev)
    vn = v[0].float().cpu().numpy()
    got, _, _ = pa.sage_attn_quant(v, v, v, mode="int8_fp8", smooth_v=smooth_v, pv_format=pv, want=("v_codes", "v_scale"))
    torch.cuda.synchronize()
    for h in range(2):
        pro = so.quantize_head(vn[h], vn[h], vn[h], mode="int8_fp8", smooth_v_on=smooth_v, pv_fmt=pv)
        assert np.array_equal(got["v_scale"][0, h].cpu().numpy(), pro["v_scale"])
        assert np.array_equal(got["v_codes"][0, h].cpu().numpy(), pro["v_codes"].view(np.uint8))


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "fp16"), (128, "bf16"), (256, "bf16")])
def test_v_codes_beyond_a_supplied_scale(d, dtype):
    """A supplied scale bounds nothing: infinite values and quotients (bfloat16: a quotient past the largest float32) and NaN have the codes
    that the dividing form gives them, which a last channel with a scale of all mantissa bits calls for."""
    pa = _pa()
    print(f"V codes beyond the scale: d={d} {dtype}", flush=True)
    inf, big = float("inf"), 3e38 if dtype == "bf16" else 6e4
    g = torch.Generator(device="cuda").manual_seed(d)
    v = torch.randn(1, 2, 131, d, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float16)
    for key, x in ((0, inf), (5, -inf), (66, float("nan")), (67, big), (68, -big), (130, inf)):
        v[:, :, key, 3] = v[:, :, key, d - 9] = x
    scale = torch.full((1, 2, d), 2.0 ** -8, device="cuda")
    divided = scale.clone()
    divided[:, :, d - 1] = float.fromhex("0x1.fffffep-9")
    codes = [pa.sage_attn_quant(v, v, v, mode="int8_fp8", kv_stats=(torch.zeros_like(scale), s), want=("v_codes",))[0]["v_codes"] for s in (scale, divided)]
    torch.cuda.synchronize()
    assert torch.equal(codes[0][..., :d - 1], codes[1][..., :d - 1])
