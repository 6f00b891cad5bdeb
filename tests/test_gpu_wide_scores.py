"""Keys and queries whose scales multiply to nearly the largest float32: the factor of a score, delta_Q delta_K kappa, stays finite wherever it is, and
a code of 0 takes the score out of it."""
import pytest
import torch

from test_gpu_parity import _pa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("kw", [dict(), dict(group_map="token"), dict(group_map="fine"), dict(causal=True), dict(kv_splits=3)])
@pytest.mark.parametrize("B,H,Hkv,N,Nk,d", [(1, 2, 1, 300, 1700, 64), (1, 2, 2, 130, 1600, 128), (1, 2, 1, 200, 1600, 256), (64, 2, 1, 2, 1600, 64), (64, 4, 1, 2, 1600, 128), (64, 2, 1, 4, 1600, 256)])
def test_a_channel_of_keys_that_no_query_has(B, H, Hkv, N, Nk, d, kw, mode):
    """Two keys are +-X in channel 5 and zero elsewhere, every query is zero there: no score contains X, so none depends on it.  X = 2^126 makes the
    scale of their groups 2^123 and, under queries of 64, the factor 2^123 to 2^124 (the 4-bit mode; 2^115 in the 8-bit one)."""
    pa = _pa()
    print(f"wide scores: B={B} H={H}/{Hkv} N={N} N_kv={Nk} d={d} {kw} {mode}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + d)
    q, k, v = (torch.randn((B, h, n, d), generator=g, device="cuda") for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    q[..., 5] = k[..., 5] = 0.0
    q[:, :, ::2, 9], q[:, :, 1::2, 9] = 64.0, -64.0
    k[:, :, (3, Nk - 70)] = 0.0
    res = []
    for X in (2.0**14, 2.0**126):         # (either leaves nothing but codes of 0 in the rest of its groups)
        k[:, :, 3, 5], k[:, :, Nk - 70, 5] = X, -X
        res.append(pa.sage_attn_fwd_ex(q.bfloat16(), k.bfloat16(), v.bfloat16(), mode=mode, return_lse=True, **kw))
    (a, la), (b, lb) = res
    assert torch.isfinite(b).all() and torch.isfinite(lb).all()
    assert torch.equal(a, b) and torch.equal(la, lb)
