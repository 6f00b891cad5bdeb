"""Tile order of packed batches: every tile is taken once, whatever the number of positions in the last band, of heads and of
sequences, ragged or (nearly) equal (tests/test_packed_order_rule.py) - each sequence has the bits that it has alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("lens,H,Hkv,d,mode", [((1,), 1, 1, 64, "int4_fp8"), ((129, 0, 512, 1), 3, 1, 128, "int4_fp8"), ((513, 640, 77), 8, 2, 64, "int8_fp8"),
                                               ((700, 1025, 128, 1153), 5, 5, 128, "int8_fp8"), ((300, 900), 2, 1, 256, "int4_fp8"),
                                               ((1024,) + (90,) * 30 + (130,), 32, 8, 64, "int4_fp8"), ((1025,) + (90,) * 30 + (130,), 32, 8, 64, "int4_fp8"),
                                               ((640, 601, 640, 580), 3, 1, 64, "int4_fp8"), ((700,) * 3, 5, 5, 128, "int4_fp8"), ((1100, 1030, 1100, 900, 1090), 2, 2, 256, "int4_fp8")])
def test_packed_sequences_equal_themselves_alone(lens, H, Hkv, d, mode, causal):
    import paper_2411_10958_amd as pa
    print(f"packed order: {lens[:5]} ({len(lens)}) H={H}/{Hkv} d={d} {mode} causal={causal}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(sum(lens) + H + d)
    q, k, v = (torch.randn(sum(lens), h, d, generator=g, device="cuda").half() for h in (H, Hkv, Hkv))
    cu = torch.tensor([0] + list(lens)).cumsum(0).to(torch.int32).cuda()
    kw = dict(causal=causal, mode=mode, return_lse=True, kv_splits=1)
    out, lse = pa.sage_attn_fwd_ex(q, k, v, cu_seqlens_q=cu, max_seqlen_q=max(lens), max_seqlen_k=max(lens), **kw)
    a = 0
    for n in lens:
        if n:
            o, l = pa.sage_attn_fwd_ex(*(x[None, a:a + n].contiguous() for x in (q, k, v)), layout="NHD", **kw)
            torch.cuda.synchronize()
            assert torch.equal(out[a:a + n], o[0]) and torch.equal(lse[:, a:a + n], l[0]), n
        a += n
