"""Token-major calls whose rows reach 8 KB (4096 elements) run the preprocessing heads first (csrc/sage_common.h,
make_tensor_map); head-major ones never do.  Workgroup order is all that differs, so the results are the same bits: for K and V
in each of their kernels, with Q in the other order and in the same one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(B, H, Hkv, N, Nk, d):
    gen = torch.Generator(device="cuda").manual_seed(H + d)
    draw = lambda heads, n: (torch.randn((B, heads, n, d), generator=gen, device="cuda") * 2.0 +
                             torch.randn((1, heads, 1, d), generator=gen, device="cuda") * 3.0).to(torch.bfloat16)
    return draw(H, N), draw(Hkv, Nk), draw(Hkv, Nk)


def _nhd(x):
    return x.transpose(1, 2).contiguous()


# KV rows of 4096 elements (and more); the last one: Q heads first, K and V not
@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,H,Hkv,N,Nk,d,causal", [(2, 32, 32, 333, 590, 128, True), (1, 64, 64, 130, 257, 64, False),
                                                    (1, 16, 16, 300, 300, 256, True), (1, 40, 40, 200, 65, 128, False),
                                                    (1, 32, 8, 150, 300, 128, True)])
def test_same_bits_as_head_major(B, H, Hkv, N, Nk, d, causal, mode):
    import paper_2411_10958_amd as pa
    print(f"8 KB rows: B={B} H={H}/{Hkv} N={N} N_kv={Nk} d={d} causal={causal} {mode}", flush=True)
    if causal and Nk < N:
        N = Nk
    q, k, v = _tensors(B, H, Hkv, N, Nk, d)
    qn, kn, vn = _nhd(q), _nhd(k), _nhd(v)
    for extra in (dict(), dict(return_lse=True), dict(smooth_v=True), dict(group_map="tensor"), dict(delta_s="fp64"), dict(kv_splits=1, pv_format="e5m2")):
        ref = pa.sage_attn_fwd_ex(q, k, v, causal=causal, mode=mode, **extra)
        out = pa.sage_attn_fwd_ex(qn, kn, vn, causal=causal, mode=mode, layout="NHD", **extra)
        torch.cuda.synchronize()
        if "return_lse" in extra:
            assert torch.equal(ref[1], out[1])
            ref, out = ref[0], out[0]
        assert torch.equal(out.transpose(1, 2), ref), extra


@pytest.mark.parametrize("Hkv,d", [(32, 128), (16, 256), (64, 64)])
def test_running_statistics_and_packed_batches(Hkv, d):
    """The statistics update in two chunks, and a packed batch against its sequences head-major."""
    import paper_2411_10958_amd as pa
    print(f"8 KB rows: statistics and packed batch, H_kv={Hkv} d={d}", flush=True)
    q, k, v = _tensors(2, Hkv, Hkv, 90, 700, d)
    state = None
    for part in (slice(0, 513), slice(513, 700)):
        km, vs, state = pa.sage_attn_kv_stats_update(_nhd(k[:, :, part]), _nhd(v[:, :, part]), state, layout="NHD")
    ref_km, ref_vs = pa.sage_attn_kv_stats(k, v)
    torch.cuda.synchronize()
    assert torch.equal(km, ref_km) and torch.equal(vs, ref_vs)
    lens = [300, 1, 64, 230]
    cu = torch.tensor([0, 300, 301, 365, 595], dtype=torch.int32, device="cuda")
    q, k, v = _tensors(1, Hkv, Hkv, 595, 595, d)
    for mode in ("int4_fp8", "int8_fp8"):
        out, lse = pa.sage_attn_fwd_ex(_nhd(q)[0], _nhd(k)[0], _nhd(v)[0], causal=True, mode=mode, cu_seqlens_q=cu,
                                       max_seqlen_q=300, max_seqlen_k=300, kv_splits=1, return_lse=True)
        for b, n in enumerate(lens):
            part = slice(int(cu[b]), int(cu[b]) + n)
            one, one_lse = pa.sage_attn_fwd_ex(*(x[:, :, part].contiguous() for x in (q, k, v)), causal=True, mode=mode, kv_splits=1,
                                               return_lse=True)
            torch.cuda.synchronize()
            assert torch.equal(one[0].transpose(0, 1), out[part]) and torch.equal(one_lse[0], lse[:, part])
