"""K and V quantized by one launch or by two (kv_pair in csrc/sage_prologue.hip): a head quantized in a call on one side of the line
has the codes and scales that it has in a call on the other."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _pa():
    import paper_2411_10958_amd as pa
    return pa


# sequences, N, N_kv, d, H, Hkv, mode, smooth_v: one sequence more than the pair takes (tests/test_launch_routes.py holds the launches to
# that).  4-bit with few rows of block means, with many; 8-bit
PAIR_CASES = [
    (145, 100, 2047, 64, 2, 1, "int4_fp8", False), (145, 129, 1985, 128, 1, 1, "int4_fp8", True), (21, 70, 2000, 256, 3, 1, "int4_fp8", False),
    (26, 1000, 2001, 64, 35, 1, "int4_fp8", True), (26, 700, 2048, 128, 44, 1, "int4_fp8", False), (11, 520, 2040, 256, 5, 1, "int4_fp8", False),
    (25, 300, 2048, 256, 1, 1, "int8_fp8", True), (25, 67, 2047, 256, 1, 1, "int8_fp8", False), (145, 64, 2001, 128, 2, 1, "int8_fp8", False), (145, 33, 2048, 64, 1, 1, "int8_fp8", True)]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,smooth_v", PAIR_CASES)
def test_one_launch_equals_two(B, N, Nk, d, H, Hkv, mode, smooth_v):
    pa = _pa()
    print(f"K/V pair: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode} smooth_v={smooth_v}", flush=True)
    g = torch.Generator().manual_seed(B + N + Nk + d)
    q, k, v = (torch.randn(B, h, n, d, generator=g).to(torch.bfloat16).cuda() for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    kw = dict(mode=mode, smooth_v=smooth_v, return_lse=True, kv_splits=1)      # (the log-sum-exp keeps both calls off the small-call sequence)
    two, lse_two = pa.sage_attn_fwd_ex(q, k, v, **kw)
    one, lse_one = pa.sage_attn_fwd_ex(q[:-1], k[:-1], v[:-1], **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(two).all()
    assert torch.equal(one, two[:-1]) and torch.equal(lse_one, lse_two[:-1])


# the 4-bit lines for larger calls, one sequence more than the pair takes: blocks for up to 24 rows, the product of blocks and rows, blocks for more
# than 256 rows.  No case of fewer blocks or rows takes two launches (tests/test_launch_routes.py)
LARGE_PAIR_CASES = [(145, 100, 2047, 64, 1, 1), (145, 129, 1985, 128, 12, 1), (94, 1200, 2001, 64, 20, 1), (670, 400, 2048, 128, 7, 1),
                    (74, 1024, 2040, 128, 32, 1), (26, 1100, 2010, 128, 29, 1)]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv", LARGE_PAIR_CASES)
def test_one_launch_equals_two_on_larger_calls(B, N, Nk, d, H, Hkv):
    pa = _pa()
    print(f"K/V pair, larger: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + N + Nk + d)
    q, k, v = (torch.randn(B, h, n, d, generator=g, device="cuda").to(torch.bfloat16) for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    kw = dict(return_lse=True, kv_splits=1)
    more, lse_more = pa.sage_attn_fwd_ex(q, k, v, **kw)
    less, lse_less = pa.sage_attn_fwd_ex(q[:-1], k[:-1], v[:-1], **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(more).all()
    assert torch.equal(less, more[:-1]) and torch.equal(lse_less, lse_more[:-1])


# packed batches, counted by their longest sequence: one sequence more than the pair takes
PACKED_PAIR_CASES = [(145, 100, 2047, 64, 1, 1, "int4_fp8"), (145, 300, 2000, 128, 8, 1, "int4_fp8"), (94, 1200, 2001, 64, 20, 1, "int4_fp8"), (26, 1100, 2010, 128, 29, 1, "int4_fp8"),
                     (25, 100, 2048, 256, 1, 1, "int4_fp8"), (25, 900, 2000, 256, 8, 1, "int4_fp8"), (145, 64, 2001, 128, 2, 1, "int8_fp8"), (25, 67, 2047, 256, 1, 1, "int8_fp8")]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode", PACKED_PAIR_CASES)
def test_one_launch_equals_two_on_packed_batches(B, N, Nk, d, H, Hkv, mode):
    pa = _pa()
    print(f"K/V pair, packed: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode}", flush=True)
    nq, nk = ([n] + [max(1, n * (7 * i % 11) // 10 % (n + 1)) for i in range(1, B)] for n in (N, Nk))
    g = torch.Generator(device="cuda").manual_seed(B + N + Nk + d)
    q, k, v = (torch.randn(sum(n), h, d, generator=g, device="cuda").half() for h, n in ((H, nq), (Hkv, nk), (Hkv, nk)))
    cq, ck = (torch.tensor([0] + n).cumsum(0).to(torch.int32).cuda() for n in (nq, nk))
    kw = dict(mode=mode, max_seqlen_q=N, max_seqlen_k=Nk, return_lse=True, kv_splits=1)
    more, lse_more = pa.sage_attn_fwd_ex(q, k, v, cu_seqlens_q=cq, cu_seqlens_k=ck, **kw)
    a, b = sum(nq[:-1]), sum(nk[:-1])
    less, lse_less = pa.sage_attn_fwd_ex(q[:a], k[:b], v[:b], cu_seqlens_q=cq[:-1], cu_seqlens_k=ck[:-1], **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(more).all()
    assert torch.equal(less, more[:a]) and torch.equal(lse_less, lse_more[:, :a])


# the lines of small_call: 32 chunks of 256 keys, 20480 workgroups times chunks, 768 key blocks (384 with many rows of block means) at 256 channels; last: whether the
# three launches serve it
SMALL_CASES = [
    (1, 130, 8192, 128, 3, 1, "int4_fp8", True), (1, 130, 8193, 64, 3, 1, "int8_fp8", False), (128, 128, 256, 64, 32, 32, "int4_fp8", True), (129, 128, 256, 64, 32, 32, "int4_fp8", False),
    (128, 128, 256, 64, 32, 32, "int8_fp8", True), (241, 128, 256, 64, 17, 17, "int8_fp8", False), (24, 70, 2048, 256, 1, 1, "int4_fp8", True), (25, 70, 2048, 256, 1, 1, "int4_fp8", False),
    (12, 600, 2048, 256, 5, 1, "int4_fp8", True), (13, 600, 2048, 256, 5, 1, "int4_fp8", False),
    (32, 60, 64, 256, 16, 4, "int8_fp8", True), (27, 60, 64, 256, 19, 1, "int8_fp8", True)]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,three", SMALL_CASES)
def test_three_launches_equal_the_general_sequence(B, N, Nk, d, H, Hkv, mode, three):
    pa = _pa()
    print(f"three launches: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + N + Nk + d)
    q, k, v = (torch.randn(B, h, n, d, generator=g, device="cuda").half() for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    out = pa.sage_attn_fwd_ex(q, k, v, mode=mode, kv_splits=1)
    general, _ = pa.sage_attn_fwd_ex(q, k, v, mode=mode, kv_splits=1, return_lse=True)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.equal(out, general)


# statistics finished under Q (up to 8 chunks with the log-sum-exp; 9 are finished before Q) or given; ragged lengths and token-major rows
@pytest.mark.parametrize("smooth_k", [True, False])
@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,layout", [(1, 65, 1, 64, 2, 1, "HND"), (3, 130, 2048, 128, 4, 2, "HND"), (2, 129, 2049, 128, 2, 2, "HND"),
                                                   (2, 300, 2047, 128, 32, 32, "NHD"), (1, 257, 1000, 256, 17, 17, "NHD"), (5, 1500, 1500, 64, 33, 33, "HND")])
def test_statistics_finished_under_q(B, N, Nk, d, H, Hkv, layout, mode, smooth_k):
    pa = _pa()
    print(f"statistics under Q: B={B} N={N} N_kv={Nk} d={d} H={H}/{Hkv} {mode} {layout} smooth_k={smooth_k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + N + Nk + d)
    q, k, v = (torch.randn((B, h, n, d) if layout == "HND" else (B, n, h, d), generator=g, device="cuda").bfloat16() + 1 for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    kw = dict(mode=mode, layout=layout, kv_splits=1, smooth_k=smooth_k)
    out, lse = pa.sage_attn_fwd_ex(q, k, v, return_lse=True, **kw)
    plain = pa.sage_attn_fwd_ex(q, k, v, **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.equal(out, plain)
    if smooth_k:
        given, lse_given = pa.sage_attn_fwd_ex(q, k, v, return_lse=True, kv_stats=pa.sage_attn_kv_stats(k, v, layout=layout), **kw)
        torch.cuda.synchronize()
        assert torch.equal(out, given) and torch.equal(lse, lse_given)
