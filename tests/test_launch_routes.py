"""Which kernels a call launches and on what grids, from the library's own launches with the HIP runtime replaced: no GPU."""
import itertools
import re

import pytest

from launch_recorder import launches
from test_gpu_attention_from_raw_kv import REDUCE_CASES
from test_gpu_few_workgroups import CASES, THREE_LAUNCHES
from test_gpu_kv_pair import LARGE_PAIR_CASES, PACKED_PAIR_CASES, PAIR_CASES, SMALL_CASES

POINTER = 4096
BASE = dict(B=1, H=32, H_kv=32, d=128, dtype=1, mode=1, layout=1)


def test_no_grid_has_more_than_65535_rows():
    """y of a grid is 16 bits: token counts around the lines where the pieces of a token-major tensor, which go to y where its rows
    are long, reach that (64 keys, or two workgroups for them, 128 queries, 256 keys)."""
    calls = []
    tokens = [n * 65535 + e for n in (32, 64, 128, 256) for e in (-64, -32, -31, 0, 1, 64) if n * 65535 + e <= 1 << 24] + [1 << 24]
    for n, mode, causal, opt in itertools.product(tokens, (0, 1), (0, 1), (dict(), dict(lse=POINTER), dict(flags=1), dict(H=64, H_kv=64, d=64),
                                                                          dict(H=16, H_kv=16, d=256), dict(layout=0), dict(group_map=4), dict(pv_format=1),
                                                                          dict(k_mean_in=POINTER, v_scale_in=POINTER))):
        for shape in (dict(N=n), dict(N=1, N_kv=n), dict(N=200, N_kv=n)):
            calls.append(("sage_attn_fwd_ex", {**BASE, "mode": mode, "causal": causal, **opt, **shape}))
        calls.append(("sage_attn_fwd_ex", {**BASE, "B": 3, "N": n, "mode": mode, "causal": causal, "cu_seqlens_q": POINTER, **opt, "layout": 1}))
    ran = 0
    for (entry, kw), (status, seq) in zip(calls, launches(calls)):
        assert status in (0, -2), kw                # (-2: more tiles than an int of the launch may count)
        ran += status == 0
        for x in seq:
            assert max(x.grid[1:]) <= 65535, (kw, x)
    assert ran > len(calls) * 0.9


def _names(**kw):
    (status, seq), = launches([("sage_attn_fwd_ex", kw)])
    assert status == 0, kw
    return [x.kernel for x in seq]


def _mode(mode):
    return 0 if mode == "int4_fp8" else 1


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,smooth_v", PAIR_CASES)
def test_one_sequence_more_takes_two_launches(B, N, Nk, d, H, Hkv, mode, smooth_v):
    call = dict(N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, dtype=1, mode=_mode(mode), flags=int(smooth_v), lse=POINTER, kv_splits=1)
    assert "k_quant_kv" in _names(B=B - 1, **call)
    two = _names(B=B, **call)
    assert "k_quant_kv" not in two and "k_quant_k" in two and "k_quant_v" in two


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv", LARGE_PAIR_CASES)
def test_the_lines_of_the_pair_on_larger_calls(B, N, Nk, d, H, Hkv):
    call = dict(N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, dtype=1, mode=0, lse=POINTER, kv_splits=1)
    for b, two in ((B, True), (B - 1, False)):
        names = _names(B=b, **call)
        assert ("k_quant_kv" in names) == (not two) and ("k_quant_v" in names) == two, (b, names)


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode", PACKED_PAIR_CASES)
def test_the_lines_of_the_pair_on_packed_batches(B, N, Nk, d, H, Hkv, mode):
    call = dict(N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, dtype=0, mode=_mode(mode), layout=1, lse=POINTER, kv_splits=1, cu_seqlens_q=POINTER, cu_seqlens_k=POINTER)
    for b, two in ((B, True), (B - 1, False)):
        names = _names(B=b, **call)
        assert ("k_quant_kv" in names) == (not two) and ("k_quant_v" in names) == two, (b, names)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("packed", [dict(), dict(layout=1, cu_seqlens_q=POINTER, cu_seqlens_k=POINTER)])
def test_the_pair_has_no_holes(d, packed):
    """With more blocks, or more rows, the pair is left for good."""
    sizes = [1, 2, 8, 16, 24, 25, 26, 31, 32, 64, 128, 160, 256, 257, 300, 400, 600, 700, 768, 769, 800, 801, 1000, 2000, 3000, 4096, 4608, 4609, 6000, 12000, 24000, 24001, 40000]
    calls = [("sage_attn_fwd_ex", dict(B=b, N=1, N_kv=64, d=d, H=r, H_kv=1, dtype=1, mode=0, lse=POINTER, kv_splits=1, k_mean_in=POINTER, v_scale_in=POINTER, flags=32, **packed))
             for r in [x for x in sizes if x <= 400] for b in sizes if b * r <= 65535]
    res = launches(calls)
    pair = {(kw["H"], kw["B"]): "k_quant_kv" in [x.kernel for x in seq] for (_, kw), (_, seq) in zip(calls, res)}
    assert all(status == 0 for status, _ in res)
    for (r, b), p in pair.items():
        if p:
            assert all(q for (r2, b2), q in pair.items() if r2 == r and b2 < b or b2 == b and 24 < r2 < r or b2 == b and r2 < r <= 24), (r, b)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,Nk,d,H,Hkv,reduces", REDUCE_CASES)
def test_decode_calls_reduce_the_statistics_in_the_kernel_or_before(B, Nk, d, H, Hkv, reduces, mode):
    call = dict(B=B, N=2, N_kv=Nk, d=d, H=H, H_kv=Hkv, dtype=0, mode=mode, causal=1, lse=POINTER)
    names = _names(**call)
    assert "k_attn_raw" in names and ("k_finalize_stats" in names) == (not reduces), names
    given = _names(k_mean_in=POINTER, v_scale_in=POINTER, **call)
    assert given[0] == "k_attn_raw", given
    if B * Hkv >= 64:                      # ... in one chunk as in several
        one = _names(kv_splits=1, **call)
        assert "k_attn_raw" in one and "k_merge_splits" not in one and ("k_finalize_stats" in one) == (not reduces), one


@pytest.mark.parametrize("extra", [dict(), dict(causal=1), dict(kv_splits=1), dict(layout=1, cu_seqlens_q=POINTER, cu_seqlens_k=POINTER), dict(k_mean_in=POINTER, v_scale_in=POINTER)])
@pytest.mark.parametrize("d,H", [(64, 8), (128, 32), (256, 64)])
@pytest.mark.parametrize("mode,N,lone", [(0, 1, True), (0, 2, False), (1, 1, False)])
def test_one_query_in_the_4_bit_mode_has_a_kernel_of_its_own(mode, N, lone, d, H, extra):
    """(the last template argument of k_attn_raw)"""
    (status, seq), = launches([("sage_attn_fwd_ex", {**dict(B=16, N=N, N_kv=3000, d=d, H=H, H_kv=8, dtype=1, mode=mode, lse=POINTER), **extra})])
    raw = [x.mangled for x in seq if x.kernel == "k_attn_raw"]
    assert status == 0 and len(raw) == 1 and re.search(r"ILi%dE.*Lb([01])EEE" % d, raw[0])[1] == str(int(lone)), raw


@pytest.mark.parametrize("B,H,Hkv,N,Nk,d,mode", [(1, 2, 2, 256, 256, 64, 0), (39, 64, 8, 58, 586, 256, 1), (2, 8, 1, 300, 300, 128, 0), (18, 64, 8, 217, 435, 128, 1)])
def test_quantizer_of_q_and_statistics_leave_no_workgroup_empty(B, H, Hkv, N, Nk, d, mode):
    call = dict(B=B, H=H, H_kv=Hkv, N=N, N_kv=Nk, d=d, mode=mode, dtype=1)
    for stats, chunks in ((dict(), (Nk + 255) // 256), (dict(k_mean_in=POINTER, v_scale_in=POINTER), 0)):
        (_, seq), = launches([("sage_attn_fwd_ex", {**call, **stats})])
        assert seq[0].kernel == "k_quant_q_and_stats" and seq[0].grid == (H // Hkv * ((N + 127) // 128) + chunks, B * Hkv, 1)


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,three", SMALL_CASES)
def test_small_calls_take_the_side_their_case_means(B, N, Nk, d, H, Hkv, mode, three):
    names = _names(B=B, N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, mode=_mode(mode), kv_splits=1)
    assert (names[:2] == ["k_quant_q_and_stats", "k_quant_kv"]) == three and ("k_col_stats" in names) == (not three)


# decode-shaped calls that the attention kernel with the quantizers in it made slower, where the general path is three launches: B, H, Hkv,
# N, N_kv, d, mode (29.2 -> 34.2 us, 37.6 -> 45.6, 26.3 -> 30.4, 34.7 -> 36.9, 30.1 -> 33.0)
@pytest.mark.parametrize("B,H,Hkv,N,Nk,d,mode", [(9, 2, 1, 2, 746, 128, 0), (1, 8, 8, 4, 454, 256, 0), (3, 32, 4, 4, 409, 128, 0), (9, 16, 2, 1, 1178, 64, 0),
                                                 (5, 4, 1, 4, 863, 128, 1)])
def test_few_workgroups_keep_the_three_launches(B, H, Hkv, N, Nk, d, mode):
    call = dict(B=B, H=H, H_kv=Hkv, N=N, N_kv=Nk, d=d, mode=mode, causal=1, kv_splits=1)
    assert _names(**call) == ["k_quant_q_and_stats", "k_quant_kv", "k_attn_fwd"]
    # ... and the kernel stays where it saves launches: statistics supplied, or the log-sum-exp wanted
    assert _names(**call, k_mean_in=POINTER, v_scale_in=POINTER) == ["k_attn_raw"]
    assert _names(**call, lse=POINTER) == ["k_col_stats", "k_attn_raw"]


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,splits,raw4,raw8", CASES)
def test_few_workgroups_take_the_side_their_case_means(B, N, Nk, d, H, Hkv, splits, raw4, raw8):
    for mode, raw in ((0, raw4), (1, raw8)):
        call = dict(B=B, N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, kv_splits=splits, mode=mode, causal=Nk >= N and H % 2 == 0, layout=Nk % 2, lse=POINTER)
        assert ("k_attn_raw" in _names(**call)) == bool(raw), mode


@pytest.mark.parametrize("B,N,Nk,d,H,Hkv,mode,raw", THREE_LAUNCHES)
def test_three_launches_take_the_side_their_case_means(B, N, Nk, d, H, Hkv, mode, raw):
    names = _names(B=B, N=N, N_kv=Nk, d=d, H=H, H_kv=Hkv, kv_splits=1, mode=_mode(mode), dtype=1, causal=1)
    assert names == (["k_col_stats", "k_attn_raw"] if raw else ["k_quant_q_and_stats", "k_quant_kv", "k_attn_fwd"])
