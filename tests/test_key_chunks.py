"""Key chunks the library picks for launches of fewer than 256 tiles: whole rounds of workgroups (chunks_of_few_tiles in csrc/sage_api.hip)."""
import math
import random

import pytest

from launch_recorder import launches
from test_abi_and_host import _args, _lib

STATIC_BYTES = 64 << 20


def _chunks(**kw):
    pa, _ = _lib()
    return pa.sage_attn_kv_splits(_args(pa, **kw))


# queries of a KV head within 32 columns (the kernel that reads K and V itself): 512 workgroups in one round, or two or three full ones where
# one leaves much of the chip idle - past an eighth of the time, past a sixth for chunks of 15 key blocks or fewer
@pytest.mark.parametrize("tiles,chunks,short", [(26, 19, 19), (72, 7, 7), (96, 5, 5), (103, 4, 4), (110, 4, 4), (113, 4, 4), (129, 7, 3), (146, 7, 3), (147, 3, 3),
                                                (170, 3, 3), (171, 5, 5), (204, 5, 5), (205, 7, 2), (219, 7, 2), (220, 2, 2), (255, 2, 2)])
@pytest.mark.parametrize("G", [1, 4])
def test_short_queries_fill_whole_rounds(tiles, chunks, short, G):
    for d in (64, 128, 256):
        assert _chunks(B=tiles, H=G, H_kv=1, N=1, N_kv=64 * 300, d=d) == chunks
        assert _chunks(B=tiles, H=G, H_kv=1, N=1, N_kv=64 * 15 * chunks, d=d) == short
        assert chunks == short or _chunks(B=tiles, H=G, H_kv=1, N=1, N_kv=64 * 15 * chunks + 1, d=d) == chunks


@pytest.mark.parametrize("d,tiles,blocks,chunks", [(256, 144, 300, 3), (256, 200, 300, 2), (256, 45, 300, 11), (128, 45, 300, 11), (128, 144, 300, 5), (128, 144, 75, 4), (128, 180, 60, 3),
                                                   (128, 180, 61, 4), (128, 250, 300, 3), (64, 144, 300, 7), (64, 144, 106, 7), (64, 144, 105, 6), (64, 100, 300, 5), (64, 250, 300, 4),
                                                   (64, 511, 96, 2), (64, 385, 95, 1), (64, 512, 300, 1), (128, 385, 300, 1)])
def test_longer_queries_fill_the_chip(d, tiles, blocks, chunks):
    assert _chunks(B=1, H=tiles, H_kv=tiles, N=128, N_kv=64 * blocks, d=d) == chunks


# where the general rule is not the faster one: the keys of short queries allow fewer chunks than fill two rounds; 64-wide heads between three and four workgroups
# per CU, and in three long chunks; 256-wide heads under a causal mask over about as many keys as queries
@pytest.mark.parametrize("tiles,blocks,chunks", [(171, 40, 5), (171, 39, 4), (192, 32, 4), (193, 39, 2), (204, 39, 2), (204, 40, 5), (192, 31, 2), (172, 24, 2), (205, 55, 2), (213, 55, 2), (205, 106, 7)])
def test_short_queries_on_few_keys(tiles, blocks, chunks):
    for d in (64, 128, 256):
        assert _chunks(B=tiles, H=4, H_kv=1, N=1, N_kv=64 * blocks, d=d) == chunks


@pytest.mark.parametrize("tiles,blocks,chunks", [(154, 90, 4), (154, 91, 6), (160, 120, 3), (160, 121, 6), (170, 121, 6), (180, 61, 4), (192, 75, 4), (193, 75, 3), (204, 75, 3), (204, 76, 5), (205, 160, 3),
                                                (205, 161, 4), (255, 160, 3), (255, 161, 4)])
def test_64_wide_heads_fill_a_fourth_workgroup_per_CU_or_none(tiles, blocks, chunks):
    assert _chunks(B=1, H=tiles, H_kv=tiles, N=128, N_kv=64 * blocks, d=64) == chunks


@pytest.mark.parametrize("H,N,Nk,causal,packed,chunks", [(12, 2000, 2000, 1, 0, 3), (12, 2000, 2000, 0, 0, 2), (12, 2000, 2500, 1, 0, 3), (12, 2000, 2501, 1, 0, 2), (5, 4608, 4608, 1, 0, 3),
                                                         (5, 4609, 4609, 1, 0, 2), (6, 4480, 4480, 1, 0, 3), (8, 3800, 3800, 1, 0, 2), (8, 3800, 3800, 1, 1, 3), (8, 3800, 3800, 0, 1, 2), (9, 2000, 2000, 1, 0, 3)])
def test_256_wide_heads_under_a_causal_mask(H, N, Nk, causal, packed, chunks):
    assert _chunks(B=1, H=H, H_kv=H, N=N, N_kv=Nk, d=256, causal=causal, **(dict(layout=1, cu_seqlens_q=4096) if packed else {})) == chunks


def test_a_packed_batch_is_counted_by_its_longest_sequence():
    for d, tiles, chunks in ((128, 144, 4), (64, 144, 4), (128, 45, 11), (256, 144, 3)):
        assert _chunks(B=1, H=tiles, H_kv=tiles, N=128, N_kv=64 * 300, d=d, layout=1, cu_seqlens_q=4096) == chunks


def test_never_more_than_asked_for_or_than_the_keys_allow():
    for d in (64, 128, 256):
        for N in (1, 128):
            for tiles in range(1, 256):
                for blocks in (1, 8, 15, 16, 40, 200, 5000):
                    S = _chunks(B=1, H=tiles, H_kv=tiles, N=N, N_kv=64 * blocks, d=d)
                    assert 1 <= S <= 64 and S <= max(1, blocks // 8), (d, N, tiles, blocks, S)


def _tiles(kw):
    G = kw["H"] // kw["H_kv"]
    return kw["B"] * (kw["H_kv"] if 2 <= G <= 8 and G * kw["N"] <= 128 else kw["H"] * -(-kw["N"] // 128))


def _launched_chunks(entry, kw):
    """(status, chunks per tile of the attention kernel that `entry` launches)"""
    (status, seq), = launches([(entry, {**dict(d=128, dtype=1, mode=0), **kw})])
    if status:
        return status, None
    if "k_merge_splits" not in [x.kernel for x in seq]:
        return status, 1
    grid, = [x.grid[0] for x in seq if x.kernel in ("k_attn_fwd", "k_attn_raw")]
    return status, next(S for S in range(1, 65) if grid in (_tiles(kw) * S, 8 * -(-_tiles(kw) * S // 8)))


# The built-in workspace: what does not fit it in the automatic chunks runs in ceil(512 / tiles) if those fit, in as many as do if not, from 256 tiles on in one
@pytest.mark.parametrize("kw,auto,static", [(dict(B=1, H=65, H_kv=65, N=256, N_kv=64 * 90, d=64), 5, 4), (dict(B=1, H=130, H_kv=65, N=128, N_kv=64 * 85, d=64, mode=1), 5, 4),
                                            (dict(B=40, H=1, H_kv=1, N=128, N_kv=64 * 77), 9, 7), (dict(B=1, H=32, H_kv=8, N=256, N_kv=64 * 72, d=256, mode=1), 8, 5),
                                            (dict(B=2, H=32, H_kv=8, N=1, N_kv=64 * 105, d=256, mode=1), 13, 4), (dict(B=100, H=1, H_kv=1, N=1, N_kv=64 * 69, d=64), 5, 4),
                                            (dict(B=96, H=2, H_kv=2, N=1, N_kv=64 * 33, d=64, mode=1), 4, 1), (dict(B=1, H=16, H_kv=8, N=2048, N_kv=11000, mode=1, causal=1), 3, 1)])
def test_the_built_in_workspace(kw, auto, static):
    pa, _ = _lib()
    need = lambda **x: pa.sage_attn_workspace_bytes(_args(pa, **{**kw, **x}))
    assert need() > STATIC_BYTES >= need(kv_splits=static) and _chunks(**kw) == auto
    assert static == (1 if _tiles(kw) >= 256 else -(-512 // _tiles(kw))) or need(kv_splits=static + 1) > STATIC_BYTES
    assert _chunks(workspace_bytes=STATIC_BYTES, **kw) == static
    assert _launched_chunks("sage_attn_fwd_static", kw) == (0, static)
    assert _launched_chunks("sage_attn_fwd_ex", dict(kw, workspace_bytes=STATIC_BYTES)) == (0, static)
    assert _launched_chunks("sage_attn_fwd_ex", kw) == (0, auto)
    assert _launched_chunks("sage_attn_fwd_static", dict(kw, kv_splits=auto))[0] == -3            # (asked for: as many or none)


def test_a_kept_workspace_serves_smaller_calls():
    """... of fewer sequences, queries or keys: the partial results of their chunks, more per tile, may need more than the larger call's."""
    pa, _ = _lib()
    rng = random.Random(3)
    calls, fewer = [], 0
    for _ in range(4000):
        Hkv = rng.choice([1, 2, 4, 8])
        G = rng.choice([1, 1, 2, 4, 8, 16])
        if Hkv * G * 2 > 128:
            continue
        draw = lambda hi: int(round(math.exp(rng.uniform(0, math.log(hi)))))
        B, N, Nk = draw(256), draw(600), draw(20000)
        Nk = max(N, Nk)
        base = dict(H=Hkv * G, H_kv=Hkv, d=rng.choice([64, 128, 256]), mode=rng.choice([0, 1]), causal=rng.choice([0, 1]), flags=rng.choice([0, 0, 1]))
        kept = pa.sage_attn_workspace_bytes(_args(pa, B=B, N=N, N_kv=Nk, **base))
        n = rng.randint(1, N)
        small = dict(base, B=rng.randint(max(1, B - 20), B), N=n, N_kv=rng.randint(max(n, Nk // 2), Nk))
        calls.append(("sage_attn_fwd_ex", {**small, "dtype": 1, "workspace_bytes": kept}))
        fewer += pa.sage_attn_workspace_bytes(_args(pa, **small)) > kept
        if len(calls) % 3 == 0:
            calls.append(("sage_attn_kv_stats", {**small, "flags": 0, "dtype": 1, "workspace_bytes": kept}))
    assert fewer > 100
    assert all(status == 0 for status, _ in launches(calls))


@pytest.mark.parametrize("kw", [dict(B=27, H=32, H_kv=8, N=1, N_kv=8192), dict(B=3, H=16, H_kv=16, N=300, N_kv=9000, d=256), dict(B=40, H=16, H_kv=8, N=64, N_kv=300)])
def test_too_small_a_workspace(kw):
    """Chunk by chunk down to what one takes; a byte less is refused, and so is a chunk count that was asked for and does not fit."""
    pa, _ = _lib()
    need = lambda **x: pa.sage_attn_workspace_bytes(_args(pa, **{**kw, **x}))
    one, auto = need(kv_splits=1), _chunks(**kw)
    last = None
    for S in range(-(-512 // _tiles(kw)) if auto > 1 else 1, 1, -1):
        for extra, chunks in ((0, S), (-1, S - 1)):
            size = need(kv_splits=S) + extra
            if size >= need():
                continue
            assert _chunks(workspace_bytes=size, **kw) == chunks and _launched_chunks("sage_attn_fwd_ex", dict(kw, workspace_bytes=size)) == (0, chunks)
            last = chunks
    assert last in (1, None)
    (status, _), (refused, none), (asked, _) = launches([("sage_attn_fwd_ex", {**dict(d=128, dtype=1, mode=0), **kw, **x}) for x in
                                                        (dict(workspace_bytes=one), dict(workspace_bytes=one - 1), dict(workspace_bytes=need(kv_splits=2) - 1, kv_splits=2))])
    assert status == 0 and refused == -3 and not none and (asked == -3 or need(kv_splits=2) == one)
