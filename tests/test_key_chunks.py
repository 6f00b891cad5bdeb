"""Key chunks the library picks for launches of fewer than 256 tiles: whole rounds of workgroups (chunks_of_few_tiles in csrc/sage_api.hip)."""
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


# what fitted the built-in workspace with ceil(512 / tiles) chunks still does: in as many chunks as that, where it would not in more
@pytest.mark.parametrize("kw", [dict(B=140, H=1, H_kv=1, N=1, N_kv=64 * 115, d=64), dict(B=1, H=65, H_kv=65, N=256, N_kv=64 * 90, d=64), dict(B=1, H=70, H_kv=70, N=256, N_kv=64 * 75, d=64),
                                dict(B=1, H=56, H_kv=2, N=512, N_kv=64 * 76, d=64), dict(B=150, H=2, H_kv=1, N=1, N_kv=700, d=128)])
def test_the_built_in_workspace_takes_what_it_took(kw):
    pa, _ = _lib()
    a = _args(pa, **kw)
    tiles = kw["B"] * (kw["H_kv"] if kw["N"] == 1 and kw["H"] > kw["H_kv"] else kw["H"] * ((kw["N"] + 127) // 128))
    up = max(1, min(-(-512 // tiles), 64, -(-kw["N_kv"] // 64) // 8)) if tiles < 256 else 1
    fitted = pa.sage_attn_workspace_bytes(_args(pa, kv_splits=up, **kw)) <= STATIC_BYTES
    call = dict(dict(B=1, H=1, H_kv=1, d=128, dtype=1, mode=a.mode, layout=0, causal=0), **kw)
    (status, _), = launches([("sage_attn_fwd_static", call)])
    assert not fitted or status == 0, (kw, up)
