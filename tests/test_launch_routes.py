"""Which kernels a call launches and on what grids, from the library's own launches with the HIP runtime replaced: no GPU."""
import itertools

from launch_recorder import launches

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
