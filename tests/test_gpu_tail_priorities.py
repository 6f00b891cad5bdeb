"""Workgroups that end a launch change their priority as their keys run out (tail_left in csrc/sage_attn_kernel.hip), in stretches of the
block loop: around every change, with whole and ragged last blocks, with and without a mask, the bits are those of calls too small to have it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# blocks of 64 keys around the changes (40, 20 and 8 left at 64 channels, 28, 12 and 4 at 128 and 256), fewer than the last of them, more than the first
BLOCKS = {64: (1, 7, 8, 9, 20, 21, 40, 41, 60), 128: (1, 3, 4, 5, 12, 13, 28, 29, 45), 256: (2, 4, 5, 12, 13, 28, 29)}


def _equal_parts(pa, heads, N, Nk, d, **kw):
    g = torch.Generator(device="cuda").manual_seed(N + Nk + d)
    q, k, v = (torch.randn(1, heads, n, d, generator=g, device="cuda").bfloat16() for n in (N, Nk, Nk))
    out, lse = pa.sage_attn_fwd_ex(q, k, v, return_lse=True, **kw)
    parts = [pa.sage_attn_fwd_ex(*(x[:, a:a + 40].contiguous() for x in (q, k, v)), return_lse=True, **kw) for a in range(0, heads, 40)]
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    assert torch.equal(out, torch.cat([o for o, _ in parts], 1)) and torch.equal(lse, torch.cat([x for _, x in parts], 1))


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,blocks", [(d, b) for d in BLOCKS for b in BLOCKS[d]])
def test_without_a_mask(d, blocks, mode):
    import paper_2411_10958_amd as pa
    for Nk in (64 * blocks, 64 * blocks - 17):                  # 3 tiles a head: 360 workgroups, the parts 120
        print(f"tail: d={d} N_kv={Nk} {mode}", flush=True)
        _equal_parts(pa, 120, 300, Nk, d, mode=mode, kv_splits=1)


@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
@pytest.mark.parametrize("d,blocks", [(64, 9), (64, 21), (64, 42), (128, 5), (128, 13), (128, 30), (256, 5), (256, 29)])
def test_causal_in_chunks(d, blocks, mode):
    """The wavefronts of a tile meet the mask at different blocks of its last chunk."""
    import paper_2411_10958_amd as pa
    for Nk in (128 * blocks, 128 * blocks + 45):                # 2 tiles a head in 2 chunks: 480 workgroups, the parts 160
        print(f"tail, causal: d={d} N_kv={Nk} {mode}", flush=True)
        _equal_parts(pa, 120, 230, Nk, d, mode=mode, causal=True, kv_splits=2)
