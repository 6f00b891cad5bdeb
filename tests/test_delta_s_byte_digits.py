"""The digit form of the Delta-S product (Sec. 3.1: Delta-S = q_bar_i . gamma(K)^T): a CPU model of its number scheme against
the oracle's correctly rounded float64 product, and the GPU kernel at the edges of its steps.

The model is numpy integer arithmetic written for this test: every number of a row is divided by 2^E (E three above the
exponent of the row's largest magnitude), rounded to 48 bits and cut into six signed bytes, the planes are multiplied as exact
integers, the pairs with digit indices a + b <= 6 are kept and recombined in float64."""
import numpy as np
import pytest

import workloads as wl
from oracle import sage_oracle as so

f32, f64 = np.float32, np.float64


def _digits(X):
    mx = np.abs(X).max(axis=1).astype(f32)
    eb = (mx.view(np.uint32) >> 23).astype(np.int64)            # biased exponent of the row's largest magnitude
    N = np.rint(X.astype(f64) * np.ldexp(1.0, 48 + 124 - eb)[:, None]).astype(np.int64) + 0x808080808080
    return [((N >> (40 - 8 * a)) & 255) - 128 for a in range(6)], np.where(mx > 0, np.ldexp(1.0, eb - 124), 0.0)


def _digit_product(qbar, gK, kappa, max_pair):
    (qd, qu), (kd, ku) = _digits(qbar), _digits(gK)
    s = np.zeros((qbar.shape[0], gK.shape[0]), f64)
    for k in range(max_pair, -1, -1):                           # smallest weights first
        acc = sum(qd[a] @ kd[k - a].T for a in range(6) if 0 <= k - a < 6)
        s = acc.astype(f64) * 2.0 ** (-8 * (k + 2)) + s
    return (s * (qu[:, None] * (ku[None, :] * f64(kappa)))).astype(f32)


def test_six_bytes_and_pairs_up_to_six_give_the_rounded_float64_product():
    for seed in range(6):
        rng = np.random.default_rng(100 + seed)
        d = 128 if seed % 2 else 64
        q, k = (wl.awkward_values(rng, (1, 2048, d), "bf16" if seed % 3 else "fp16")[0] for _ in range(2))
        _, gK = so.smooth_k(k)
        qbar, _ = so.smooth_q(q)
        kappa = f32(f32(1.0 / np.sqrt(d)) * so.LOG2E_F32)
        D = so.delta_s(qbar, gK, kappa)
        diff = np.abs(_digit_product(qbar, gK, kappa, 6).astype(f64) - D)
        assert np.all(diff <= np.spacing(np.abs(D))) and (diff > 0).mean() <= 1e-5


def test_a_value_that_nearly_cancels_needs_the_pairs_of_index_sum_six():
    spec = wl.CONFIGS["causal16k"]
    q, k = wl.make_head(spec, "q", 0, 5, 0), wl.make_head(spec, "k", 0, 5, 0)
    _, gK = so.smooth_k(k)
    qbar, _ = so.smooth_q(q)
    kappa = f32(f32(1.0 / np.sqrt(spec.d)) * so.LOG2E_F32)
    rows, keys = slice(48, 49), slice(7168, 7232)
    D = so.delta_s(qbar[rows], gK[keys], kappa)
    d5, d6 = (np.abs(_digit_product(qbar[rows], gK[keys], kappa, m).astype(f64) - D) for m in (5, 6))
    assert (d5 > 0).any() and not (d6 > 0).any()


def test_joined_accumulators_stay_below_31_bits():
    """256 acc_4 + acc_5 (and the other neighbours) at d = 128: rows of one repeated value, over values whose digits are the
    largest a 24-bit number can have in any five neighbouring places."""
    vals = [s * f * 2.0 ** -e for s in (1, -1) for e in range(0, 47) for f in (1.0, 8421504 / 2 ** 23, 16777215 / 2 ** 23,
                                                                             8421503 / 2 ** 23, 8355711 / 2 ** 22)]
    X = np.repeat(np.array(vals, f32)[:, None], 128, axis=1)
    X[:, 0] = 1.9999999                                         # the row's largest: every row has the same exponent
    dg, _ = _digits(X)
    for k in (0, 2, 4):
        a, b = (sum(np.abs(dg[i].astype(np.int64)) @ np.abs(dg[j - i].astype(np.int64)).T for i in range(6) if 0 <= j - i < 6) for j in (k, k + 1))
        assert (256 * a + b).max() < 2 ** 31
    assert np.abs(dg[0]).max() <= 64


def test_bytes_represent_every_value_within_21_binades_of_the_row_maximum_exactly():
    rng = np.random.default_rng(5)
    X = (rng.uniform(0.5, 1.0, (64, 128)) * rng.choice([-1.0, 1.0], (64, 128)) * np.exp2(rng.integers(-21, 1, size=(64, 128)))).astype(f32)
    X[:, 0] = 1.5                                               # the row's largest magnitude: exponent 0; the others lie in [2^-22, 1)
    dg, up = _digits(X)
    back = sum(dg[a].astype(f64) * 2.0 ** (-8 * (a + 1)) for a in range(6)) * up[:, None]
    small = np.abs(X) < 2.0 ** -21                              # exponent -22: one bit below the grid 2^-45
    assert np.array_equal(back[~small].astype(f32), X[~small]) and (~small).sum() > 7000
    assert np.all(np.abs(back - X.astype(f64)) <= 2.0 ** -46)
    assert np.abs(dg[0]).max() <= 64 and all(-128 <= dg[a].min() and dg[a].max() <= 127 for a in range(1, 6))


# rows of block means per KV head: one, a few (told apart by division), just below, at and above a step of 16, and steps that
# cross from one head to the next; with a causal mask the rows start where a key block becomes visible
@pytest.mark.gpu
@pytest.mark.parametrize("H,Hkv,N,Nk,d,causal", [(1, 1, 100, 100, 128, True), (4, 2, 300, 300, 64, True), (3, 1, 640, 700, 128, True), (5, 1, 384, 384, 256, True),
                                                (1, 1, 1920, 1920, 64, True), (1, 1, 2048, 2048, 128, True), (2, 1, 2049, 2100, 128, True), (3, 1, 2200, 2200, 64, False),
                                                (2, 1, 4300, 4300, 64, True), (2, 1, 2177, 2177, 256, True)])
@pytest.mark.parametrize("form", ["digits", "fp64"])
def test_attention_reads_only_rows_that_were_formed(H, Hkv, N, Nk, d, causal, form):
    """The workspace starts as NaN: a Delta-S value that attention uses and no step wrote would reach the output.  The two exact
    forms agree but for single values next to a rounding boundary, so nearly every output row is the same."""
    import torch
    import paper_2411_10958_amd as pa
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, h, n, d), generator=g, device="cuda") * 2 + torch.randn((1, h, 1, d), generator=g, device="cuda") * 3
               for h, n in ((H, N), (Hkv, Nk), (Hkv, Nk)))
    q, k, v = (x.bfloat16() for x in (q, k, v))

    def run(f):
        out = torch.empty_like(q)
        a = pa.make_args(q, k, v, out, causal, kv_splits=1, delta_s=f)
        ws = torch.full((pa.sage_attn_workspace_bytes(a),), 255, dtype=torch.uint8, device="cuda")
        return pa.sage_attn_fwd_ex(q, k, v, out=out, causal=causal, workspace=ws, kv_splits=1, delta_s=f)
    out, ref = run(form), run("fp32")
    assert torch.isfinite(out).all()
    other = run("fp64" if form == "digits" else "digits")
    assert (out != other).any(-1).float().mean() <= 1e-2
    assert (out.float() - ref.float()).norm() <= 2e-3 * ref.float().norm()    # FP32 sums move a few codes of P~ by one step


# the same of a packed batch (the first visible block of each sequence is its own; one with fewer keys than queries) and of a split key range
@pytest.mark.gpu
@pytest.mark.parametrize("lens_q,lens_k,H,Hkv,d,splits", [("300,1,2100,129", "", 4, 2, 64, 1), ("640,65,1920", "700,65,2300", 3, 1, 128, 1), ("2177,40", "100,40", 2, 1, 128, 1),
                                                          ("2049", "4200", 2, 1, 128, 4), ("700,512", "5000,1100", 2, 2, 256, 3)])
@pytest.mark.parametrize("form", ["digits", "fp64"])
def test_packed_and_split_attention_reads_only_rows_that_were_formed(lens_q, lens_k, H, Hkv, d, splits, form):
    import torch
    import paper_2411_10958_amd as pa
    lq = [int(x) for x in lens_q.split(",")]
    lk = [int(x) for x in lens_k.split(",")] if lens_k else lq
    g = torch.Generator(device="cuda").manual_seed(sum(lq))
    q, k, v = ((torch.randn((n, h, d), generator=g, device="cuda") * 2 + torch.randn((1, h, d), generator=g, device="cuda") * 3).bfloat16()
               for h, n in ((H, sum(lq)), (Hkv, sum(lk)), (Hkv, sum(lk))))
    cu = [torch.tensor([0, *np.cumsum(x)], dtype=torch.int32).cuda() for x in (lq, lk)]
    kw = dict(cu_seqlens_q=cu[0], cu_seqlens_k=cu[1], max_seqlen_q=max(lq), max_seqlen_k=max(max(lk), max(lq)), causal=True, kv_splits=splits)

    def run(f, fill):
        out = torch.empty_like(q)
        a = pa.make_varlen_args(q, k, v, out, delta_s=f, **kw)
        ws = torch.full((pa.sage_attn_workspace_bytes(a),), fill, dtype=torch.uint8, device="cuda")
        return pa.sage_attn_fwd_ex(q, k, v, out=out, workspace=ws, delta_s=f, **kw)
    out = run(form, 255)
    assert torch.isfinite(out).all() and torch.equal(out, run(form, 0))
    other = run("fp64" if form == "digits" else "digits", 255)
    assert (out != other).any(-1).float().mean() <= 1e-2


@pytest.mark.gpu
def test_a_nan_key_reaches_the_output_where_few_rows_meet_many_key_blocks():
    """16 rows of block means on 384 key blocks: Delta-S in float64, whose products carry a NaN of K (through its mean) to every
    query of that head."""
    import torch
    import paper_2411_10958_amd as pa
    g = torch.Generator(device="cuda").manual_seed(0)
    q, k, v = (torch.randn((1, 12, 2000, 128), generator=g, device="cuda").bfloat16() for _ in range(3))
    k[0, 3, 77, 5] = float("nan")
    out = pa.sage_attn_fwd_ex(q, k, v, causal=False, kv_splits=1)
    assert out[0, 3].isnan().any(-1).all()
    assert torch.isfinite(out[0, [i for i in range(12) if i != 3]]).all()
