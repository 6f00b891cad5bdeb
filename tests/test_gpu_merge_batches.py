"""The merge of the key chunks of a tile takes their partial results in batches of four (up to four chunks) or eight: chunk counts on both
sides of a batch's end, a causal mask that leaves later chunks empty, packed tiles and a log-sum-exp, against the CPU oracle with the same chunks."""
import pytest
import torch

import workloads as wl
from oracle import parity
from test_gpu_parity import _pa, _lse_close

pytestmark = pytest.mark.gpu


# chunks, N, N_kv, d, H, Hkv, causal (8 key blocks a chunk; short causal queries see the empty end of no chunk, N = N_kv leaves chunks empty)
@pytest.mark.parametrize("splits,N,Nk,d,H,Hkv,causal", [
    (2, 130, 1024, 64, 2, 1, False), (4, 65, 2048, 128, 2, 2, True), (5, 40, 2560, 64, 4, 2, False), (5, 2560, 2560, 64, 1, 1, True),
    (7, 33, 3584, 128, 2, 1, True), (8, 3, 4096, 64, 8, 2, True), (9, 65, 4608, 64, 1, 1, False), (16, 40, 8192, 64, 2, 1, True),
    (17, 40, 8704, 256, 1, 1, False)])
@pytest.mark.parametrize("mode", ["int4_fp8", "int8_fp8"])
def test_batches_of_chunks(splits, N, Nk, d, H, Hkv, causal, mode):
    pa = _pa()
    spec = wl.WorkloadSpec("merge", 1, H, Hkv, N, d, "bf16", causal, 3.0, 1.5, 2, 10.0, 1.0, 900 + splits, 0.0, Nk)
    data = wl.make_inputs(spec, seed=5)
    q, k, v = (wl.to_torch(data[x], "bf16", torch.device("cuda:0")) for x in "qkv")
    assert pa.sage_attn_kv_splits(pa.make_args(q, k, v, causal=causal, mode=mode, kv_splits=splits)) == splits
    print(f"{splits} chunks, {N} queries on {Nk} keys, d = {d}, {mode}", flush=True)
    out, lse = pa.sage_attn_fwd_ex(q, k, v, causal=causal, mode=mode, kv_splits=splits, return_lse=True)
    torch.cuda.synchronize()
    pros = parity.check_heads(wl.from_torch(out), data, causal, mode, "bf16", want_lse=True, splits=splits)
    for h in range(H):
        _lse_close(lse[0, h].cpu().numpy(), pros[0][h]["lse"], pros[0][h])
