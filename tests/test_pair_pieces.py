"""The order of the workgroups in the paired launches (pair_second in csrc/sage_common.h, run on the host; k_quant_q_and_stats in
csrc/sage_prologue.hip).  Workgroup L runs on XCD L % 8, and the workgroups of an XCD go to its 32 CUs in turn."""
import os
import subprocess

import numpy as np
import pytest

from paper_2411_10958_amd import build

SOURCE = """
#include "sage_common.h"
#include <cstdio>
int main() { for (unsigned L = 0; L < 8192; ++L) putchar(sage::pair_second(L) ? '1' : '0'); }
"""


@pytest.fixture(scope="module")
def second(tmp_path_factory):
    folder = tmp_path_factory.mktemp("pair")
    src, exe = folder / "pair.cpp", folder / "pair"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", os.path.join(build.PKG, "csrc"), "-o", str(exe), str(src)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=60).stdout
    return np.array(list(out), dtype=int)


def test_a_pair_has_one_of_each_kind(second):
    assert np.array_equal(second[::2] + second[1::2], np.ones(4096, int))


@pytest.mark.parametrize("n", [16, 32, 64, 512, 1024, 4096])
def test_both_kinds_on_every_xcd_and_cu(second, n):
    for xcd in range(8):
        assert second[:n][xcd::8].sum() == n // 16
    if n >= 512:
        for cu in range(256):
            assert second[:n][cu::256].sum() == n // 512


@pytest.mark.parametrize("nq", [1, 2, 3, 4, 5, 6, 8, 12, 32])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 8])
def test_query_blocks_on_every_xcd(nq, chunks):
    """The turn that launch_prologue_t gives the rows of k_quant_q_and_stats: over 32 rows each XCD has its share of the query blocks."""
    row, even = nq + chunks, (nq + chunks) & -(nq + chunks)
    shift, mask = (0, 7) if even >= 8 else ((1, 3) if even == 4 else (2, even - 1))
    count = np.zeros(8, int)
    for y in range(32):
        places = [(x + ((y >> shift) & mask)) % row for x in range(row)]
        assert sorted(places) == list(range(row)) and mask < row
        for x, place in enumerate(places):
            count[(y * row + x) % 8] += place < nq
    assert count.min() == count.max() == 32 * nq // 8


def test_heads_from_reciprocals():
    """x / nQb as k_quant_q_and_stats forms it, (x + 1/2) (1 / nQb) in float32, cut to an integer."""
    x = np.arange(1 << 16, dtype=np.uint32)
    for n in [*range(1, 2050), 3000, 4096, 5461, 8191, 8192, 16384, 20480]:
        inv = np.float32(1.0) / np.float32(n)
        assert np.array_equal(((x.astype(np.float32) + np.float32(0.5)) * inv).astype(np.int32), x // n), n
