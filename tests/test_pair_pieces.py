"""pair_piece (csrc/sage_common.h): which piece of K or V a workgroup of the paired launch works on, run on the host.  Workgroup L runs on
XCD L % 8, and the workgroups of an XCD go to its 32 CUs in turn."""
import os
import subprocess

import numpy as np
import pytest

from paper_2411_10958_amd import build

SOURCE = """
#include "sage_common.h"
#include <cstdio>
int main() {
  unsigned M;
  while (scanf("%u", &M) == 1)
    for (unsigned L = 0; L < 2 * M; ++L) {
      const sage::PairPiece p = sage::pair_piece(L, M);
      printf("%u %d%c", p.piece, (int)p.second, L + 1 < 2 * M ? ' ' : '\\n');
    }
}
"""
SIZES = [1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 100, 768, 1001, 2048]


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    folder = tmp_path_factory.mktemp("pair")
    src, exe = folder / "pair.cpp", folder / "pair"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", os.path.join(build.PKG, "csrc"), "-o", str(exe), str(src)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], input=" ".join(map(str, SIZES)), capture_output=True, text=True, check=True, timeout=60).stdout
    res = {}
    for M, line in zip(SIZES, out.splitlines()):
        w = list(map(int, line.split()))
        res[M] = list(zip(w[::2], w[1::2]))
    return res


@pytest.mark.parametrize("M", SIZES)
def test_every_piece_once_and_both_kinds_on_every_xcd(pieces, M):
    assert sorted(pieces[M]) == [(p, kind) for p in range(M) for kind in (0, 1)]
    for xcd in range(8):
        kinds = [kind for L, (_, kind) in enumerate(pieces[M]) if L % 8 == xcd]
        assert abs(2 * sum(kinds) - len(kinds)) <= 2
    if M >= 512:
        for cu in range(256):
            kinds = [kind for L, (_, kind) in enumerate(pieces[M]) if L % 256 == cu]
            assert abs(2 * sum(kinds) - len(kinds)) <= 2


def test_quotients_of_the_paired_launches():
    """quotient() in csrc/sage_prologue.hip, (L + 1/2) (1 / n) in float32, cut to an integer: every L of the launches that use it (at most
    two pieces for each of 20480 workgroups)."""
    L = np.arange(1 << 16, dtype=np.uint32)
    for n in [*range(1, 2050), 3000, 4096, 5461, 8191, 8192, 16384, 20480, 40960]:
        inv = np.float32(1.0) / np.float32(n)
        assert np.array_equal(((L.astype(np.float32) + np.float32(0.5)) * inv).astype(np.int32), L // n), n
