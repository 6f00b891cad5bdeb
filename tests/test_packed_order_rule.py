"""Which packed batches send their tiles out in bands of positions (packed_in_bands in csrc/sage_attn_core.h, run on the host): the ragged ones,
whatever their number of tiles, and no batch of equal sequences."""
import os
import subprocess

import pytest

from paper_2411_10958_amd import build

SOURCE = """
#include "sage_common.h"
#include "sage_attn_core.h"
#include <cstdio>
int main() { int c, t, b, n; while (scanf("%d %d %d %d", &c, &t, &b, &n) == 4) putchar(sage::packed_in_bands(c != 0, t, b, n) ? '1' : '0'); }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    folder = tmp_path_factory.mktemp("bands")
    src, exe = folder / "bands.cpp", folder / "bands"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", os.path.join(build.PKG, "csrc"), "-I", os.path.join(build.ROOT, "include"),
                    "-o", str(exe), str(src)], check=True, capture_output=True)

    def call(lens, causal):
        text = f"{int(causal)} {sum(lens)} {len(lens)} {max(lens)}\n"
        return subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=60).stdout == "1"
    return call


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("lens", [(1,), (4096,) * 8, (500,) * 41, (8192,) * 64, (3000,) * 3, (1 << 24,) * 127, (2000, 1990, 2000, 1985)])
def test_equal_sequences_keep_the_order_of_a_batch(rule, lens, causal):
    assert not rule(lens, causal)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("lens", [(1000,) * 30 + (6000,), (700,) * 60 + (2500,), (16000, 2000, 2000, 8000, 500, 100), (513, 1, 1)])
def test_ragged_ones_do_not_whatever_their_tiles(rule, lens, causal):
    assert rule(lens, causal)


def test_the_lines(rule):
    assert rule((3200,) * 30 + (3199, 0), False) and not rule((3200,) * 31 + (0,), False)
    assert rule((1600,) * 12 + (1599, 0, 0, 0), True) and not rule((1600,) * 13 + (0,) * 3, True)
    assert rule((513, 1, 1), True) and not rule((512, 1, 1), True) and rule((512, 1, 1), False)
