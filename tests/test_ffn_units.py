"""Host logic, no GPU: how many units of 16 gate and 16 up rows a workgroup of the FFN's streaming kernel takes (csrc/ffn_stream.h)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_19867_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include "ffn_stream.h"
int main() {
  int blocks, units, K, cus;
  while (std::scanf("%d %d %d %d", &blocks, &units, &K, &cus) == 4) std::printf("%d\\n", spd::ffn_stream_units(blocks, units, K, cus));
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("units") / "ask")
    subprocess.run([gxx, "-std=c++17", "-x", "c++", "-", "-I", CSRC, "-o", exe], input=PROGRAM, text=True, check=True)

    def ask(cases):       # blocks of 16 tokens, inter, hidden, compute units
        text = "".join(f"{b} {inter // 16} {hidden} {cus}\n" for b, inter, hidden, cus in cases)
        return [int(x) for x in subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout.split()]
    return ask


def test_short_hidden_sizes_are_not_halved(ask):
    """Two waves that halve a unit's slices lose where there are few of them: the halves' sums are added up through LDS."""
    shapes = [(inter, cus) for inter in (512, 1408, 3072, 7168) for cus in (32, 96, 192, 256)]
    for blocks, line in ((1, 512), (2, 512), (4, 544), (8, 544)):
        for hidden in (32, 256, 384, 480, 512):
            if hidden < line:
                assert min(ask([(blocks, inter, hidden, cus) for inter, cus in shapes])) >= 4, (blocks, hidden)
        got = ask([(blocks, inter, line, cus) for inter, cus in shapes])
        assert got == ask([(blocks, inter, 8192, cus) for inter, cus in shapes]) and min(got) == 2, blocks


def test_units_go_by_the_rounds_that_the_compute_units_take(ask):
    assert ask([(4, 14336, 4096, cus) for cus in (64, 96, 128, 160, 192, 256)]) == [7, 5, 7, 6, 5, 4]
    assert ask([(4, 7168, 8192, cus) for cus in (128, 160, 192, 256)]) == [4, 3, 3, 2]
    assert ask([(8, 7168, 8192, cus) for cus in (128, 160, 192, 256)]) == [4, 4, 4, 2]
