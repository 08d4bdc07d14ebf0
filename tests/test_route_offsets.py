"""The closed-form walk of Eq. 1 that the forward kernels and the planner share
(route_next_offset in csrc/bf1_route.h), compiled with the host compiler and
compared with the oracle's route for whole ranges of blocks and local widths,
and with the planner's closed row starts at the largest blocks there are."""

import os
import shutil
import subprocess

import pytest

from oracle import bf1_oracle as orc

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2608_20427_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdint>
#include "bf1_route.h"
int main() {
    long long L, j;
    while (std::scanf("%lld %lld", &L, &j) == 2) {
        std::printf("%lld", (long long)(bf1::route_row_start(j + 1, L) - bf1::route_row_start(j, L)));
        for (int32_t o = (int32_t)j; o >= 0; o = bf1::route_next_offset(o, (int32_t)L))
            std::printf(" %lld", j - o);
        std::printf("\n");
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("walk")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-O1", "-fsanitize=undefined", "-fno-sanitize-recover", "-std=c++17", "-I", CSRC, str(src),
                    "-o", str(exe)], check=True)

    def run(pairs):
        text = "".join(f"{L} {j}\n" for L, j in pairs)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        return [[int(x) for x in line.split()] for line in out]
    return run


@pytest.mark.parametrize("L", [0, 1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 500])
def test_walk_is_the_route(walk, L):
    js = list(range(0, 530)) + [2**r + d for r in range(10, 18) for d in (-1, 0, 1)] + [2**18 - 1]
    for j, (size, *blocks) in zip(js, walk([(L, j) for j in js])):
        want = sorted(orc.route(j, L))
        assert blocks == want and size == len(want), (j, L)


def test_walk_with_every_block_local(walk):
    # L past every block, up to the largest the interface takes
    for j, (size, *blocks) in zip((0, 1, 5, 700), walk([(2**31 - 1, j) for j in (0, 1, 5, 700)])):
        assert blocks == list(range(j + 1)) and size == j + 1
