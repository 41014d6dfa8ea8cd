"""Grids of the QK contractions at HIP's bound (a launch has fewer than 2^32 threads): grid_parts of csrc/sk_grid.h,
compiled for the host, covers every workgroup once and in order with launches below the bound."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_03994_amd", "csrc")
MAIN = """
#include <cstdio>
#include <cstdlib>
#include "sk_grid.h"
int main(int, char **v) {
  sk::grid_parts(atoll(v[1]), [](uint32_t b, uint32_t n) { printf("%u %u\\n", b, n); });
}
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def run(blocks):
        out = subprocess.run([str(d / "main"), str(blocks)], check=True, capture_output=True, text=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


# nine matrices of 1 x 2^19 with 256 vectors: 8192 workgroups per row
@pytest.mark.parametrize("blocks", [0, 1, 2 ** 23, 2 ** 23 + 1, 2 ** 24, 9 * 256 * 8192, 2 ** 32 - 1])
def test_grid_parts(blocks, parts):
    at = 0
    for first, count in parts(blocks):
        assert first == at and 0 < count and count * 256 < 2 ** 32
        at += count
    assert at == blocks
