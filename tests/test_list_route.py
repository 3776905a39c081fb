"""The rule that chooses between the two routes of a tile-list build
(csrc/list_route.h), built for the CPU: models and frames measured on either
side of it. A small model in a large frame is sorted: comparing reads the
square of the tiles."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include "list_route.h"
int main(int, char** a) {
  std::printf("%d", (int)gs::compares_all(std::atoll(a[1]), std::atoll(a[2]), std::atoll(a[3])));
}
"""


@pytest.fixture(scope="module")
def compares(tmp_path_factory):
    d = tmp_path_factory.mktemp("list_route")
    (d / "t.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_02851_amd", "csrc"),
                           str(d / "t.cpp"), "-o", str(d / "t")])
    return lambda *a: subprocess.check_output([str(d / "t")] + [str(x) for x in a]) == b"1"


@pytest.mark.parametrize("n,views,tiles", [(1, 1, 1), (1000, 1, 64), (16384, 1, 480), (8192, 1, 3600), (2000, 1, 8160),
                                           (8192, 4, 2500), (2000, 64, 3136), (100, 1, 9702)])
def test_compared(compares, n, views, tiles):
    assert compares(n, views, tiles)


@pytest.mark.parametrize("n,views,tiles", [(16385, 1, 1), (100, 1, 9800), (16, 4, 10000), (3000, 1, 8160), (12000, 1, 3600),
                                           (12000, 4, 2500), (4096, 64, 1024), (1000, 2, 16320), (1000, 1, 32400),
                                           (500, 8, 65280), (1, 256, 1 << 31), (16384, 256, 1)])
def test_sorted(compares, n, views, tiles):
    assert not compares(n, views, tiles)
