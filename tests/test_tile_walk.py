"""The persistent walk of the batch kernels over their items, compiled for the host:
every item is taken once, and no workgroup takes two where each could take one."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2002_03644_amd", "csrc", "hlbm_device.hpp")

HARNESS = r"""
#include <algorithm>
#define __device__
#define __forceinline__ inline
using std::min;
struct Dim { int x; };
static Dim gridDim, blockIdx;
%s
extern "C" void walk(int n, int grid, int *taken, int *most) {
  gridDim.x = grid;
  *most = 0;
  for (int b = 0; b < grid; ++b) {
    blockIdx.x = b;
    const TileWalk w = tile_walk(n);
    int count = 0;
    for (int it = w.first; it < w.end; it += w.step, ++count)
      if (it >= 0 && it < n) ++taken[it];
      else taken[0] += 1000;
    *most = std::max(*most, count);
  }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    s = open(SRC).read()
    body = s[s.index("struct TileWalk {"):]
    body = body[:body.index("\n}\n") + 3]
    d = tmp_path_factory.mktemp("walk")
    src, so = str(d / "walk.cpp"), str(d / "walk.so")
    with open(src, "w") as f:
        f.write(HARNESS % body)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", src, "-o", so])
    return ctypes.CDLL(so).walk


def run(walk, n, grid):
    taken, most = np.zeros(n, np.int32), ctypes.c_int()
    walk(n, grid, taken.ctypes.data_as(ctypes.c_void_p), ctypes.byref(most))
    assert (taken == 1).all(), (n, grid)
    return most.value


@pytest.mark.parametrize("n", [1, 5, 7, 8, 9, 63, 444, 812, 966, 1000, 1023, 1024])
def test_one_item_each(walk, n):
    """A grid of as many workgroups as items."""
    assert run(walk, n, n) == 1


@pytest.mark.parametrize("grid", [1, 7, 8, 256, 512, 768, 1280])
def test_rounds(walk, grid):
    """Resident workgroups with more items: as few rounds as there can be."""
    for n in (grid, grid + 1, grid + 7, 2 * grid - 1, 2 * grid, 3 * grid + 5, 17 * grid + 3):
        assert run(walk, n, grid) == -(-n // grid), (n, grid)
