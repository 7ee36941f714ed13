"""The grids of the fp32 row products, walked workgroup by workgroup on the host (csrc/f32_grid.h is plain C++)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14864_amd", "csrc")
WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "f32_grid.h"
using namespace dynmo;
// columns, row tiles that the grid is made for, row tiles that there are
int main(int, char** a) {
  const int64_t cols = atoll(a[1]), limit = atoll(a[2]), rows = atoll(a[3]);
  const RowGrid g = row_grid(cols, limit);
  std::vector<unsigned char> seen(cols * rows, 0);
  for (unsigned z = 0; z < g.z; ++z)
    for (unsigned y = 0; y < g.y; ++y)
      for (unsigned x = 0; x < g.x; ++x) {
        int r = 0, c = 0;
        if (!tile_of_workgroup(g.list, x, y, z, g.x, rows, cols, &r, &c)) continue;
        if (r < 0 || r >= rows || c < 0 || c >= cols) return printf("workgroup %u %u %u: tile %d %d\n", x, y, z, r, c), 1;
        if (seen[r * cols + c]++) return printf("tile %d %d twice\n", r, c), 1;
      }
  for (int64_t i = 0; i < cols * rows; ++i)
    if (!seen[i]) return printf("tile %lld never\n", (long long)i), 1;
  printf("%u %u %u\n", g.x, g.y, g.z);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "walk.cpp").write_text(WALK)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(d / "walk.cpp"), "-o", str(d / "walk")], check=True)
    return str(d / "walk")


def dims(walk, cols, limit, rows):
    r = subprocess.run([walk, str(cols), str(limit), str(rows)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    return [int(v) for v in r.stdout.split()]


@pytest.mark.parametrize("cols,limit,rows", [(1, 1, 1), (33, 31, 24), (33, 31, 31), (33, 31, 0), ((1 << 21) - 1, 8, 8),
                                             ((1 << 20) + 1, 16, 16), ((1 << 20) + 1, 16, 5), ((1 << 21) + 5, 9, 9), (3, 65535, 65535),
                                             (513, 65535, 11)])
def test_every_tile_has_one_workgroup(walk, cols, limit, rows):
    dims(walk, cols, limit, rows)


@pytest.mark.parametrize("cols,limit", [((1 << 21) - 1, 8), (258111, 65), (1 << 18, 64), ((1 << 20) + 1, 16)])
def test_grids_can_be_launched(walk, cols, limit):
    """2^24 - 8, - 1, 2^24 and 2^24 + 16 tiles: fewer than 2^32 threads in every dimension (workgroups of 256), y and z of 16 bits."""
    x, y, z = dims(walk, cols, limit, limit)
    assert max(x, y, z) * 256 < 1 << 32 and max(y, z) < 1 << 16
