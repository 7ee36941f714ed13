"""The tile lists of the bf16 row products, walked workgroup by workgroup on the host (csrc/tile_list.h is plain C++)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_14864_amd", "csrc")
WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "tile_list.h"
using namespace dynmo;
// rows and columns of a tile, the most tiles that there can be
int main(int, char** a) {
  const int rows = atoi(a[1]), cols = atoi(a[2]), limit = atoi(a[3]);
  const TileList l = tile_list(limit);
  for (int experts : {1, 7, 8, 16, 17, 64})
    for (int one_each = 0; one_each < 2; ++one_each)
      for (int total = 0; total <= limit; total += limit < 2000 || total + 1 == limit ? 1 : limit > 100000 ? limit / 3 - 1 : 61) {
        std::vector<unsigned char> seen(total, 0);
        for (unsigned b = 0; b < l.blocks; ++b) {
          const int pos = list_position(l, b, total, rows, cols, experts, one_each);
          if (pos < 0) return printf("total %d, workgroup %u: %d\n", total, b, pos), 1;
          if (pos < total && seen[pos]++) return printf("total %d: tile %d twice\n", total, pos), 1;
        }
        for (int i = 0; i < total; ++i)
          if (!seen[i]) return printf("total %d: tile %d never\n", total, i), 1;
      }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("list")
    (d / "walk.cpp").write_text(WALK)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(d / "walk.cpp"), "-o", str(d / "walk")], check=True)
    return str(d / "walk")


@pytest.mark.parametrize("rows,cols", [(64, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("limit", [1, 127, 128, 255, 256, 449, 512, 600, 1023, 1024, 5000, 20000001])
def test_every_tile_has_one_workgroup(walk, rows, cols, limit):
    r = subprocess.run([walk, str(rows), str(cols), str(limit)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
