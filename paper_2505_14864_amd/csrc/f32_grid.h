// Which workgroup takes which tile of an fp32 row product.  Plain C++, so that the host can walk a grid tile by tile.
#pragma once

#include <stdint.h>

namespace dynmo {

constexpr int64_t kMaxWidth = 1 << 20;        // of a grid that need not be wider: its width in threads is a 32-bit number
constexpr int64_t kMaxList = (1 << 24) - 8;   // workgroups of a list, of 256 threads each: fewer than 2^32 threads in a dimension

constexpr int64_t tiles_of(int64_t n, int tile) { return (n + tile - 1) / tile; }

// A list, of which every XCD takes a contiguous eighth, so that its L2 holds the weights of an expert or two and the rows that go
// with them; column tiles side by side in all XCDs made each of them fetch everything (us before / so, 1500 516 1030 8 2: gate/up 90 /
// 83, down 54 / 48, dA 60 / 56, gradients, of which dX, 182 / 176; 2048 1024 1024 8 2 +-1 %).  Where the list would be too
// long for one dimension: row tiles on y, column tiles on x and z.
struct RowGrid {
  unsigned x, y, z;
  bool list;
};
constexpr RowGrid row_grid(int64_t cols, int64_t rows) {
  const int64_t tiles = cols * rows;
  if (tiles <= kMaxList) return {(unsigned)((tiles + 7) / 8 * 8), 1, 1, true};
  const int64_t width = cols < kMaxWidth ? cols : kMaxWidth;
  return {(unsigned)width, (unsigned)rows, (unsigned)((cols + width - 1) / width), false};
}

// The tile of workgroup (x, y, z) of a grid of that kind, `width` wide; false if it has none.  `rows` are the row tiles that
// there are, at most those that the grid was made for.
constexpr bool tile_of_workgroup(bool list, unsigned x, unsigned y, unsigned z, unsigned width, int64_t rows, int64_t cols, int* row,
                                 int* col) {
  int64_t r = y, c = (int64_t)z * width + x;
  if (list) {  // workgroup x runs on XCD x % 8
    const int total = (int)(rows * cols), eighth = (total + 7) / 8, slot = (int)(x >> 3);
    if (slot >= eighth) return false;
    const int at = (int)(x & 7) * eighth + slot;
    r = at / (int)cols;
    c = at - (int)r * (int)cols;
  }
  *row = (int)r;
  *col = (int)c;
  return r < rows && c < cols;
}

}  // namespace dynmo
