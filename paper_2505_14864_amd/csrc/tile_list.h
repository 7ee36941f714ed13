// Which tile of a bf16 row product's list a workgroup of ffn_tile.hip takes.  Plain C++, so that the host can walk a list.
#pragma once

#include <stdint.h>

namespace dynmo {

constexpr int kOneEach = 256;     // tiles: one per compute unit
constexpr int kNearlyTwo = 448;

struct TileList {
  int group;           // consecutive tiles that go to one XCD where they go in runs
  uint32_t inv_group;  // 2^31 / group, rounded up: (2 x * inv_group) / 2^32 is x / group, of any x for a power of two, else below 2^23
  unsigned blocks;     // workgroups
};
// `tiles`: the most that there can be; `longest`: the group of 1024 and more; `walk`: tiles per workgroup
constexpr TileList tile_list(int tiles, int longest = 16, int walk = 1) {
  const int group = tiles >= 1024 ? longest : tiles >= 128 ? tiles / 64 : 1, run = 8 * group * walk;
  return {group, ((1u << 31) + group - 1) / group, (unsigned)(((int64_t)tiles + run - 1) / run * 8 * group)};
}
constexpr int run_of(const TileList& l, int slot) { return (int)((uint64_t)(2 * (uint32_t)slot) * l.inv_group >> 32); }

// The position in the list of workgroup `block` (XCD block % 8), `total` tiles long; from `total` on if it has none.  Tiles of
// rows x cols; `one_each`: no expert has more than one row tile.
//
// Up to a tile per compute unit, and up to two where that is even, every XCD takes an eighth of the list: its tiles share operand tiles
// in its L2, and those small products are bound by what has to pass between the L2s and memory (the dX of 8 experts, 1200 rows, 520 x
// 1032: 71 MB in runs of three tiles, of 22 that it needs).  Runs of `group` / eighths, mean of the times relative to runs:
//   up to 256 tiles   128 x 256 tiles 0.92 (9 products), 128 x 128 0.95 (80), 64 x 64 0.95 (163), none over 1.05
// With a second tile on some compute units an eighth of well filled row tiles is slower than the same tiles spread over all XCDs, so
// from there on it is right only where the tiles are alike:
//   128 x 256, 257 to 448 tiles: runs (E = 8, 121 rows, 424 x 12160, dA 22.6 / 28.6 us; 64, 4992, 2048 x 1024, dA 83 / 93); above, eighths
//     (56, 68 rows, 1312 x 3840, dA 66 / 54; 512 tiles of 64 experts 65 / 55)
//   128 x 128: eighths where no expert has two row tiles (E = 48, 384 rows, dA 11.2 / 9.7) or an expert has half an XCD and more (2, 9083
//     rows, down 33 / 28; 14, 4533, gate/up 47 / 43); else runs (32, 2496 rows, 1000 x 2048, dX 131 / 138, 512 x 1024, dA 17.6 / 19.8)
//   64 x 64: the same, with more than an XCD per expert (E = 2, 2673 rows, down 31 / 24; 3, 4766, gate/up 47 / 41); else runs of eight,
//     which are dealt evenly (8, 360 rows, 2048 x 1024: dX 19.8 / 21.9 / 18.1; in runs of `group` a quarter of the chip can wait for
//     the last run)
// More tiles go in runs of `group` (1280 tiles of 128 x 256, dX of 64 experts: 193 / 200).
constexpr int list_position(const TileList& l, unsigned block, int total, int rows, int cols, int experts, bool one_each) {
  const int slot = (int)(block >> 3), xcd = (int)(block & 7), eighth = (total + 7) >> 3;
  const int run = run_of(l, slot);
  const bool even = cols > 128 ? total > kNearlyTwo : one_each || experts <= (rows == 64 ? 7 : 16);
  const bool eighths = total <= kOneEach || (total <= 2 * kOneEach && even);
  int pos = eighths ? (slot < eighth ? xcd * eighth + slot : total) : (run * 8 + xcd) * l.group + slot - run * l.group;
  if (rows == 64) {
    const int dealt = (total >> 6) * 8, over = slot - dealt, last = (total - 8 * dealt + 7) >> 3;
    const int by_eight = over < 0 ? (slot >> 3) * 64 + xcd * 8 + (slot & 7) : over < last ? 8 * dealt + xcd * last + over : total;
    pos = !eighths && total <= 2 * kOneEach ? by_eight : pos;
  }
  return pos;
}

}  // namespace dynmo
