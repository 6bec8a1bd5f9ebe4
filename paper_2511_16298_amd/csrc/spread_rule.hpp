// Host-only rules of the spread passes: which calls take them and how their
// row pass is cut.  Free of HIP, so that they can be tested on any host.
#pragma once

#include <stdint.h>

namespace ss {

// Gaussians per workgroup of the column pass.
constexpr uint32_t kColumnItems = 2048;

// What the frames of a call have in common for the spread passes.
struct SpreadShape {
  uint32_t max_tx = 0, max_ty = 0;  // most tile columns and rows of a frame
  uint64_t max_tiles = 0;           // most tiles of a frame
  uint64_t sum_tx = 0;              // tile columns of all frames
  uint64_t col_blocks = 0;          // column-pass workgroups
  void add(uint32_t n, uint32_t tx, uint32_t ty) {
    max_tx = tx > max_tx ? tx : max_tx;
    max_ty = ty > max_ty ? ty : max_ty;
    const uint64_t tiles = static_cast<uint64_t>(tx) * ty;
    max_tiles = tiles > max_tiles ? tiles : max_tiles;
    sum_tx += tx;
    col_blocks += (n + kColumnItems - 1) / kColumnItems;
  }
};

// Column items per tile column, about.  The pairs are not known on the host:
// half the capacity where the caller has sized it closely, but at most three
// items per Gaussian (two to two and a half are usual), so that room to spare
// does not count as work.
inline uint64_t mean_column_items(uint32_t n, uint32_t capacity, const SpreadShape& sh) {
  if (sh.sum_tx == 0) return 0;
  const uint64_t room = capacity / 2, most = 3ull * n;
  return (room < most ? room : most) / sh.sum_tx;
}

// Whether the spread passes are the faster way for a call that they can serve
// at all.  Against the digit passes (us, digit / spread; splats of 1-3, about
// 7 and 16-32 px):
//  - Axes of 8 to 160 tiles.  A workgroup's bit matrix has a row per digit, so
//    long axes cost LDS and steps whatever the items (240 x 135 tiles, 1.5M
//    Gaussians: 219 / 237; 2.5M small ones: 196 / 265; 256 x 256, 1M: 176 /
//    205; 160 x 90, 1M: 159 / 134), and short ones leave a pass that hardly
//    sorts (256 x 1, 200k: 81 / 94; 100 x 4 with large splats: 122 / 128; 40 x
//    8: 128 / 119).
//  - Up to 256 tiles the digit path has one pass over the pairs.  A single
//    frame of 12 tiles an axis still gains from 2^17 Gaussians (16 x 16: 89 /
//    81, 119 / 111), below that unless its splats are large for the image (50k:
//    65 / 61, 90 / 93); a batch of such frames where its columns are well
//    filled (128 frames of 10,000: 218 / 225, of 20,000: 300 / 261).
//  - A row-pass workgroup per tile column is too many for too few items where
//    thousands of columns are thinly filled (64 full-HD frames of 5,000
//    Gaussians: 128 / 175, of 15,000: 175 / 206, of 20,000: 222 / 221, of
//    50,000: 394 / 336).
//  - Splats that hardly leave their tile, by the million, on more than 120
//    tiles an axis (128 x 128, splats of 1-3 px, 1M: 127 / 122, 1.2M: 146 / 156,
//    2M: 185 / 205; 120 x 68, 2M: 185 / 183).
inline bool spread_pays(uint32_t n, uint32_t n_frames, uint32_t capacity, const SpreadShape& sh) {
  const uint32_t longest = sh.max_tx > sh.max_ty ? sh.max_tx : sh.max_ty;
  const uint32_t shortest = sh.max_tx > sh.max_ty ? sh.max_ty : sh.max_tx;
  if (n == 0 || longest > 160 || shortest < 8) return false;
  const uint64_t mean = mean_column_items(n, capacity, sh);
  if (sh.max_tiles <= 256) {
    if (shortest < 12) return false;
    return n_frames == 1 ? n >= (1u << 17) || capacity < 8ull * n : n >= (1u << 19) && mean >= 2048;
  }
  if (longest > 120 && n >= (1u << 20) && capacity < 2ull * n) return false;
  return sh.sum_tx <= 2048 || mean >= 512;
}

// Items per workgroup of the row pass.  Large ones (4,096 items, 1,024
// threads) have the fewest workgroups to look back over (6M-Gaussian frame
// 478 -> 456 us against 2,048, full HD 146 -> 145, 64-frame batch 2.59 ->
// 2.46 ms), while their LDS lets two share a CU: up to 80 tile rows.  But
// every tile column has a workgroup of its own, however few its items, so
// where the columns are more than the GPU holds large workgroups at once
// (512), their share of the items decides.  Seven frames of 93,000 Gaussians
// (3,300 items a column) take 134 us with 4,096, 127 with 2,048, 130 with
// 1,024 items; 39 of 175,000 (6,100) 475 / 471 / 487; 46 of 27,000 (950) 250 /
// 225 / 220; 15 of 18,000 (630) 121 / 113 / 107.
inline uint32_t row_pass_items(uint32_t n, uint32_t capacity, const SpreadShape& sh) {
  const uint64_t mean = mean_column_items(n, capacity, sh);
  if (sh.sum_tx > 512) {
    if (mean < 1024) return 1024;
    if (mean < 8192) return 2048;
  }
  return sh.max_ty <= 80 ? 4096 : 2048;
}

}  // namespace ss
