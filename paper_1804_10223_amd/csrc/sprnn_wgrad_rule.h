// Which of the ways to the weight gradient a call takes: estimates of their times, plain host arithmetic.
//
//   product        one tiled product on the matrix cores, sampled at the nonzeros (sprnn_wgrad.hip): work for every element
//                  of the dense matrix, little per vector
//   lane sums      one accumulator per nonzero in the lanes that hold it in the forward pass (sprnn_wgrad_lanes.hip): work
//                  for the nonzeros only, and all of h to every workgroup in every timestep
#ifndef SPRNN_WGRAD_RULE_H_
#define SPRNN_WGRAD_RULE_H_

#include <algorithm>
#include <cstdint>

namespace sprnn {

struct WGradTile {
  int rows = 0, cols = 0;            // shape of one workgroup's part of the dense product
};

// The grid of tiles and how the eight XCDs share it: parts_m x (8 / parts_m) rectangles.
struct TileGrid {
  int tiles_m, tiles_n, parts_m;
};

// The division among the XCDs whose largest rectangle (`*most` tiles) has the fewest tiles, then the fewest rows and
// columns to fetch.
inline TileGrid tile_grid(int rows, int cols, WGradTile tile, int* most) {
  TileGrid best = {(rows + tile.rows - 1) / tile.rows, (cols + tile.cols - 1) / tile.cols, 1};
  long long least = 0;
  for (int parts = 1; parts <= 8; parts *= 2) {
    const int m = (best.tiles_m + parts - 1) / parts, n = (best.tiles_n + 8 / parts - 1) / (8 / parts);
    const long long cost = (long long)m * n * 100000 + (long long)m * tile.rows + (long long)n * tile.cols;
    if (parts == 1 || cost < least) { least = cost; best.parts_m = parts; *most = m * n; }
  }
  return best;
}

// Clocks of the product: 8000 to start a workgroup and to store its nonzeros, and per slab of 32 vectors 400 around the
// barrier and 0.1 per element of the tile; an XCD works through its rectangle in turns of one tile per CU.
inline double product_clocks(int rows, int cols, WGradTile tile, int num_cus, int64_t slabs) {
  int most = 0;
  (void)tile_grid(rows, cols, tile, &most);
  const int per_xcd = std::max(num_cus / 8, 1);
  return (double)((most + per_xcd - 1) / per_xcd) * (8000.0 + (double)slabs * (400.0 + 0.1 * tile.rows * tile.cols));
}

// The tile shape for a matrix of this size on a device with this many CUs, at 16 slabs.  (Each of the four shapes is the
// fastest somewhere: 64 x 64 where there are few tiles, 128 x 192 where the 128 x 128 tiles of a matrix just exceed the
// CUs: 2304 x 2304 93 against 73 us, 4096 x 1024 52 against 70.)
inline WGradTile choose_weight_gradient_tile(int rows, int cols, int num_cus) {
  constexpr int shapes[][2] = {{64, 64}, {64, 128}, {128, 128}, {128, 192}};
  WGradTile best;
  double least = 0.0;
  for (const auto& s : shapes) {
    WGradTile t;
    t.rows = s[0];
    t.cols = s[1];
    const double cost = product_clocks(rows, cols, t, num_cus, 16);
    if (best.rows == 0 || cost < least) { best = t; least = cost; }
  }
  return best;
}

// A layer's call, as far as the choice of a way depends on it.
struct WGradCall {
  int rows = 0, cols = 0, num_cus = 0;   // of the handle's matrix, of the device
  WGradTile tile;
  int batch = 0;
  int64_t steps = 0;
};

// Microseconds, launch included; a clock above is 0.68 ns as measured (20000 x 20000, 64 vectors 597 us, 256 vectors 1295).
inline double product_us(const WGradCall& c) {
  return 4.0 + product_clocks(c.rows, c.cols, c.tile, c.num_cus, (c.steps * c.batch + 31) / 32) * 0.68e-3;
}

// Microseconds of the lane sums: what a step takes is bringing h to the workgroup in rounds of one 16-byte piece per lane,
// four of them at a time (one batch 0.85 to 1.4 us with everything else in a step, each further one 0.75).  Of 512 lanes,
// whatever the handle's mapping has (384 to 768): the two ways add in different orders, and handles of one matrix are to
// give the same bits.
inline double lane_sums_us(const WGradCall& c) {
  const int64_t rounds = ((int64_t)c.cols * c.batch * 4 / 16 + 511) / 512, batches = std::max<int64_t>((rounds + 3) / 4, 1);
  const double first = c.batch == 1 ? 0.85 : (c.batch == 2 ? 1.4 : (c.batch == 4 ? 1.05 : 1.2));
  return 8.0 + (double)c.steps * (first + 0.75 * (double)(batches - 1));
}

// sprnn_weight_gradient.  Both sides measured, lane sums / product in us: 2304 at 30 %, batch 4, T 16 28 / 14, T 256 285 / 74;
// LSTM 1024 at 20 %, batch 8, T 256 323 / 110; but 5120 at 5 %, batch 4, T 16 37 / 52 (T 256 521 / 332); 8192 at 2 %, batch 1,
// T 64 65 / 110; LSTM 4096 at 4 %, batch 2, T 64 114 / 157; 20000 at 0.5 %, batch 1, T 64 131 / 597; 40000 at 0.1 %, T 16
// 63 / 1788.  (The product counts vectors in 32 bits.)
constexpr int64_t kMostProductVectors = 0x7fffffff - 256;
inline bool lane_sums_are_faster(const WGradCall& c) {
  return c.steps * c.batch > kMostProductVectors || lane_sums_us(c) < product_us(c);
}

}  // namespace sprnn
#endif
