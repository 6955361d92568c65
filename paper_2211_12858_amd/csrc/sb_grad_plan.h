// Work split of the register softmax kernel for wide rows (host side, from the
// shape alone: no HIP call).
#ifndef SB_GRAD_PLAN_H_
#define SB_GRAD_PLAN_H_
#include <cstdint>

namespace sb {

constexpr int WIDE_C = 32;  // columns per lane
constexpr int WIDE_MAX_WAVES = 16;
constexpr int WIDE_MAX_D = 64 * WIDE_MAX_WAVES;
// Blocks for 256 CUs of 16 waves, which fit whatever the compiler makes of a block
// of 16.  (20, as many as some instances' registers leave room for, put two blocks
// of 9 or 10 waves on a CU: 300,007 x 513 with hessians 658 us, 629 so; 95,001 x 513
// 255 and 206; 300,007 x 190 without hessians 157 and 130.)
constexpr int WIDE_CUS = 256;
constexpr int WIDE_CU_WAVES = 16;

struct WidePlan {
  int rows;   // rows per tile: 64 x 32 columns per wave, or 32 x 64 past 512 columns
  int waves;  // per block
  int tiles;
  int grid;   // blocks, all with the same number of tiles but the last ones
};

// As many blocks as fit on MI355X at once and at most n_parts.  Block b's
// column sums are norm partial b, so the blocks set the order in which the norms are
// added: they follow from the shape, not from the device the call finds.
constexpr WidePlan wide_plan(int64_t n, int32_t d, int32_t n_parts) {
  WidePlan p{};
  p.rows = d <= WIDE_C * WIDE_MAX_WAVES ? 64 : 32;
  const int cols = WIDE_C * (64 / p.rows);
  p.waves = (d + cols - 1) / cols;
  p.tiles = (int)((n + p.rows - 1) / p.rows);
  int most = WIDE_CUS * (WIDE_CU_WAVES / p.waves);
  if (most > n_parts) most = n_parts;
  if (most > p.tiles) most = p.tiles;
  const int per = (p.tiles + most - 1) / most;
  p.grid = (p.tiles + per - 1) / per;
  return p;
}

}  // namespace sb
#endif
