// What one launch holds.
#pragma once

#include <cstdint>

namespace fea {

// Rows that one launch takes in grid.x when a row is `blocks` workgroups of
// `threads`: a dispatch counts its threads in 32 bits, and a launch of 2^32 or
// more is refused or, silently, runs only its low 32 bits' worth.
constexpr int64_t grid_rows(int64_t blocks, int threads) {
  const int64_t rows = ((int64_t(1) << 32) - 1) / threads / blocks;
  return rows > 1 ? rows : 1;
}

}  // namespace fea
