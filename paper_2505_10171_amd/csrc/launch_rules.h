// launch_rules.h -- host rules of the launchers that are plain arithmetic (no HIP).
#pragma once
#include <algorithm>

namespace lbm {

// blocks of 256 threads that one dimension of a grid takes (2^32 - 1 threads)
constexpr long long GRID_BLOCKS = 0xFFFFFFFFll / 256;

// Blocks per particle that fill its capillary box (`side` nodes a side) when those of
// `rows` particles share a flat grid with `fluid_blocks` others: a node per thread, or
// what the grid has room for (the blocks stride over the box): 501 particles of which
// one has R = 102 would take 17.4 M blocks of the 16.8 M.
inline int capillary_blocks(long long fluid_blocks, long long rows, int side) {
  const long long nodes = (long long)side * side * side;
  const long long room = (GRID_BLOCKS - fluid_blocks) / std::max(1ll, rows);
  return (int)std::max(1ll, std::min((nodes + 255) / 256, room));
}

}  // namespace lbm
