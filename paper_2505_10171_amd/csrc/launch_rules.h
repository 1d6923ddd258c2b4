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

// Whether a kernel may store an output at the caller's pointer: device memory of the
// GPU that holds the workspace (own; -1 if unknown).  Anything else that a copy
// reaches, another GPU's memory above all, which a kernel may not have access to, is
// written by a copy.
inline bool stores_directly(bool device_memory, int device, int own) {
  return device_memory && own >= 0 && device == own;
}

}  // namespace lbm
