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

// Blocks of 256 per particle of a launch whose grid rows are `rows` particles and whose
// boxes have at most `side` nodes a side: a node per thread, but no more than PARTICLE_BLOCKS
// in all (128 per CU); the blocks stride over a box that is larger.  The largest sphere
// of the context sizes the rows of all, and a block that finds nothing to do takes
// 0.4 to 1.3 ns of the launch all the same.
constexpr int PARTICLE_BLOCKS = 32768;
inline int particle_blocks(long long rows, int side) {
  const long long nodes = (long long)side * side * side;
  const long long most = std::max(1ll, PARTICLE_BLOCKS / std::max(1ll, rows));
  return (int)std::max(1ll, std::min((nodes + 255) / 256, most));
}

// Whether the mask update searches the particles in each block (k_mask, one launch) or
// claims nodes in memory (three): by the most particles of one simulation, as a search
// costs about 6 ps per particle and block, the claims 3 to 5 ns per block.  Search against
// claims: 500 spheres of radius 4 32 and 37 us, 500 of radius 8 97 and 102, 700 of radius
// 4 45 and 48, 1,000 of radius 8 282 and 192, 4,096 of radius 4 884 and 224.
inline bool mask_by_search(int np_max) { return np_max <= 512; }

}  // namespace lbm
