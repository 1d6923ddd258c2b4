// launch_rules.h -- host rules of the launchers that are plain arithmetic (no HIP).
#pragma once
#include <algorithm>

namespace lbm {

// Whether a kernel may store an output at the caller's pointer: device memory of the
// GPU that holds the workspace (own; -1 if unknown).  Anything else that a copy
// reaches, another GPU's memory above all, which a kernel may not have access to, is
// written by a copy.
inline bool stores_directly(bool device_memory, int device, int own) {
  return device_memory && own >= 0 && device == own;
}

// blocks of 256 threads for a box of `side` nodes a side, a node per thread
inline long long box_blocks(double side) { return ((long long)(side * side * side) + 255) / 256; }

// Blocks per particle of a launch whose grid rows are `rows` particles, all with as many
// as the largest box takes (`side`); `own`: what their own boxes would take together.
// Where the boxes are much alike, a node per thread.  Else most blocks would find nothing to
// do, which takes 0.4 to 1.3 ns of the launch each: PARTICLE_BLOCKS in all (128 per CU),
// and the blocks stride over a box that is larger.
constexpr long long PARTICLE_BLOCKS = 32768;
inline int particle_blocks(long long rows, int side, long long own) {
  const long long full = box_blocks(side), r = std::max(1ll, rows);
  if (r * full <= std::max(4 * own, PARTICLE_BLOCKS)) return (int)full;
  return (int)std::max(1ll, std::min(full, PARTICLE_BLOCKS / r));
}

// The same where they share a flat grid with `fluid_blocks` others: a grid dimension takes
// 2^32 - 1 threads and is cut short beyond, without an error.
constexpr long long GRID_BLOCKS = 0xFFFFFFFFll / 256;
inline int particle_blocks_flat(long long fluid_blocks, long long rows, int side, long long own) {
  const long long room = (GRID_BLOCKS - fluid_blocks) / std::max(1ll, rows);
  return (int)std::max(1ll, std::min((long long)particle_blocks(rows, side, own), room));
}

// Whether the mask update searches the particles in each block (k_mask, one launch) or
// claims nodes in memory (three): by the most particles of one simulation, as a search
// costs about 6 ps per particle and block, the claims 3 to 5 ns per block.  Search against
// claims in a step: 500 spheres of radius 4 32 and 37 us, 500 of radius 8 97 and 102, 700 of
// radius 4 45 and 48, 1,000 of radius 8 282 and 192, 4,096 of radius 4 884 and 224.
// After a push, whose many fresh nodes the claims visit in a pass of their own: 1,000 of
// radius 8 579 and 682, 4,096 of radius 4 886 and 643.
inline bool mask_by_search(int np_max, bool pushed) { return np_max <= (pushed ? 1024 : 512); }

}  // namespace lbm
