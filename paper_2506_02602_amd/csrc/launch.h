// launch.h -- block sizes that a mechanism's LDS allows (host code, no HIP).
#pragma once
#include <cstddef>

namespace chemgpu {

// The compaction slots of a block: (N + 4) doubles and 6 ints a lane.
constexpr size_t slot_bytes(int ns, int block) { return (size_t)block * ((ns + 4) * 8 + 6 * 4); }
constexpr size_t kSlotLimit = 65536;
constexpr bool block_fits(int ns, int block) { return slot_bytes(ns, block) <= kSlotLimit; }

// A default block, halved until its slots fit: a call that names no block is
// refused for no mechanism.
constexpr int fit_block(int ns, int block) {
  while (block > 64 && !block_fits(ns, block)) block /= 2;
  return block;
}

// The size rule's block (chemgpu.hip): 256, or 128 where a cell takes a whole
// wave of the cooperative kernel.
constexpr int size_block(int ns, bool wide) { return fit_block(ns, wide ? 128 : 256); }

}  // namespace chemgpu
