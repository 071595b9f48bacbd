// Host arithmetic that lays a call's work out over workgroups, from the bounds
// the caller gives. Plain integers and doubles without HIP, so that it can be
// compiled and tested alone. Bounds may lie anywhere in the int32 range, so
// block counts are taken in 64 bits.
#pragma once

#include <algorithm>
#include <cstdint>

namespace bros {

// Blocks of the longest context a call can meet: its bound in tokens, and what a table row holds.
inline int32_t longest_blocks(int32_t max_ctx, int32_t max_blocks_per_seq) {
  const int64_t blocks = ((int64_t)max_ctx + 15) / 16;
  return (int32_t)std::max<int64_t>(1, std::min<int64_t>(blocks, max_blocks_per_seq));
}

}  // namespace bros
