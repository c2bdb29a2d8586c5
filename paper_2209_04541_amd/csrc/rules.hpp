// Index arithmetic and dispatch rules that need no device: host-only types, so
// they can be checked on the CPU.
#pragma once

#include <cstdint>

namespace pgabb {

// Middle of two positions lo <= hi of one array.  A block's columns have up to
// 2^31 - 1 positions, whose sums do not fit 32 bits.
constexpr int32_t halfway(int32_t lo, int32_t hi) { return lo + ((hi - lo) >> 1); }

}  // namespace pgabb
