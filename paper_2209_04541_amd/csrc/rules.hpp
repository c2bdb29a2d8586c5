// Index arithmetic and dispatch rules that need no device: host-only types, so
// they can be checked on the CPU.
#pragma once

#include <cstdint>

namespace pgabb {

// Middle of two positions lo <= hi of one array.  A block's columns have up to
// 2^31 - 1 positions, whose sums do not fit 32 bits.
constexpr int32_t halfway(int32_t lo, int32_t hi) { return lo + ((hi - lo) >> 1); }

// Whether `ends` ends of edges over n vertices are counted by their low bits,
// one value of the high bits after the other (build.hip: k_degrees_hi), and not
// sorted by all bits and counted in runs.  The first clears and reads 2^low_bits
// counters in LDS per value, whatever the ends that share it, so it pays only
// from some 24,576 ends a value on.  Builds by low bits / in runs, us, uniform
// pairs at 1 K, 8 K, 16 K, 32 K and 128 K ends a value: 2^20 vertices 694 / 546,
// 650 / 613, 683 / 688, 832 / 866, -; 2^22 1032 / 706, 1202 / 1100, 1719 / 1623,
// 2696 / 2626, 8981 / 9131; 2^24 2003 / 1428, -, 6112 / 5621, 10429 / 10301, -.
// R-MAT scale 20, 31 K 782 / 814; scale 21, 62 K 2190 / 2296, 122 K 3928 / 4249.
// 70,000 pairs over 2^26 vertices took 13.4 ms by low bits, 3.8 in runs.
constexpr int64_t kEndsPerHigh = 24576;
constexpr bool degrees_by_low_bits(int64_t ends, int64_t n, int low_bits) {
    return ends >= kEndsPerHigh * ((n >> low_bits) + 1);
}

// Work items a wave takes per work-counter update: what the caller asked for,
// else the chosen number, times the parts of a launch that is split by
// staged-list length (each part counts a share of the items it takes).
constexpr int grab_items(int asked, int chosen, int parts) { return asked > 0 ? asked : chosen * parts; }

}  // namespace pgabb
