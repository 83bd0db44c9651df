// Rules that choose a launch shape from sizes alone (host code, no device types).
#pragma once

#include <cstddef>
#include <cstdint>

namespace h2x {

// Leaf stage, one contraction per leaf: two waves per (leaf, slab) load every operand once; four have
// two row groups (or column halves) that load one operand twice, but half the serial rounds and
// twice the waves.  Two win where they fill the chip twice (1024 such groups fit at a time by their
// registers) and hold three or four row tiles, as long as the LDS of a group, its table of near
// rows, lets four of them share a CU (160 KB): with fewer, a CU's four SIMDs hold six or four
// waves of the two-wave form and twice as many of the other.
//   groups (two / four waves, us per product, FP32, 32 columns unless said): sphere 131072, 3044
//   leaves 950 / 971; sphere 65536, 64 columns, 1543 leaves 770 / 765; leaves of up to 32 rows, 4301
//   of them 2435 / 2346.  FP64, 32 columns: sphere 65536 789 / 781, 131072 1554 / 1576.
//   LDS (32 columns): cube 262144, tables up to 30 KB 4997 / 5066; cube 99991, 36 KB, BF16, 45 columns
//   1644 / 1650; cube 131072, 43 KB 2616 / 2403, BF16 1975 / 1822, FP64 4624 / 4573; the same
//   with leaves of up to 100 points, 56 KB, BF16 2385 / 1926.
inline bool leaf_two_waves(int64_t groups, int32_t max_leaf, size_t lds) {
    return groups >= 2048 && max_leaf > 32 && 4 * (lds + 512) <= 163840;
}

}  // namespace h2x
