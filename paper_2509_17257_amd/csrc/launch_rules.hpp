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
//   groups (two / four waves, us per product): FP64, 32 columns, sphere 65536, 1535 leaves 789 / 781;
//   95000, 2114 leaves 1087 / 1102; 131072, 3044 leaves 1554 / 1576.  Leaves of up to 32 rows, FP32,
//   4301 of them 2435 / 2346.
//   LDS (32 columns): cube 262144, tables up to 30 KB, FP32 4997 / 5066; cube 99991, 36 KB, BF16, 45
//   columns 1637 / 1651; cube 131072, 43 KB, FP32 2616 / 2403, BF16 1975 / 1822, FP64 4624 / 4573;
//   the same with leaves of up to 100 points, 56 KB, BF16 2385 / 1926.
inline bool leaf_two_waves(int64_t groups, int32_t max_leaf, size_t lds) {
    return groups >= 2048 && max_leaf > 32 && 4 * (lds + 512) <= 163840;
}

// The same for FP32 and BF16 with slabs of `tiles` 16-column tiles.  At up to two tiles 1536 two-wave
// groups fit at a time and 1024 of four waves: two waves also where they take one round and four
// would take a second, if a group's work is short (tables of up to 16 KB, leaves of one chunk:
// with leaves of up to 80 points 79040 points took 558 / 538), and else from two and a half times
// 1024 on.  32 columns, two / four waves: sphere 65536, 1535 leaves FP32 491 / 497, BF16 421 /
// 427; 60000, 1394 leaves 462 / 464, 397 / 404; 52000, 1180 leaves 413 / 406; 95000, 2114 leaves 697 /
// 688, 581 / 572; 105000, 2381 leaves 764 / 760; 131072, 3044 leaves 950 / 960; cube 60000, 1243 leaves,
// tables of 35 KB 945 / 929.
inline bool leaf_two_waves_lp(int64_t groups, int tiles, int32_t max_leaf, size_t lds) {
    if (tiles > 2) return leaf_two_waves(groups, max_leaf, lds);
    const bool one_round = groups >= 1280 && groups <= 1536 && max_leaf > 32 && max_leaf <= 64 && lds <= 16384;
    return one_round || (groups >= 2560 && leaf_two_waves(groups, max_leaf, lds));
}

}  // namespace h2x
