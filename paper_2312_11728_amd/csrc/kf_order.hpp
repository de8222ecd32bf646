// The order in which the length-sorted staged fit (layout 4) runs its tracks.
//
// Groups of kOrderGroup consecutive tracks are sorted by length, longest
// first, and cut into waves of 64.  Within a group the tracks of a wave lie
// close together: they share the cache lines of their hits and results, if the
// group's waves run at the same time and behind one L2.
//
// In a batch larger than the chip holds at once the first wave of every group,
// its 64 longest tracks, goes to the front: the front's waves share blocks (a
// block keeps its LDS until its longest track ends) and run first (a late
// block of long tracks is a tail in which the chip idles).  In a smaller one
// every block starts at once, and the front would only take the group's tracks
// apart (FP64, 50k tracks of 3 to 15 entries: 92.0 us without, 94.5 with one).
// The other waves follow group by group, every second group the other way
// round, so that a block across two groups holds tracks of like lengths.
// Blocks go to the kXcds dies in turn, so they are dealt out such that each
// die walks through a run of consecutive groups of its own.
//
// FP32, 500k tracks, the whole call (us), sorted as a whole / in groups dealt
// out in sets of eight without a front / this: lengths 3 to 15 474 / 329 / 317,
// 3 to 26 with 1% at 26 492 / 557 / 418, nine of ten cut to 8 entries 268 / 432
// / 263.  Two or four waves of each group in front: 322 and 331, 422 and 423,
// 263 and 261; none: 312, 478, 349.  Persistent blocks take their tiles as
// they come, not in turn, and run the waves in line: 492 / 394 / 414, 516 / 509
// / 484, 276 / 338 / 282.
#pragma once

#include "kf_math.hpp"

namespace kf {

constexpr int kOrderGroup = 2048;
constexpr int kGroupWaves = kOrderGroup / 64;
constexpr int kXcds = 8;

// The place of wave v of group g among the waves of n_groups whole groups, run
// in blocks of `per_block` waves (0: in line), with a front of every group's
// first `front` (0 or 1) waves.
KF_HD inline int64_t wave_place(int64_t g, int v, int64_t n_groups, int per_block, int front) {
  if (v < front) return g;
  const int rest = kGroupWaves - front;
  const int64_t n_front = n_groups * front, i = g * rest + ((g & 1) ? kGroupWaves - 1 - v : v - front);
  if (per_block == 0) return n_front + i;
  // the blocks after the front's last one in rows of kXcds: die x runs part x
  // of kXcds equal parts of the waves behind the front
  const int64_t block0 = (n_front + per_block - 1) / per_block;
  const int64_t gap = block0 * per_block - n_front;
  const int64_t rows = (n_groups * rest - gap) / (kXcds * per_block), part = rows * per_block;
  if (i < kXcds * part) {
    const int64_t die = i / part, k = i - die * part;
    return (block0 + k / per_block * kXcds + die) * per_block + k % per_block;
  }
  // what is left fills the front's last block and follows the rows
  const int64_t left = i - kXcds * part;
  return left < gap ? n_front + left : (block0 + rows * kXcds) * per_block + (left - gap);
}

}  // namespace kf
