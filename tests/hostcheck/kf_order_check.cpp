// Host check of the length-sorted order, with a front and without: the waves'
// places are a permutation, the groups' first waves come first if there is a
// front, and a die's blocks hold consecutive waves.
#include <cstdio>
#include <vector>

#include "kf_order.hpp"

int main() {
  long bad = 0, apart = 0;
  for (int k = 0; k < 10; ++k)
    for (int64_t n_groups : {1, 2, 3, 7, 8, 9, 16, 31, 33, 100, 245}) {
      const int per_block = k / 2, front = k % 2;
      const int64_t n = n_groups * kf::kGroupWaves, n_front = front * n_groups;
      std::vector<int64_t> group(n, -1);
      for (int64_t g = 0; g < n_groups; ++g)
        for (int v = 0; v < kf::kGroupWaves; ++v) {
          const int64_t at = kf::wave_place(g, v, n_groups, per_block, front);
          if (at < 0 || at >= n || group[at] >= 0) {
            ++bad;
            continue;
          }
          group[at] = g;
          if ((v < front) != (at < n_front)) ++bad;
        }
      // from one block of a die to its next the group moves by at most one,
      // but for the few waves that fill up the ends
      if (per_block == 0 || n_groups < 100) continue;
      const int64_t row = int64_t(kf::kXcds) * per_block;
      for (int64_t at = n_front + per_block; at + 2 * row < n; ++at) {
        const int64_t d = group[at + row] - group[at];
        if (d < 0 || d > 1) ++apart;
      }
    }
  std::printf("misplaced %ld, apart %ld\n", bad, apart);
  return bad || apart;
}
