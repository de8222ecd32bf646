// Host check of the alignment reduction's loads: whatever part of the hit
// arrays a batch takes up, every index a lane loads lies within the arrays,
// and the batch's entries are each loaded by their own place.
#include <cstdio>

#include "kf_adjoint.hpp"

int main() {
  const int64_t per = kf::kAlignPerBlock;
  long bad = 0, covered = 0, expected = 0;
  for (int64_t n_hits : {int64_t(1), int64_t(63), per, per + 1}) {
    for (int64_t first : {int64_t(0), n_hits / 2, n_hits - 1, n_hits}) {
      for (int64_t last : {first, (first + n_hits) / 2, n_hits}) {
        expected += last - first;
        for (int64_t b = 0; b < kf::adjoint_partial_blocks(n_hits); ++b)
          for (int64_t k = 0; k < per; ++k) {
            const int64_t e = first + b * per + k, at = kf::align_load_entry(e, last);
            if (at < 0 || at >= n_hits) ++bad;
            if (e < last && at == e) ++covered;
          }
      }
    }
  }
  std::printf("out of range %ld, covered %ld of %ld\n", bad, covered, expected);
  return bad || covered != expected;
}
