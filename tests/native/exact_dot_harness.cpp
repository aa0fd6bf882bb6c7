// Host build of the library's exact fallback (exact_dot.h) for the CPU tests, in the kernels'
// order: 64 lanes, lane l adding elements l, l + 64, ... to an accumulator of its own, the words
// summed over the lanes by a butterfly, one rounding.
#include <stdint.h>

#include <vector>

#include "exact_dot.h"

extern "C" float exact_dot_q22_host(const float* x, const int32_t* tq, int n) {
  using aatc::kAccWords;
  struct Acc { int64_t w[kAccWords] = {}; };
  std::vector<Acc> lane(64);
  for (int j = 0; j < n; ++j) aatc::acc_add(lane[j % 64].w, x[j], tq[j]);
  for (int o = 32; o >= 1; o >>= 1) {
    const std::vector<Acc> in = lane;
    for (int l = 0; l < 64; ++l)
      for (int k = 0; k < kAccWords; ++k) lane[l].w[k] = in[l].w[k] + in[l ^ o].w[k];
  }
  return aatc::acc_round(lane[17].w);              // (every lane ends with the sum)
}
