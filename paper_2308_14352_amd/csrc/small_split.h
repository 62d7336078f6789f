// How many rows a workgroup of k_small_in / k_small_out (decode_small.hip) takes. Host arithmetic, no HIP.
#pragma once
#include <algorithm>
#include <cstdint>

namespace moeq {

// Rows of a workgroup (a multiple of four) for a matrix of `rows` x `cols` and so many items (a choice of a token, or a token):
// rounds of two workgroups per compute unit, each as long as six steps of the rows that the 512 threads cover at once and the steps
// it has. The blocks of rows are dealt to the eight XCDs in turn, every item's in the same way, so the rounds are those of the XCD
// with the most blocks, on its 64 places (rows of W_out of 8192 columns at 2 bits leave 32, which counts as 64 here), not those of the whole chip: 22 blocks of 23 tokens are 506 workgroups, but 69 on the
// first six XCDs. us, rounds of 512 / of 64: 1024 x 1024, 8 bits, 23 tokens 35.4 / 27.6, 512 x 2048, 22 tokens 30.0 / 23.3.
inline int small_rows_of_wg(int rows, int cols, int64_t items) {
  const int at_once = std::max(1, 512 * 32 / cols);
  int best = 4;
  double least = 1e30;
  for (int R = 4; R <= 256; R += 4) {
    const int64_t wgs = ((rows + R - 1) / R + 7) / 8 * items;      // of the XCD with the most
    const double cost = (double)((wgs + 63) / 64) * (6 + (R + at_once - 1) / at_once) + 1e-3 * (double)wgs;
    if (cost < least) { least = cost; best = R; }
  }
  return best;
}

}  // namespace moeq
