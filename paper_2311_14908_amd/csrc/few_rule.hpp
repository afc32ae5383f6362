// few_rule.hpp -- when a prediction of a few test samples takes one pass over the training rows
// (predict_few_k) instead of tiles of 128 test samples (host arithmetic only).
#pragma once

#include <stdint.h>

namespace svmx {

constexpr int FEW_MAX = 16;             // test samples at most
constexpr int PREDICT_PAIRS_MAX = 64;   // problems per prediction launch (bounds the partial sums)

// The pass costs fp64 sums over every problem's support vectors, for each sample (taken in fours): with
// the chip full about 0.4 us a million of rows x features x samples.  Tiles cost 0.8 us a million of
// rows x features whatever m, plus 1.7 us a million features to split the n rows once, however many
// problems share them, plus about 18 us of launches for each 64 problems.  How many samples are support
// vectors is not known here; the line lies where the two are equal if all of them are.  Us a call (pass,
// tiles), all samples support vectors: 10 classes of 1,000 x 784, 1 sample 90, 124; 4: 165, 125; 16: 511,
// 126; 10 classes of 300 x 784, 4 samples 87, 90; 5: 125, 90; 5 classes of 2,000 x 300, 4 samples 89, 85;
// 16: 148, 85; 20 classes of 3,000 x 784, 4 samples 1,543, 827; 64 classes of 500 x 784, 16 samples
// 10,060, 1,668.  With few support vectors the pass can still be ahead beyond the line (4% of 10 classes
// of 1,000 x 784, 4 samples 71, 101).
// One problem always takes the pass: its tiles run on at most 64 workgroups, the pass on 64 for each
// four samples (300,000 x 784, 16 samples 1,362, 1,673; 1,000,000 x 128, 1 sample 310, 1,239; at worst
// 36, 28: 16 samples against 20,000 x 16, 5% of them support vectors).
// problems, rows: their number and the sum of their training samples.
inline bool predict_few_pays(int64_t problems, int64_t rows, int64_t n, int64_t d, int64_t m) {
  if (m > FEW_MAX) return false;
  if (problems == 1) return true;
  const double sums = m == 1 ? 1.0 : (double)((m + 3) / 4 * 4);
  const double launches = (double)((problems + PREDICT_PAIRS_MAX - 1) / PREDICT_PAIRS_MAX);
  return (double)rows * (double)d * (sums - 2.0) <= 4.2 * (double)n * (double)d + 45e6 * launches;
}

}  // namespace svmx
