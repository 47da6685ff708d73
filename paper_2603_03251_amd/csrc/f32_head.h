// Whether the fp32 LM head of a pass takes the final norm along (plain C++: no HIP types).
#pragma once

#include <cstdint>

namespace ssd {

// The norm in the head saves a launch and a round trip of the rows (2 to 3 us).  Every feature, or pair of features, then squares and
// scales its groups of 8 rows again and adds one more set of sums up over its lanes: groups x vocabulary x (width + some 1000); and one
// group streaming a large head loses wavefronts in flight to the third set of accumulators.  Single extends of one layer, us, norm
// apart / in the head (width, vocabulary, rows): one group 1024, 1024, 8 33.0 / 30.8; 512, 8192, 8 38.9 / 37.3; 1024, 8192, 8 40.9 /
// 41.3; 2048, 8192, 8 55.5 / 57.6; 256, 32000, 8 41.6 / 42.2; 512, 32000, 8 52.6 / 56.0; 2048, 32000, 1 115 / 137; several 512, 8192,
// 16 40.6 / 38.7; 2048, 1024, 96 94.2 / 92.1; 1024, 8192, 24 56.5 / 55.4; 2048, 8192, 16 64.9 / 63.0; 256, 8192, 48 43.7 / 43.6; 512,
// 8192, 48 53.7 / 54.1; 256, 8192, 96 56.8 / 59.5; 1024, 8192, 48 76.0 / 77.1; 2048, 1024, 384 258 / 261; 256, 32000, 384 372 / 440;
// 2048, 32000, 384 2670 / 2742.  The lines lie where the two meet, at 2^24 for one group and 2^26 for several; on the wrong side
// of them 4096, 1024, 24 (71.7 / 74.9) and 2048, 32000, 16 (152 / 149).  A head of fewer than 16 features has no 8 units to write a
// group's hidden states.
inline bool f32_head_takes_norm(int rows, int vocab, int d_model) {
  const int64_t groups = (rows + 7) / 8;
  return vocab >= 16 && groups * vocab * (d_model + 1024) <= (groups == 1 ? 1 << 24 : 1 << 26);
}

}  // namespace ssd
