// How a transform of planes is laid out on the chip, by sizes alone; plain C++,
// so that the host can replay it.
#pragma once

#include <stdint.h>

namespace fno {

// Waves of a work-group of eight that share a plane in the kernels for any
// extents, as a power of two: one per block of 32 rows, up to all eight, and
// more while every plane still has its place in one pass over the chip.  (More
// than that starts a second pass that is nearly empty: 304 planes of 64 x 72 and
// 12 modes with the planes of one work-group each on 256 compute units, whole
// forward call 23.1 us in fp16 and 37.9 in fp32, so 19.0 and 30.9.)
constexpr int share_waves_log2(int64_t blocks, int64_t planes, int num_cu) {
  int lw = 0;
  while (lw < 3 && ((1 << lw) < blocks || (planes << (lw + 1)) <= (int64_t)8 * num_cu)) ++lw;
  return lw;
}

}  // namespace fno
