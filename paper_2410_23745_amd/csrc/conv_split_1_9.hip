// Instantiations of the fp32 contraction on the bf16 matrix cores: tile configuration 1, windows of 9 taps.
#include "conv_split.h"

namespace syno {

void launch_split_1_9(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s) {
  launch_split_tiles<4, 1, 2, 2, 9, 1, 7>(tiles, p, X, W, out, s);
}

}  // namespace syno
