// Instantiations of the fp32 contraction on the bf16 matrix cores: tile configuration 2, windows of 4 taps (2x2).
#include "conv_split.h"

namespace syno {

void launch_split_2_4(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s) {
  launch_split_tiles<2, 1, 4, 2, 4, 2, 7>(tiles, p, X, W, out, s);
}

}  // namespace syno
