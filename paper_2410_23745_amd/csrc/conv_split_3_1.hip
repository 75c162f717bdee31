// Instantiations of the fp32 contraction on the bf16 matrix cores: tile configuration 3, windows of 1 tap.
#include "conv_split.h"

namespace syno {

void launch_split_3_1(int tiles, const SplitParams& p, const float* X, const float* W, float* out, hipStream_t s) {
  launch_split_tiles<4, 2, 1, 4, 1, 2, 4>(tiles, p, X, W, out, s);
}

}  // namespace syno
