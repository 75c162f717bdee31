// Instantiations of the bf16 convolution in chunks: tile configuration 0.
#include "conv_flow_bf16.h"

namespace syno {

SYNO_FLOW_LAUNCHER(0) {
  constexpr int N = kFlowConfigs[0].max_tiles;
  // (2x2 windows: backward-data only, the gradients of strided convolutions)
  if (taps == 4) launch_flow_tiles<4, 2, 0, true, N>(tiles, x_items, p, X, W, out, s);
  else if (adjoint) launch_flow_tiles<9, 3, 0, true, N>(tiles, x_items, p, X, W, out, s);
  else launch_flow_tiles<9, 3, 0, false, N>(tiles, x_items, p, X, W, out, s);
}

}  // namespace syno
