// Launch of the stream pass for large batches in bf16 at D = 256 (late_at_256).
#include "attn_stream.h"

namespace pkv {

void launch_late_256(const AttnLaunch& a, const AttnLayers* layers, size_t lds, hipStream_t stream) {
  const dim3 grid = stream_grid(a, layers), block(group_waves(256) * 64);
  if (layers) hipLaunchKernelGGL((attn_stream_kernel<256, false, AttnLayers, true>), grid, block, lds, stream, a, *layers);
  else hipLaunchKernelGGL((attn_stream_kernel<256, false, OneLayer, true>), grid, block, lds, stream, a, OneLayer{});
}

}  // namespace pkv
