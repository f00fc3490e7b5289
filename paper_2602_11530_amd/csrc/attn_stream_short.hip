// Launches of the stream pass for short shares at D = 128 (short_at_128).
#include "attn_stream.h"

namespace pkv {

void launch_short_128(const AttnLaunch& a, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(128)), block(group_waves(128) * 64);
  hipLaunchKernelGGL((attn_stream_kernel<128, false, OneLayer, false>), grid, block, lds, stream, a, OneLayer{});
}

void launch_chained_short_128(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(128)), block(group_waves(128) * 64);
  hipLaunchKernelGGL((attn_stream_kernel<128, false, ChainedLayers, false>), grid, block, lds, stream, a, ChainedLayers{layers});
}

}  // namespace pkv
