// Launches of the stream pass for large batches: D = 256 (large_at_256), and several layers.
#include "attn_stream.h"

namespace pkv {

void launch_large_256(const AttnLaunch& a, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(256)), block(group_waves(256) * 64);
  if (a.kv_fp8) hipLaunchKernelGGL((attn_stream_kernel<256, true, OneLayer, true>), grid, block, lds, stream, a, OneLayer{});
  else hipLaunchKernelGGL((attn_stream_kernel<256, false, OneLayer, true>), grid, block, lds, stream, a, OneLayer{});
}

template <int kD, bool kLarge>
static void launch_layers(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(kD)), block(group_waves(kD) * 64);
  hipLaunchKernelGGL((attn_stream_kernel<kD, false, ChainedLayers, kLarge>), grid, block, lds, stream, a, ChainedLayers{layers});
}

hipError_t launch_chained(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream) {
  if (a.D == 64) launch_layers<64, false>(a, layers, lds, stream);
  else if (short_at_128(a)) launch_chained_short_128(a, layers, lds, stream);
  else if (a.D == 128) launch_layers<128, true>(a, layers, lds, stream);
  else if (a.D != 256) return hipErrorInvalidValue;
  else if (large_at_256(a)) launch_layers<256, true>(a, layers, lds, stream);
  else launch_layers<256, false>(a, layers, lds, stream);
  return hipGetLastError();
}

}  // namespace pkv
