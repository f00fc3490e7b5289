// Launches of the stream pass for short batches: a workgroup for each segment (WholeLayer), and short shares at D = 128 (short_at_128).
#include "attn_stream.h"

namespace pkv {

template <int kD>
static void launch_dim(const AttnLaunch& a, size_t lds, hipStream_t stream) {
  const dim3 grid(a.Hkv, 1, a.S), block(group_waves(kD) * 64);
  if (a.kv_fp8) hipLaunchKernelGGL((attn_stream_kernel<kD, true, WholeLayer, false>), grid, block, lds, stream, a, WholeLayer{});
  else hipLaunchKernelGGL((attn_stream_kernel<kD, false, WholeLayer, false>), grid, block, lds, stream, a, WholeLayer{});
}
void launch_whole(const AttnLaunch& a, size_t lds, hipStream_t stream) {
  if (a.D == 64) launch_dim<64>(a, lds, stream);
  else if (a.D == 128) launch_dim<128>(a, lds, stream);
  else launch_dim<256>(a, lds, stream);
}

void launch_short_128(const AttnLaunch& a, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(128)), block(group_waves(128) * 64);
  hipLaunchKernelGGL((attn_stream_kernel<128, false, OneLayer, false>), grid, block, lds, stream, a, OneLayer{});
}

void launch_chained_short_128(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(128)), block(group_waves(128) * 64);
  hipLaunchKernelGGL((attn_stream_kernel<128, false, ChainedLayers, false>), grid, block, lds, stream, a, ChainedLayers{layers});
}

}  // namespace pkv
