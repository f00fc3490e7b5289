// Launch of the stream pass; the kernel is in attn_stream.h.
#include "attn_stream.h"

namespace pkv {

template <int kD>
static void launch_dim(const AttnLaunch& a, const AttnLayers* layers, size_t lds, hipStream_t stream) {
  constexpr bool kLarge = kD == 128;
  const dim3 grid(a.waves / group_waves(kD), layers ? layers->count : 1), block(group_waves(kD) * 64);
  if (layers) hipLaunchKernelGGL((attn_stream_kernel<kD, false, AttnLayers, kLarge>), grid, block, lds, stream, a, *layers);
  else if (a.kv_fp8) hipLaunchKernelGGL((attn_stream_kernel<kD, true, OneLayer, false>), grid, block, lds, stream, a, OneLayer{});
  else hipLaunchKernelGGL((attn_stream_kernel<kD, false, OneLayer, kLarge>), grid, block, lds, stream, a, OneLayer{});
}

hipError_t launch_attn_stream(const AttnLaunch& a_in, const AttnLayers* layers, hipStream_t stream) {
  AttnLaunch a = a_in;
  const StreamLds l = stream_lds(a.S, a.G, a.D, a.kv_fp8);
  a.staged_max = l.staged_max;
  a.wave_lds_floats = l.wave;
  a.turns = l.turn_bytes > 0;
  const size_t lds = l.bytes + l.turn_bytes;
  if (layers && a.kv_fp8) return hipErrorInvalidValue;
  // Layers go one after the other in each workgroup, or, where each segment has a workgroup, each in workgroups of its own.
  // Those are short, and the scalar registers that the chain keeps (then 76 to 83 spills instead of 4 to 24, now 60 to 66 instead of 0 to 10) cost them 0.8 to 2 us:
  // attention of 4 layers of 4 requests of 51..69 tokens on 8/2 heads at D = 64 8.1 us in the chain's kernel, 7.15 without, 2 layers
  // of 80 of 85..114 15.3 and 13.3.
  if (layers && a.leaves_records) return launch_chained(a, *layers, lds, stream);
  if (!layers && !a.leaves_records) launch_whole(a, lds, stream);
  else if (!layers && short_at_128(a)) launch_short_128(a, lds, stream);
  else if (a.D == 64) launch_dim<64>(a, layers, lds, stream);
  else if (a.D == 128) launch_dim<128>(a, layers, lds, stream);
  else if (a.D != 256) return hipErrorInvalidValue;
  else if (!layers && large_at_256(a)) launch_large_256(a, lds, stream);   // layers come here with short segments only
  else launch_dim<256>(a, layers, lds, stream);
  return hipGetLastError();
}

}  // namespace pkv
