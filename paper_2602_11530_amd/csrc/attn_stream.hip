// Launch of the stream pass; the kernel is in attn_stream.h.
#include "attn_stream.h"

namespace pkv {

template <int kD>
static void launch_dim(const AttnLaunch& a, const AttnLayers* layers, size_t lds, hipStream_t stream) {
  constexpr bool kLate = kD == 128;
  const dim3 grid = stream_grid(a, layers), block(group_waves(kD) * 64);
  if (layers) hipLaunchKernelGGL((attn_stream_kernel<kD, false, AttnLayers, kLate>), grid, block, lds, stream, a, *layers);
  else if (a.kv_fp8) hipLaunchKernelGGL((attn_stream_kernel<kD, true, OneLayer, false>), grid, block, lds, stream, a, OneLayer{});
  else hipLaunchKernelGGL((attn_stream_kernel<kD, false, OneLayer, kLate>), grid, block, lds, stream, a, OneLayer{});
}

hipError_t launch_attn_stream(const AttnLaunch& a_in, const AttnLayers* layers, hipStream_t stream) {
  AttnLaunch a = a_in;
  const StreamLds l = stream_lds(a.S, a.G, a.D, a.kv_fp8);
  a.staged_max = l.staged_max;
  a.wave_lds_floats = l.wave;
  a.turns = l.turn_bytes > 0;
  const size_t lds = l.bytes + l.turn_bytes;
  if (layers && a.kv_fp8) return hipErrorInvalidValue;
  if (a.D == 64) launch_dim<64>(a, layers, lds, stream);
  else if (a.D == 128) launch_dim<128>(a, layers, lds, stream);
  else if (a.D != 256) return hipErrorInvalidValue;
  else if (late_at_256(a)) launch_late_256(a, layers, lds, stream);
  else launch_dim<256>(a, layers, lds, stream);
  return hipGetLastError();
}

}  // namespace pkv
