// The host's choice of a way through the attention calls, from the C-ABI layer itself: linked against stand-ins for the launches,
// it reads "seqs query_heads kv_heads head_dim max_tokens fp8" lines and prints whether there is a reduce pass and how many
// wavefronts are launched.  Run by tests/test_routes.py (host code only, no GPU).
#include "../include/pkv.h"
#include "pkv_kernels.h"
#include <cstdio>

static int leaves_records, reduced, waves;

namespace pkv {
hipError_t launch_attn_stream(const AttnLaunch& a, const AttnLayers*, hipStream_t) {
  leaves_records = a.leaves_records;
  reduced = 0;
  waves = a.waves;
  return hipSuccess;
}
hipError_t launch_attn_reduce(const AttnLaunch&, const AttnLayers*, hipStream_t) {
  reduced = 1;
  return hipSuccess;
}
hipError_t launch_copy(const void*, void*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_block_copy(const void*, void*, const int32_t*, int64_t, int64_t, int64_t, bool, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_block_move(const void*, const int32_t*, int64_t, void*, const int32_t*, int64_t, int64_t, int64_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_append(const uint16_t*, const uint16_t*, uint16_t*, uint16_t*, const int32_t*, const int32_t*, int, int, int, int, int, int, int, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_append_fp8(const uint16_t*, const uint16_t*, void*, void*, const int32_t*, const int32_t*, float, float, int, int, int, int, int, int, int, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_read_probe(const void*, const void*, uint32_t, int64_t, void*, hipStream_t) { return hipSuccess; }
}  // namespace pkv

int main() {
  char* const base = reinterpret_cast<char*>((uintptr_t)1 << 40);   // addresses only
  const int32_t* ints = reinterpret_cast<const int32_t*>((uintptr_t)1 << 39);
  int seqs, hq, hkv, dim, tokens, fp8;
  while (scanf("%d %d %d %d %d %d", &seqs, &hq, &hkv, &dim, &tokens, &fp8) == 6) {
    pkv_attn_shape sh = {seqs, hq, hkv, dim, 16, (tokens + 15) / 16 + 3, 0, tokens, 1000};
    size_t need = 0;
    int rc = pkv_attn_workspace_bytes(&sh, &need);
    char* p[4];
    for (int i = 0; i < 4; ++i) p[i] = base + ((uintptr_t)(i + 1) << 36);
    if (rc == PKV_OK)
      rc = fp8 ? paged_decode_attn_fp8kv(p[0], p[1], p[2], ints, ints, 1.f, 1.f, 1.f, p[3], &sh, base, need, nullptr)
               : paged_decode_attn(p[0], p[1], p[2], ints, ints, 1.f, p[3], &sh, base, need, nullptr);
    if (rc != PKV_OK) return printf("status %d\n", rc), 1;
    if (reduced != leaves_records) return printf("a reduce pass: %d\n", reduced), 1;
    printf("%d %d\n", leaves_records, waves);
  }
  return 0;
}
