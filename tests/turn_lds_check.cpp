// Host-side check of the room in LDS that the stream pass turns K in: behind everything else, aligned, inside a
// compute unit's LDS together with the static arrays, and missing only where there is no room (at D = 128, where the kernel has a
// way without it, and never up to 13 query heads per KV head in bf16 and 15 in e4m3) and in e4m3 at D = 64, which needs none.  Compiled and run by tests/test_turn_lds.py (host code only, no GPU).
#include "pkv_kernels.h"
#include <cstdio>

int main() {
  using namespace pkv;
  long bad = 0, without = 0;
  for (int D : {64, 128, 256})
    for (int fp8 = 0; fp8 < 2; ++fp8)
      for (int G = 1; G <= (D == 256 ? 8 : 16); ++G)
        for (int S = 1; S <= kMaxSeqs; ++S) {
          const StreamLds l = stream_lds(S, G, D, fp8);
          const int want = group_waves(D) * kBlockTokens * D * (fp8 ? 1 : 2);
          const bool none = l.turn_bytes == 0;
          without += none;
          const bool no_need = D == 64 && fp8, no_room = l.bytes + want > 159 * 1024;
          if (none != (no_need || no_room) || (!none && l.turn_bytes != want)) bad++;
          if (no_room && !no_need && (D != 128 || G <= (fp8 ? 15 : 13))) bad++;
          if (l.bytes % 16 != 0 || l.bytes < 4 * (l.prefix + group_waves(D) * l.wave)) bad++;
          if (l.bytes + l.turn_bytes > 159 * 1024) bad++;
        }
  printf("without %ld bad=%ld\n", without, bad);
  return bad != 0;
}
