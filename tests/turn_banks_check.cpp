// Host-side check of where a block of K lies in LDS while it is turned: a place of its own for every piece, inside the block's
// room, and no two lanes of a step of the LDS unit in one bank.  Steps and banks of 16-byte accesses as measured on gfx950
// with pairs of lanes.  Compiled and run by tests/test_turn_banks.py (host code only, no GPU).
#include "pkv_kernels.h"
#include <cstdio>
#include <set>

// which of the four steps of a read, or of the eight of a write, a lane is in
static int read_step(int lane) {
  const int in = lane & 31;
  return lane / 32 * 2 + !(in < 4 || (in >= 12 && in < 16) || (in >= 20 && in < 28));
}
static int write_step(int lane) { return lane / 8; }

int main() {
  using namespace pkv;
  long bad = 0, reads = 0, writes = 0;
  for (int pieces : {8, 16, 32}) {
    std::set<int> places;
    for (int t = 0; t < kBlockTokens; ++t)
      for (int p = 0; p < pieces; ++p) places.insert(turn_place(pieces, t, p));
    bad += (int)places.size() != kBlockTokens * pieces || *places.begin() != 0 || *places.rbegin() != kBlockTokens * pieces - 1;
    for (int jj = 0; jj < pieces / 4; ++jj) {
      std::set<int> read_banks[4], write_banks[8];   // in 16 bytes: 16 of them over 64 banks, 8 over 32
      for (int lane = 0; lane < 64; ++lane) {
        const int n = lane & 15, c = lane >> 4, at = 64 * jj + lane;
        reads += !read_banks[read_step(lane)].insert(turn_place(pieces, turn_token(n), 4 * jj + c) % 16).second;
        writes += !write_banks[write_step(lane)].insert(turn_place(pieces, at / pieces, at % pieces) % 8).second;
      }
    }
  }
  printf("conflicts %ld reading, %ld writing, bad=%ld\n", reads, writes, bad);
  return reads || writes || bad;
}
