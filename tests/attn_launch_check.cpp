// Host-side check of what the attention calls launch: the C-ABI layer is linked against stand-ins
// for the two launch functions, which walk the launch as its workgroups would and note every
// piece of workspace that one of them writes.
//
//   - every write lies inside the bytes that the call asked for, in every layer of a launch
//   - no two writes of one launch overlap
//   - what the reduce pass reads of a segment are the records that were left of it, all of them
//
// And the stream pass's LDS: every part of it on a 16-byte boundary, large enough for what it holds and,
// all together, no more than a compute unit has.
//
// Compiled together with csrc/pkv_api.hip and run by tests/test_attn_launch.py (host code only, no GPU).
#include "../include/pkv.h"
#include "pkv_kernels.h"
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <utility>
#include <vector>

namespace {

char* const kWorkspace = reinterpret_cast<char*>((uintptr_t)1 << 40);   // an address only

struct Call {   // the call under way
  std::vector<int> lens;
  int64_t need = 0;
  std::vector<int> layers_of_launch;
  std::vector<std::pair<int64_t, int64_t>> written;   // by the latest launch
  long copies = 0;
  long past_end = 0, overlaps = 0, wrong = 0;
};
Call call;

struct Writes {
  std::vector<std::pair<int64_t, int64_t>> spans;   // byte ranges, relative to the workspace
  void add(const void* p, int64_t bytes) {
    const int64_t at = static_cast<const char*>(p) - kWorkspace;
    if (at < 0 || at + bytes > call.need) call.past_end++;
    spans.push_back({at, at + bytes});
  }
  void done() {
    std::sort(spans.begin(), spans.end());
    for (size_t i = 1; i < spans.size(); ++i)
      if (spans[i].first < spans[i - 1].second) call.overlaps++;
  }
};

// One launch of the stream pass over call.lens, layer by layer and segment by segment.
void walk(const pkv::AttnLaunch& a, const pkv::AttnLayers* layers) {
  using namespace pkv;
  const int group = group_waves(a.D), grid = a.waves / group, count = layers ? layers->count : 1;
  const int64_t record_bytes = (int64_t)record_floats(a.G, a.D) * sizeof(float);
  call.layers_of_launch.push_back(count);
  if (a.waves % group != 0 || grid > kLayerGroups) call.wrong++;

  std::vector<int> nblk(a.S), cum(a.S + 1, 0);
  bool any_long = false;
  for (int s = 0; s < a.S; ++s) {
    nblk[s] = (std::min(std::max(call.lens[s], 0), a.max_ctx) + kBlockTokens - 1) / kBlockTokens;
    cum[s + 1] = cum[s] + nblk[s];
    any_long = any_long || nblk[s] > a.short_blocks;
  }
  const int T = a.Hkv * cum[a.S], W = share_count(T, a.waves);
  const bool whole = !any_long && a.S * a.Hkv <= grid;
  if (a.leaves == kNoRecords && !whole) call.wrong++;   // nobody would finish the shared segments
  const bool by_row = !whole && (a.leaves == kRows || (a.leaves == kFewSegments && T <= row_blocks(a.waves)));

  Writes writes;
  if (by_row || a.leaves == kRows) writes.add(a.ws_cum, (a.S + 1) * (int64_t)sizeof(int32_t));
  for (int y = 0; y < count; ++y) {
    if (a.leaves == kManySegments || a.leaves == kFewSegments)
      for (int g = 0; g < grid; ++g) writes.add(shared_segment(a, y, g), sizeof(SharedSegment));
    if (whole) continue;
    std::map<int, int> begins;   // workgroup -> segments that begin in it and go on in another one
    for (int s = 0; s < a.S; ++s)
      for (int kvh = 0; kvh < a.Hkv && nblk[s] > 0; ++kvh) {
        const int first = a.Hkv * cum[s] + kvh * nblk[s], last = first + nblk[s] - 1;
        const int w0 = share_owner(first, T, W), w1 = share_owner(last, T, W);
        if (w0 == w1) continue;   // finished by its wavefront
        if (by_row) {
          for (int w = w0; w <= w1; ++w) writes.add(wave_record(a, a.D, s * a.Hkv + kvh, w), record_bytes);
          continue;
        }
        const int g0 = w0 / group, g1 = w1 / group;
        if (g0 == g1) continue;   // finished in its workgroup
        if ((a.leaves != kManySegments && a.leaves != kFewSegments) || ++begins[g0] > 1) call.wrong++;   // the reduce pass hears of one per workgroup
        for (int g = g0; g <= g1; ++g) writes.add(group_record(a, a.D, y, g, g == g0), record_bytes);
      }
  }
  writes.done();
  call.written = writes.spans;
}

}  // namespace

namespace pkv {
hipError_t launch_attn_stream(const AttnLaunch& a, const AttnLayers* layers, hipStream_t) {
  walk(a, layers);
  return hipSuccess;
}
hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers*, hipStream_t) {
  if (a.leaves == kNoRecords) call.wrong++;
  return hipSuccess;
}
// Rows kept in the workspace until all inputs are read.
hipError_t launch_copy(const void* src, void*, int64_t bytes, hipStream_t) {
  const int64_t at = static_cast<const char*>(src) - kWorkspace;
  if (at < 0 || at % 16 != 0 || at + bytes > call.need) call.past_end++;
  for (auto& w : call.written)
    if (w.first < at + bytes && at < w.second) call.overlaps++;
  call.copies++;
  return hipSuccess;
}
hipError_t launch_kv_block_copy(const void*, void*, const int32_t*, int64_t, int64_t, int64_t, bool, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_block_move(const void*, const int32_t*, int64_t, void*, const int32_t*, int64_t, int64_t, int64_t, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_append(const uint16_t*, const uint16_t*, uint16_t*, uint16_t*, const int32_t*, const int32_t*, int, int, int, int, int, int, int, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_kv_append_fp8(const uint16_t*, const uint16_t*, void*, void*, const int32_t*, const int32_t*, float, float, int, int, int, int, int, int, int, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_read_probe(const void*, const void*, uint32_t, int64_t, void*, hipStream_t) { return hipSuccess; }
}  // namespace pkv

static long failures = 0;

// into_q: the output begins that many bytes behind q.
static void attend(const std::vector<int>& lens, int hq, int hkv, int dim, int bound, int layers, int into_q = -1) {
  call = Call();
  call.lens = lens;
  const int longest = std::max(bound, *std::max_element(lens.begin(), lens.end()));
  pkv_attn_shape sh = {};
  sh.num_seqs = (int)lens.size();
  sh.num_q_heads = hq;
  sh.num_kv_heads = hkv;
  sh.head_dim = dim;
  sh.block_size = 16;
  sh.max_blocks_per_seq = (longest + 15) / 16 + 1;
  sh.max_context_len = bound;
  sh.num_pool_blocks = 1000;
  size_t need = 0;
  int rc = pkv_attn_workspace_bytes(&sh, &need);
  call.need = (int64_t)need;
  // layers far apart from each other and from the workspace
  std::vector<const void*> in[3];
  std::vector<void*> out;
  for (int l = 0; l < layers; ++l) {
    for (int i = 0; i < 3; ++i) in[i].push_back(reinterpret_cast<void*>(((uintptr_t)2 << 40) + ((uintptr_t)(4 * l + i) << 36)));
    out.push_back(reinterpret_cast<void*>(((uintptr_t)2 << 40) + (into_q < 0 ? (uintptr_t)(4 * l + 3) << 36 : ((uintptr_t)(4 * l) << 36) + into_q)));
  }
  const int32_t* p4 = reinterpret_cast<const int32_t*>((uintptr_t)1 << 39);
  if (rc == PKV_OK)
    rc = paged_decode_attn_layers(in[0].data(), in[1].data(), in[2].data(), p4, p4, 1.f, out.data(), layers, &sh, kWorkspace, need, nullptr);
  int launched = 0;
  for (int n : call.layers_of_launch) launched += n;
  if (call.copies != (into_q > 0 ? layers : 0)) call.wrong++;   // q itself may be the output
  if (rc != PKV_OK || launched != layers || call.past_end || call.overlaps || call.wrong) {
    if (failures++ < 20)
      printf("S=%zu heads %d/%d D=%d bound %d, %d layers (%d launched in %zu): status %d, %ld writes past the workspace's %zu bytes, %ld overlaps, %ld wrong\n",
             lens.size(), hq, hkv, dim, bound, layers, launched, call.layers_of_launch.size(), rc, call.past_end, need, call.overlaps, call.wrong);
  }
}

static void check_lds() {
  using namespace pkv;
  for (int D : {64, 128, 256})
    for (int G = 1; G <= (D == 256 ? 8 : 16); ++G)
      for (int S = 1; S <= kMaxSeqs; ++S) {
        const StreamLds l = stream_lds(S, G, D);
        const int rec = record_floats(G, D), rows = G * D / 2;   // bf16 rows, in floats
        const bool ok = l.prefix >= 2 * S + 1 && l.prefix % 4 == 0 && l.wave % 4 == 0 && rec % 4 == 0 && rows % 4 == 0 &&
                        l.wave >= 2 * rec && l.staged_max >= 1 && l.wave >= rec + l.staged_max * rows &&
                        l.bytes >= 4 * (l.prefix + group_waves(D) * l.wave) && l.bytes <= 159 * 1024;   // and the static arrays
        if (!ok && failures++ < 20)
          printf("LDS at S=%d G=%d D=%d: prefix %d, wavefront %d, staged %d, %d bytes\n", S, G, D, l.prefix, l.wave, l.staged_max, l.bytes);
      }
}

int main() {
  check_lds();
  uint64_t x = 41;
  auto rnd = [&](int n) { x = x * 6364136223846793005ULL + 1442695040888963407ULL; return (int)((uint32_t)(x >> 33) % (uint32_t)n); };
  const int heads[][2] = {{40, 8}, {8, 2}, {8, 1}, {16, 8}, {7, 7}, {16, 1}, {10, 5}};
  long calls = 0;
  for (int dim : {64, 128, 256})
    for (auto& h : heads)
      for (int limit : {16, 17, 384, 385, 768, 769, 3000, 40000})
        for (int trial = 0; trial < 6; ++trial) {
          if (dim == 256 && h[0] / h[1] > 8) continue;
          const int most = limit > 1000 ? 40 : 300;
          std::vector<int> lens(1 + rnd(trial < 3 ? most : 12));
          for (int& n : lens) n = rnd(8) == 0 ? 0 : 1 + rnd(limit);
          lens[rnd((int)lens.size())] = limit;
          for (int layers : {1, 2, 4, 5, 8, 9, 17}) {
            attend(lens, h[0], h[1], dim, limit, layers);        // the bound says how long they are
            if (layers < 9) attend(lens, h[0], h[1], dim, 50000, layers);   // and does not
            if (layers == 2) attend(lens, h[0], h[1], dim, trial % 2 ? limit : 50000, layers, 128 * (trial % 3));
            calls += 2;
          }
        }
  // as many segments as workgroups, and one more or less than the limits of the two layouts
  for (int seqs : {63, 64, 65, 255, 256, 257, 2048}) {
    attend(std::vector<int>(seqs, 300), 5, 1, 128, 300, 9);
    attend(std::vector<int>(seqs, 300), 5, 1, 256, 300, 9);
    attend(std::vector<int>(seqs, 1600), 16, 1, 64, 0, 3);
  }
  printf("calls about %ld, failures=%ld\n", calls, failures);
  return failures != 0;
}
