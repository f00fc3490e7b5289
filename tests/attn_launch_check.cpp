// Host-side check of what the attention calls launch: the C-ABI layer is linked against stand-ins
// for the two launch functions, which walk the launch as its workgroups would and note every
// piece of workspace that one of them writes.
//
//   - every write lies inside the bytes that the call asked for, in every layer of a launch
//   - no two writes of one launch overlap
//   - the reduce pass hears of a segment that workgroups share from each of them but the last, which
//     say how many they are and the how-manieth they are, and of nothing else
//   - what it reads of a segment are the records that were left of it, all of them
//   - the workgroups and the sets of lanes that it has for a segment take every record of every
//     chunk of its rows once
//
// And the stream pass's LDS: every part of it on a 16-byte boundary, large enough for what it holds and,
// all together, no more than a compute unit has.
//
// Compiled together with csrc/pkv_api.hip and run by tests/test_attn_launch.py (host code only, no GPU).
#include "../include/pkv.h"
#include "pkv_kernels.h"
#include <algorithm>
#include <cmath>
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
  if (!a.leaves_records && !whole) call.wrong++;   // nobody would finish the shared segments

  Writes writes;
  for (int y = 0; y < count; ++y) {
    if (a.leaves_records)
      for (int g = 0; g < grid; ++g) writes.add(shared_segment(a, y, g), sizeof(SharedSegment));
    if (whole) continue;
    std::map<int, SharedSegment> heard;   // of a segment that goes on behind the workgroup, as those that read of it need it
    for (int s = 0; s < a.S; ++s)
      for (int kvh = 0; kvh < a.Hkv && nblk[s] > 0; ++kvh) {
        const int first = a.Hkv * cum[s] + kvh * nblk[s], last = first + nblk[s] - 1;
        const int w0 = share_owner(first, T, W), w1 = share_owner(last, T, W);
        if (w0 == w1) continue;   // finished by its wavefront
        const int g0 = w0 / group, g1 = w1 / group;
        if (g0 == g1) continue;   // finished in its workgroup
        if (!a.leaves_records) call.wrong++;   // the reduce pass would not hear of it
        const float* record = group_record(a, a.D, y, g0, true);
        for (int g = g0; g <= g1; ++g) {
          writes.add(group_record(a, a.D, y, g, g == g0), record_bytes);
          const int j = g - g0;
          if (group_record(a, a.D, y, g, g == g0) != record + (2 * j - (j > 0)) * record_floats(a.G, a.D)) call.wrong++;
          if (g < g1 && !heard.insert({g, {(s * a.Hkv + kvh) * a.G, (g1 - g0 + 1) | j << 16}}).second) call.wrong++;   // one per workgroup
        }
      }
    const ShareMap shares(T, W);
    for (int g = 0; g < grid; ++g) {
      SharedSegment word = {0, 0};
      if ((g + 1) * group < W) {
        const int from = shares.start(g * group), next = shares.start((g + 1) * group);
        const int s = (int)(std::upper_bound(cum.begin(), cum.end(), (next - 1) / a.Hkv) - cum.begin()) - 1;   // not an empty one: the last that begins there
        const int kvh = (next - 1 - a.Hkv * cum[s]) / nblk[s], begin = a.Hkv * cum[s] + kvh * nblk[s];
        word = group == 8 ? word_of_group<8>(shares, g, from, next, (s * a.Hkv + kvh) * a.G, begin, nblk[s])
                          : word_of_group<4>(shares, g, from, next, (s * a.Hkv + kvh) * a.G, begin, nblk[s]);
      }
      const auto want = heard.find(g);
      if (want == heard.end() ? word.told != 0 : word.row != want->second.row || word.told != want->second.told) call.wrong++;
      if (word.told && word.slice() >= word.records() - 1) call.wrong++;
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
  if (!a.leaves_records) call.wrong++;
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

// What workgroups and sets of lanes take of a segment of `count` records whose rows are `chunks` chunks.
static void check_split() {
  using namespace pkv;
  for (int x = 0; x < 64; ++x)   // with the device's reciprocal, which may be a unit in the last place off
    for (int n = 1; n <= 64; ++n)
      for (float per : {std::nextafterf(1.f / n, 0.f), 1.f / n, std::nextafterf(1.f / n, 2.f)})
        if (((int)(((float)x + 0.5f) * per) != x / n || RecordSplit::quotient(x, n) != x / n) && failures++ < 20) printf("quotient of %d and %d\n", x, n);
  for (int chunks = 1; chunks <= kReduceSubs; ++chunks)
    for (int count = 2; count <= kLayerGroups; ++count) {
      const RecordSplit split(count, chunks);
      std::vector<int> taken(chunks * count, 0), finished(chunks, 0);
      for (int slice = 0; slice < count - 1; ++slice) {   // the workgroups that leave word
        if (slice * split.mine >= chunks) continue;
        for (int sub = 0; sub < kReduceSubs; ++sub) {
          const int set = sub / split.mine, chunk = slice * split.mine + sub % split.mine;
          if (set >= split.sets || chunk >= chunks) continue;
          for (int i = set; i < count; i += split.sets) taken[chunk * count + i]++;
          finished[chunk] += set == 0;
        }
      }
      const auto once = [](const std::vector<int>& v) { return std::all_of(v.begin(), v.end(), [](int n) { return n == 1; }); };
      if ((!once(taken) || !once(finished) || split.mine * split.sets > kReduceSubs) && failures++ < 20)
        printf("%d records of %d chunks: %d chunks a workgroup, %d sets\n", count, chunks, split.mine, split.sets);
    }
}

int main() {
  check_lds();
  check_split();
  uint64_t x = 41;
  auto rnd = [&](int n) { x = x * 6364136223846793005ULL + 1442695040888963407ULL; return (int)((uint32_t)(x >> 33) % (uint32_t)n); };
  const int heads[][2] = {{40, 8}, {8, 2}, {8, 1}, {16, 8}, {7, 7}, {16, 1}, {10, 5}, {8, 8}};
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
  // the shortest records
  for (int seqs : {31, 32, 33, 63, 64, 65})
    for (int blocks : {49, 63, 64, 65, 127, 128, 129, 500})
      for (int bound : {16 * blocks, 16 * blocks + 1, 20000})
        for (int into_q : {-1, 0, 128, 256}) {
          attend(std::vector<int>(seqs, 16 * blocks), 1, 1, 64, bound, 2, into_q);
          std::vector<int> uneven(seqs, 16);
          uneven[seqs / 2] = 16 * blocks;
          attend(uneven, 1, 1, 64, bound, 1, into_q);
        }
  printf("calls about %ld, failures=%ld\n", calls, failures);
  return failures != 0;
}
