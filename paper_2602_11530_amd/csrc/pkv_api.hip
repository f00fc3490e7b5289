// C-ABI layer of libpkv: argument validation (all of it before any launch, so
// it can be exercised without a GPU), launch geometry, status codes.
#include "../../include/pkv.h"

#include "pkv_kernels.h"

#include <atomic>

// Workspace of paged_decode_attn_static: device memory that exists from the
// moment the library is loaded on a GPU until the process ends, so that entry
// point never allocates.  In host code this name is only a handle for
// hipGetSymbolAddress; the address kernels are given is looked up per device.
constexpr size_t kStaticScratchBytes = PKV_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local hipError_t g_last_launch_error = hipSuccess;
thread_local int32_t* g_id_faults = nullptr;   // see pkv_set_id_fault_counter

inline bool misaligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Library's partition choice when the caller leaves it open.  With the stream
// decomposition a partition only bounds how many tokens one partial result may
// stand for before it is folded into its segment's record, so the largest value
// is the cheapest.
constexpr int kDefaultPartition = pkv::kMaxPartition;

// Query heads.  Keeps every size product far inside 64 bits.
constexpr int kMaxHeads = 16384;

struct Geometry {
  int G, P, max_ctx;
  int64_t slots;   // records that the workspace has room for
};

// A record for every (wavefront, request, KV head) that meet, at most, as wavefronts' own records would need.  Workgroups leave far
// fewer; the rest takes those of further layers of a launch, or rows (launch_layer).
int64_t record_slots(int S, int Hkv) { return (int64_t)Hkv * S + pkv::kStreamWaves; }

int check_shape(const pkv_attn_shape* sh, Geometry* g) {
  if (!sh) return PKV_ERR_NULL;
  if (sh->num_seqs < 0 || sh->num_seqs > pkv::kMaxSeqs) return PKV_ERR_SHAPE;
  if (sh->num_q_heads <= 0 || sh->num_kv_heads <= 0 || sh->num_q_heads > kMaxHeads)
    return PKV_ERR_SHAPE;
  const int D = sh->head_dim;
  if (D != 64 && D != 128 && D != 256) return PKV_ERR_SHAPE;
  const int B = sh->block_size;
  if (B != 16 && B != 32 && B != pkv::kMaxBlockSize) return PKV_ERR_SHAPE;
  if (sh->num_q_heads % sh->num_kv_heads != 0) return PKV_ERR_SHAPE;
  const int G = sh->num_q_heads / sh->num_kv_heads;
  if (G > pkv::kMaxGroup) return PKV_ERR_SHAPE;
  // a wavefront keeps two whole records (G rows of D floats) in its share of LDS
  if (D == 256 && G > 8) return PKV_ERR_SHAPE;
  if (sh->max_blocks_per_seq <= 0) return PKV_ERR_SHAPE;
  if ((int64_t)sh->max_blocks_per_seq * B > INT32_MAX) return PKV_ERR_SHAPE;
  const int cap = sh->max_blocks_per_seq * B;
  if (sh->max_context_len < 0 || sh->max_context_len > cap) return PKV_ERR_SHAPE;
  const int max_ctx = sh->max_context_len ? sh->max_context_len : cap;
  int P = sh->partition_size;
  if (P < 0) return PKV_ERR_SHAPE;
  if (P == 0) P = kDefaultPartition;
  if (P % B != 0 || P < B || P > pkv::kMaxPartition) return PKV_ERR_SHAPE;
  // 4 KiB slabs (16 tokens of one KV head) are numbered in 32 bits on the device
  if (sh->num_pool_blocks < 1 ||
      sh->num_pool_blocks > INT32_MAX / ((int64_t)sh->num_kv_heads * (B / pkv::kBlockTokens)))
    return PKV_ERR_SHAPE;
  // stream positions, slots and rows are 32-bit on the device
  const int64_t max_blocks = (max_ctx + pkv::kBlockTokens - 1) / pkv::kBlockTokens;
  if ((int64_t)sh->num_kv_heads * sh->num_seqs * max_blocks > INT32_MAX) return PKV_ERR_SHAPE;
  if ((int64_t)sh->num_seqs * sh->num_q_heads > INT32_MAX) return PKV_ERR_SHAPE;
  g->G = G;
  g->P = P;
  g->max_ctx = max_ctx;
  g->slots = record_slots(sh->num_seqs, sh->num_kv_heads);
  return PKV_OK;
}

// Workspace: the partial records, then room for a prefix array, which nothing uses but which is part of the size that callers know.
size_t workspace_bytes(const pkv_attn_shape* sh, const Geometry& g) {
  if (sh->num_seqs == 0) return 0;
  const size_t records = (size_t)g.slots * pkv::record_floats(g.G, sh->head_dim) * sizeof(float);
  return records + (((size_t)(sh->num_seqs + 1) * sizeof(int32_t) + 15) & ~(size_t)15);
}

int launch_status(hipError_t e) {
  if (e == hipSuccess) return PKV_OK;
  g_last_launch_error = e;
  return PKV_ERR_LAUNCH;
}

// Every GPU holds its own copy of `scratch` at its own address; the address is
// looked up once per device, with that device current, and kept.
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

int static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return launch_status(e);
  if (dev < 0 || dev >= kMaxDevices) return launch_status(hipErrorInvalidDevice);
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return launch_status(e);
    if (!p) return launch_status(hipErrorInvalidSymbol);
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return PKV_OK;
}

}  // namespace

extern "C" {

int pkv_version(void) { return 1003; }

const char* pkv_status_string(int status) {
  switch (status) {
    case PKV_OK: return "ok";
    case PKV_ERR_NULL: return "a required pointer is NULL";
    case PKV_ERR_SHAPE: return "unsupported or inconsistent sizes";
    case PKV_ERR_ALIGN: return "a pointer or byte count is not 16-byte aligned";
    case PKV_ERR_WORKSPACE: return "workspace missing or too small";
    case PKV_ERR_LAUNCH: return "HIP refused the launch";
    case PKV_ERR_HOST: return "the host buffer is not pinned host memory";
    default: return "unknown status";
  }
}

const char* pkv_last_launch_error(void) { return hipGetErrorString(g_last_launch_error); }

int pkv_set_id_fault_counter(int32_t* device_counter) {
  if (reinterpret_cast<uintptr_t>(device_counter) & 3u) return PKV_ERR_ALIGN;
  g_id_faults = device_counter;
  return PKV_OK;
}

int pkv_probe_stream_read(const void* k_buf, const void* v_buf, int64_t num_slabs,
                          int64_t total_blocks, void* sink, void* stream) {
  if (num_slabs < 1 || total_blocks < 0 || total_blocks > INT32_MAX) return PKV_ERR_SHAPE;
  if (total_blocks == 0) return PKV_OK;
  if (!k_buf || !v_buf) return PKV_ERR_NULL;
  if (misaligned16(k_buf) || misaligned16(v_buf) || (reinterpret_cast<uintptr_t>(sink) & 3u))
    return PKV_ERR_ALIGN;
  // slab numbers are 32-bit on the device; a larger buffer is used up to 2^30 slabs (4 TiB)
  const uint32_t slabs = num_slabs > ((int64_t)1 << 30) ? (1u << 30) : (uint32_t)num_slabs;
  return launch_status(pkv::launch_stream_read_probe(k_buf, v_buf, slabs, total_blocks, sink,
                                                     static_cast<hipStream_t>(stream)));
}

int pkv_attn_partition_size(const pkv_attn_shape* shape) {
  Geometry g;
  const int rc = check_shape(shape, &g);
  return rc != PKV_OK ? rc : g.P;
}

int pkv_attn_workspace_bytes(const pkv_attn_shape* shape, size_t* out_bytes) {
  if (!out_bytes) return PKV_ERR_NULL;
  Geometry g;
  const int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  *out_bytes = workspace_bytes(shape, g);
  return PKV_OK;
}

// Validation shared by the single-layer and the multi-layer call; fills the
// launch descriptor except for the per-layer pointers.
static int prepare_attn(const int32_t* block_tables, const int32_t* context_lens, float scale, bool kv_fp8,
                        const pkv_attn_shape* shape, void* workspace, size_t workspace_bytes_given,
                        pkv::AttnLaunch* a, bool* empty) {
  Geometry g;
  const int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  *empty = shape->num_seqs == 0;
  if (*empty) return PKV_OK;
  if (!block_tables || !context_lens) return PKV_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(block_tables) & 3u) || (reinterpret_cast<uintptr_t>(context_lens) & 3u))
    return PKV_ERR_ALIGN;
  const size_t need = workspace_bytes(shape, g);
  if (need) {
    if (!workspace || workspace_bytes_given < need) return PKV_ERR_WORKSPACE;
    if (misaligned16(workspace)) return PKV_ERR_ALIGN;
  }
  a->block_tables = block_tables;
  a->context_lens = context_lens;
  a->S = shape->num_seqs;
  a->Hq = shape->num_q_heads;
  a->Hkv = shape->num_kv_heads;
  a->G = g.G;
  a->D = shape->head_dim;
  a->waves = pkv::kLayerGroups * pkv::group_waves(shape->head_dim);
  const int group = pkv::group_waves(shape->head_dim);
  const int64_t segments = (int64_t)a->S * a->Hkv;
  const int64_t max_blocks = (g.max_ctx + pkv::kBlockTokens - 1) / pkv::kBlockTokens;
  a->short_blocks = pkv::short_segment(segments, a->D, kv_fp8);
  a->leaves_records = 1;
  if (segments <= a->waves / group && max_blocks <= a->short_blocks) {
    // Cut along its segments, a workgroup for each.  Nothing is left in the workspace, and the layers of such
    // a launch may be more than it has room for.
    a->leaves_records = 0;
    a->waves = (int)segments * group;
  }
  a->id_faults = g_id_faults;
  a->MAXB = shape->max_blocks_per_seq;
  a->upb = shape->block_size / pkv::kBlockTokens;
  a->P = g.P;
  a->max_ctx = g.max_ctx;
  a->NB = (int)shape->num_pool_blocks;
  a->scale_log2e = scale * 1.4426950408889634f;
  a->out_scale = 1.f;
  a->kv_fp8 = kv_fp8;
  a->ws_rec = static_cast<float*>(workspace);
  a->ws_words = a->ws_rec + (int64_t)pkv::kRecordsBeforeWords * pkv::record_floats(a->G, a->D);
  a->layer_ws_floats = pkv::layer_ws_floats(g.G, a->D);
  return PKV_OK;
}

static int check_layer_pointers(const void* q, const void* k_pool, const void* v_pool, const void* out) {
  if (!q || !k_pool || !v_pool || !out) return PKV_ERR_NULL;
  if (misaligned16(q) || misaligned16(k_pool) || misaligned16(v_pool) || misaligned16(out))
    return PKV_ERR_ALIGN;
  return PKV_OK;
}

static pkv::AttnLayer layer_of(const void* q, const void* k_pool, const void* v_pool, void* out) {
  return pkv::AttnLayer{static_cast<const uint16_t*>(q), k_pool, v_pool, static_cast<uint16_t*>(out)};
}

// The launches for the layer of `a`, or for `layers`.
static int launch_attn(const pkv::AttnLaunch& a, const pkv::AttnLayers* layers, hipStream_t st) {
  hipError_t e = pkv::launch_attn_stream(a, layers, st);
  if (e == hipSuccess && a.leaves_records) e = pkv::launch_attn_reduce(a, layers, st);
  if (e != hipSuccess) return launch_status(e);
  return PKV_OK;
}

static uint64_t row_bytes(const pkv::AttnLaunch& a) { return (uint64_t)a.S * a.Hq * a.D * 2; }

// Does layer x's output overlap these bytes?
static bool overlaps(const pkv::AttnLaunch& a, const pkv::AttnLayer& x, const void* p, uint64_t bytes) {
  const uint64_t out = reinterpret_cast<uintptr_t>(x.out), at = reinterpret_cast<uintptr_t>(p);
  return out < at + bytes && at < out + row_bytes(a);
}

static bool overlaps_pools(const pkv::AttnLaunch& a, const pkv::AttnLayer& x, const pkv::AttnLayer& y) {
  const uint64_t pool = (uint64_t)a.NB * a.Hkv * a.upb * pkv::kBlockTokens * a.D * (a.kv_fp8 ? 1 : 2);
  return overlaps(a, x, y.k_pool, pool) || overlaps(a, x, y.v_pool, pool);
}

// Does what layer x writes overlap what layer y reads or writes?  Then they cannot share a launch.
static bool writes_into(const pkv::AttnLaunch& a, const pkv::AttnLayer& x, const pkv::AttnLayer& y) {
  return overlaps(a, x, y.q, row_bytes(a)) || overlaps(a, x, y.out, row_bytes(a)) || overlaps_pools(a, x, y);
}

// Does a layer write into its own inputs?  The stream pass stores rows while others are still being read, which
// is right where the output is q itself: a segment's rows of q are read by those who write them.
static bool writes_own_input(const pkv::AttnLaunch& a, const pkv::AttnLayer& x) {
  return (x.out != x.q && overlaps(a, x, x.q, row_bytes(a))) || overlaps_pools(a, x, x) ||
         overlaps(a, x, a.block_tables, (uint64_t)a.S * a.MAXB * 4) || overlaps(a, x, a.context_lens, (uint64_t)a.S * 4);
}

// One layer.  Where it writes into its own inputs the rows are kept at the end of the workspace's room for records until all
// is read: a layer's records and words leave three quarters of it.
static int launch_layer(pkv::AttnLaunch a, const pkv::AttnLayer& layer, hipStream_t st) {
  a.layer = layer;
  if (!writes_own_input(a, layer)) return launch_attn(a, nullptr, st);
  a.layer.out = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(a.ws_rec + record_slots(a.S, a.Hkv) * pkv::record_floats(a.G, a.D)) - row_bytes(a));
  const int rc = launch_attn(a, nullptr, st);
  if (rc != PKV_OK) return rc;
  return launch_status(pkv::launch_copy(a.layer.out, layer.out, row_bytes(a), st));
}

int paged_decode_attn(const void* q, const void* k_pool, const void* v_pool,
                      const int32_t* block_tables, const int32_t* context_lens, float scale,
                      void* out, const pkv_attn_shape* shape, void* workspace,
                      size_t workspace_bytes_given, void* stream) {
  pkv::AttnLaunch a;
  bool empty = false;
  int rc = prepare_attn(block_tables, context_lens, scale, false, shape, workspace, workspace_bytes_given,
                        &a, &empty);
  if (rc != PKV_OK || empty) return rc;
  rc = check_layer_pointers(q, k_pool, v_pool, out);
  if (rc != PKV_OK) return rc;
  return launch_layer(a, layer_of(q, k_pool, v_pool, out), static_cast<hipStream_t>(stream));
}

int paged_decode_attn_fp8kv(const void* q, const void* k_pool, const void* v_pool,
                            const int32_t* block_tables, const int32_t* context_lens, float scale,
                            float k_scale, float v_scale, void* out, const pkv_attn_shape* shape,
                            void* workspace, size_t workspace_bytes_given, void* stream) {
  Geometry g;
  int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  if (!(k_scale > 0.f) || !(v_scale > 0.f) || !(k_scale < __builtin_inff()) ||
      !(v_scale < __builtin_inff()))
    return PKV_ERR_SHAPE;
  pkv::AttnLaunch a;
  bool empty = false;
  rc = prepare_attn(block_tables, context_lens, scale, true, shape, workspace, workspace_bytes_given, &a,
                    &empty);
  if (rc != PKV_OK || empty) return rc;
  rc = check_layer_pointers(q, k_pool, v_pool, out);
  if (rc != PKV_OK) return rc;
  // K = k_scale * e4m3: the factor joins the softmax scale; V = v_scale * e4m3: applied once
  // to the normalised row
  a.scale_log2e = scale * k_scale * 1.4426950408889634f;
  a.out_scale = v_scale;
  return launch_layer(a, layer_of(q, k_pool, v_pool, out), static_cast<hipStream_t>(stream));
}

int paged_decode_attn_static(const void* q, const void* k_pool, const void* v_pool,
                             const int32_t* block_tables, const int32_t* context_lens, float scale,
                             void* out, const pkv_attn_shape* shape, void* stream) {
  Geometry g;
  int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  if (shape->num_seqs == 0) return PKV_OK;
  if (workspace_bytes(shape, g) > kStaticScratchBytes) return PKV_ERR_WORKSPACE;
  rc = check_layer_pointers(q, k_pool, v_pool, out);
  if (rc != PKV_OK) return rc;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != PKV_OK) return rc;
  pkv::AttnLaunch a;
  bool empty = false;
  rc = prepare_attn(block_tables, context_lens, scale, false, shape, ws, kStaticScratchBytes, &a, &empty);
  if (rc != PKV_OK || empty) return rc;
  return launch_layer(a, layer_of(q, k_pool, v_pool, out), static_cast<hipStream_t>(stream));
}

int paged_decode_attn_layers(const void* const* q, const void* const* k_pools,
                             const void* const* v_pools, const int32_t* block_tables,
                             const int32_t* context_lens, float scale, void* const* out,
                             int32_t num_layers, const pkv_attn_shape* shape, void* workspace,
                             size_t workspace_bytes_given, void* stream) {
  if (num_layers < 0) return PKV_ERR_SHAPE;
  pkv::AttnLaunch a;
  bool empty = false;
  int rc = prepare_attn(block_tables, context_lens, scale, false, shape, workspace, workspace_bytes_given,
                        &a, &empty);
  if (rc != PKV_OK || empty || num_layers == 0) return rc;
  if (!q || !k_pools || !v_pools || !out) return PKV_ERR_NULL;
  // every layer is checked before the first launch: an error enqueues nothing
  for (int32_t l = 0; l < num_layers; ++l) {
    rc = check_layer_pointers(q[l], k_pools[l], v_pools[l], out[l]);
    if (rc != PKV_OK) return rc;
  }
  // Several layers to a launch, as many as the workspace holds records for: a workgroup goes on
  // to the next layer when it is done with its share of one, and the start, the uneven end and the reduce
  // pass of a launch are paid once (6 layers of 24 requests in two launches: 812 -> 789 us).  A batch that
  // leaves no records needs none of it.  Layers that depend on each other keep their order.
  Geometry g;
  (void)check_shape(shape, &g);
  const int64_t room = a.leaves_records ? g.slots * pkv::record_floats(a.G, a.D) / a.layer_ws_floats : pkv::kMaxLaunchLayers;
  const int most = room < pkv::kMaxLaunchLayers ? (int)room : pkv::kMaxLaunchLayers;
  const int launches = (num_layers + most - 1) / most;
  const int even = (num_layers + launches - 1) / launches;
  pkv::AttnLayers layers;
  for (int32_t l = 0; l < num_layers; l += layers.count) {
    layers.count = 0;
    while (layers.count < even && l + layers.count < num_layers) {
      const int32_t next = l + layers.count;
      const pkv::AttnLayer y = layer_of(q[next], k_pools[next], v_pools[next], out[next]);
      bool apart = layers.count == 0 || !writes_own_input(a, y);
      for (int i = 0; i < layers.count; ++i)
        apart = apart && !writes_into(a, layers.layer[i], y) && !writes_into(a, y, layers.layer[i]);
      if (!apart) break;
      layers.layer[layers.count++] = y;
      if (writes_own_input(a, y)) break;
    }
    rc = layers.count > 1 ? launch_attn(a, &layers, static_cast<hipStream_t>(stream))
                          : launch_layer(a, layers.layer[0], static_cast<hipStream_t>(stream));
    if (rc != PKV_OK) return rc;
  }
  return PKV_OK;
}

int kv_append(const void* k_new, const void* v_new, void* k_pool, void* v_pool,
              const int32_t* block_tables, const int32_t* context_lens,
              const pkv_attn_shape* shape, void* stream) {
  Geometry g;
  const int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  if (shape->num_seqs == 0) return PKV_OK;
  if (!k_new || !v_new || !k_pool || !v_pool || !block_tables || !context_lens) return PKV_ERR_NULL;
  if (misaligned16(k_new) || misaligned16(v_new) || misaligned16(k_pool) || misaligned16(v_pool) ||
      (reinterpret_cast<uintptr_t>(block_tables) & 3u) || (reinterpret_cast<uintptr_t>(context_lens) & 3u))
    return PKV_ERR_ALIGN;
  const hipError_t e = pkv::launch_kv_append(
      static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new),
      static_cast<uint16_t*>(k_pool), static_cast<uint16_t*>(v_pool), block_tables, context_lens,
      shape->num_seqs, shape->num_kv_heads, shape->head_dim, shape->max_blocks_per_seq,
      shape->block_size, g.max_ctx, (int)shape->num_pool_blocks, g_id_faults,
      static_cast<hipStream_t>(stream));
  return launch_status(e);
}

int kv_append_fp8(const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                  const int32_t* block_tables, const int32_t* context_lens, float k_scale,
                  float v_scale, const pkv_attn_shape* shape, void* stream) {
  Geometry g;
  const int rc = check_shape(shape, &g);
  if (rc != PKV_OK) return rc;
  if (!(k_scale > 0.f) || !(v_scale > 0.f) || !(k_scale < __builtin_inff()) ||
      !(v_scale < __builtin_inff()))
    return PKV_ERR_SHAPE;
  if (shape->num_seqs == 0) return PKV_OK;
  if (!k_new || !v_new || !k_pool || !v_pool || !block_tables || !context_lens) return PKV_ERR_NULL;
  if (misaligned16(k_new) || misaligned16(v_new) || misaligned16(k_pool) || misaligned16(v_pool) ||
      (reinterpret_cast<uintptr_t>(block_tables) & 3u) || (reinterpret_cast<uintptr_t>(context_lens) & 3u))
    return PKV_ERR_ALIGN;
  const hipError_t e = pkv::launch_kv_append_fp8(
      static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), k_pool, v_pool,
      block_tables, context_lens, k_scale, v_scale, shape->num_seqs, shape->num_kv_heads,
      shape->head_dim, shape->max_blocks_per_seq, shape->block_size, g.max_ctx,
      (int)shape->num_pool_blocks, g_id_faults, static_cast<hipStream_t>(stream));
  return launch_status(e);
}

// Host-visible checks of a block copy; *empty is set when there is nothing to do.
static int check_copy(const void* pool, const void* staging, const int32_t* block_ids,
                      int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks, bool* empty) {
  *empty = false;
  if (n_blocks < 0 || block_bytes <= 0 || num_pool_blocks < 0) return PKV_ERR_SHAPE;
  if (block_bytes % 16 != 0) return PKV_ERR_ALIGN;
  if (n_blocks > INT32_MAX || block_bytes > ((int64_t)1 << 30)) return PKV_ERR_SHAPE;
  *empty = n_blocks == 0;
  if (*empty) return PKV_OK;
  if (!pool || !staging || !block_ids) return PKV_ERR_NULL;
  if (misaligned16(pool) || misaligned16(staging) || (reinterpret_cast<uintptr_t>(block_ids) & 3u))
    return PKV_ERR_ALIGN;
  return PKV_OK;
}

// The far end of an offload or reload must be page-locked host memory: only
// then is the copy asynchronous and done by the DMA engines at link speed.
static int check_pinned(const void* host, size_t bytes) {
  // the first and the last byte must both lie in page-locked host memory
  const char* ends[2] = {static_cast<const char*>(host), static_cast<const char*>(host) + (bytes - 1)};
  for (const char* p : ends) {
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
      (void)hipGetLastError();   // an unknown pointer is reported as an error; clear it
      return PKV_ERR_HOST;
    }
    if (attr.type != hipMemoryTypeHost) return PKV_ERR_HOST;
  }
  return PKV_OK;
}

static int copy_call(const void* pool, const void* staging, const int32_t* block_ids,
                     int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks, bool gather,
                     void* stream) {
  bool empty = false;
  const int rc = check_copy(pool, staging, block_ids, n_blocks, block_bytes, num_pool_blocks, &empty);
  if (rc != PKV_OK || empty) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const hipError_t e =
      gather ? pkv::launch_kv_block_copy(pool, const_cast<void*>(staging), block_ids, n_blocks,
                                         block_bytes, num_pool_blocks, true, g_id_faults, st)
             : pkv::launch_kv_block_copy(staging, const_cast<void*>(pool), block_ids, n_blocks,
                                         block_bytes, num_pool_blocks, false, g_id_faults, st);
  return launch_status(e);
}

int kv_blocks_gather(const void* pool, const int32_t* block_ids, void* staging, int64_t n_blocks,
                     int64_t block_bytes, int64_t num_pool_blocks, void* stream) {
  return copy_call(pool, staging, block_ids, n_blocks, block_bytes, num_pool_blocks, true, stream);
}

int kv_blocks_scatter(const void* staging, void* pool, const int32_t* block_ids, int64_t n_blocks,
                      int64_t block_bytes, int64_t num_pool_blocks, void* stream) {
  return copy_call(pool, staging, block_ids, n_blocks, block_bytes, num_pool_blocks, false, stream);
}

int kv_blocks_move(const void* src_pool, const int32_t* src_ids, void* dst_pool,
                   const int32_t* dst_ids, int64_t n_blocks, int64_t block_bytes,
                   int64_t src_pool_blocks, int64_t dst_pool_blocks, void* stream) {
  if (n_blocks < 0 || block_bytes <= 0 || src_pool_blocks < 0 || dst_pool_blocks < 0) return PKV_ERR_SHAPE;
  if (block_bytes % 16 != 0) return PKV_ERR_ALIGN;
  if (n_blocks > INT32_MAX || block_bytes > ((int64_t)1 << 30)) return PKV_ERR_SHAPE;
  if (n_blocks == 0) return PKV_OK;
  if (!src_pool || !dst_pool || !src_ids || !dst_ids) return PKV_ERR_NULL;
  if (misaligned16(src_pool) || misaligned16(dst_pool) || (reinterpret_cast<uintptr_t>(src_ids) & 3u) ||
      (reinterpret_cast<uintptr_t>(dst_ids) & 3u))
    return PKV_ERR_ALIGN;
  return launch_status(pkv::launch_kv_block_move(src_pool, src_ids, src_pool_blocks, dst_pool, dst_ids,
                                                 dst_pool_blocks, n_blocks, block_bytes, g_id_faults,
                                                 static_cast<hipStream_t>(stream)));
}

int kv_blocks_offload(const void* pool, const int32_t* block_ids, void* staging, void* host_dst,
                      int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks, void* stream) {
  bool empty = false;
  int rc = check_copy(pool, staging, block_ids, n_blocks, block_bytes, num_pool_blocks, &empty);
  if (rc != PKV_OK || empty) return rc;
  if (!host_dst) return PKV_ERR_NULL;
  rc = check_pinned(host_dst, (size_t)n_blocks * (size_t)block_bytes);
  if (rc != PKV_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e = pkv::launch_kv_block_copy(pool, staging, block_ids, n_blocks, block_bytes,
                                           num_pool_blocks, true, g_id_faults, st);
  if (e != hipSuccess) return launch_status(e);
  e = hipMemcpyAsync(host_dst, staging, (size_t)n_blocks * (size_t)block_bytes,
                     hipMemcpyDeviceToHost, st);
  return launch_status(e);
}

int kv_blocks_reload(const void* host_src, void* staging, void* pool, const int32_t* block_ids,
                     int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks, void* stream) {
  bool empty = false;
  int rc = check_copy(pool, staging, block_ids, n_blocks, block_bytes, num_pool_blocks, &empty);
  if (rc != PKV_OK || empty) return rc;
  if (!host_src) return PKV_ERR_NULL;
  rc = check_pinned(host_src, (size_t)n_blocks * (size_t)block_bytes);
  if (rc != PKV_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e = hipMemcpyAsync(staging, host_src, (size_t)n_blocks * (size_t)block_bytes,
                                hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return launch_status(e);
  e = pkv::launch_kv_block_copy(staging, pool, block_ids, n_blocks, block_bytes, num_pool_blocks,
                                false, g_id_faults, st);
  return launch_status(e);
}

}  // extern "C"
