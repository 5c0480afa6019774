// C-ABI entry points: host-side argument checks, kernel selection, ring drivers.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "cp_common.h"

using namespace cp;

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

int check_shape(const cp_shape* s) {
  if (s == nullptr) return CP_ERR_NULL;
  if (s->dtype != CP_BF16 && s->dtype != CP_FP32) return CP_ERR_UNSUPPORTED;
  if (s->head_dim != 64 && s->head_dim != 128) return CP_ERR_UNSUPPORTED;
  if (s->n_q_heads < 1 || s->n_kv_heads < 1 || s->n_q_heads % s->n_kv_heads != 0)
    return CP_ERR_SHAPE;
  if (s->batch < 1 || s->total_q < 0 || s->total_kv < 0) return CP_ERR_SHAPE;
  if (s->total_q > 0x7fffffffLL || s->total_kv > 0x7fffffffLL) return CP_ERR_SHAPE;
  if ((s->flags & ~CP_SHAPE_UNIQUE_BID) != 0 || s->reserved_f != 0.f) return CP_ERR_SHAPE;
  if (!(s->softmax_scale == s->softmax_scale) || isinf(s->softmax_scale)) return CP_ERR_SHAPE;
  return CP_OK;
}

inline float resolve_scale(float scale, int head_dim) {
  return scale > 0.f ? scale : 1.0f / sqrtf((float)head_dim);
}

// Calls of the MFMA kernel: one sequence of either head_dim, packed batches of head_dim 128.
inline bool mfma_applies(const cp_shape& s) {
  return attn_mfma_applies(s.dtype, s.head_dim, s.n_q_heads, s.n_kv_heads) &&
         (s.batch == 1 || s.head_dim == 128);
}

inline int32_t kv_blocks(int64_t n_kv) { return (int32_t)((n_kv + kAttnBlock - 1) / kAttnBlock); }

// One rank's queries against one shard, as an attention launch sees it.
AttnShape single_shape(const cp_shape& s) {
  AttnShape a = {};
  a.dtype = s.dtype; a.head_dim = s.head_dim;
  a.n_q_heads = s.n_q_heads; a.n_kv_heads = s.n_kv_heads;
  a.total_q = s.total_q; a.n_blocks = kv_blocks(s.total_kv); a.n_shards = 1; a.batch = s.batch;
  return a;
}

inline size_t elem_size(int32_t dtype) { return dtype == CP_FP32 ? 4 : 2; }

AttnTable single_table(const cp_shape& s, const void* q, const void* k, const void* v,
                       const int32_t* q_pos, const int32_t* kv_pos, void* out, float* lse) {
  AttnTable t = {};
  t.n_ranks = t.n_shards = 1;
  t.q[0] = q; t.q_pos[0] = q_pos; t.out[0] = out; t.lse[0] = lse;
  t.k[0] = k; t.v[0] = v; t.kv_pos[0] = kv_pos;
  t.n_kv[0] = (int32_t)s.total_kv;
  t.tok_begin[1] = (int32_t)s.total_q;
  t.blk_begin[1] = kv_blocks(s.total_kv);
  return t;
}

}  // namespace

// Scratch of cp_attn_decode_static: split-KV partials live here instead of in a caller's
// workspace, so that the call allocates nothing. Every GPU holds its own copy of the array at
// its own address; in host code the array's name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[CP_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CP_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return CP_ERR_LAUNCH;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return CP_OK;
}

}  // namespace

extern "C" {

int cp_version(void) { return 100; }

const char* cp_strerror(int status) {
  switch (status) {
    case CP_OK: return "ok";
    case CP_ERR_NULL: return "a required pointer is NULL";
    case CP_ERR_SHAPE: return "invalid or inconsistent shape";
    case CP_ERR_UNSUPPORTED: return "dtype / head_dim / combination not supported";
    case CP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case CP_ERR_LAUNCH: return "HIP kernel launch failed";
    case CP_ERR_ALIGN: return "tensor pointer is not 16-byte aligned";
    default: return "unknown status";
  }
}

int cp_shard_positions(int64_t total, int64_t offset, int32_t n_ranks, int32_t rank,
                       int32_t* pos_out, int64_t* n_out) {
  if (n_out == nullptr) return CP_ERR_NULL;
  if (total < 0 || n_ranks < 1 || rank < 0 || rank >= n_ranks) return CP_ERR_SHAPE;
  if (offset < 0 || total + offset > 0x7fffffffLL) return CP_ERR_SHAPE;
  const int64_t n_chunks = 2 * (int64_t)n_ranks;
  const int64_t size = (total + n_chunks - 1) / n_chunks;
  const int64_t chunk[2] = {rank, n_chunks - 1 - rank};
  int64_t n = 0;
  for (int c = 0; c < 2; ++c) {
    const int64_t lo = std::min(chunk[c] * size, total);
    const int64_t hi = std::min((chunk[c] + 1) * size, total);
    for (int64_t p = lo; p < hi; ++p, ++n)
      if (pos_out != nullptr) pos_out[n] = (int32_t)(p + offset);
  }
  *n_out = n;
  return CP_OK;
}

size_t cp_workspace_bytes(const cp_shape* shape, int32_t kind) {
  if (check_shape(shape) != CP_OK) return 0;
  switch (kind) {
    case CP_WS_PARTIAL:
      if (!mfma_applies(*shape)) return 0;
      return attn_mfma_workspace_bytes(single_shape(*shape)) +
             (shape->batch > 1
                  ? varseq_workspace_bytes(shape->batch, shape->total_q, shape->total_kv)
                  : 0);
    case CP_WS_DECODE:
      return decode_workspace_bytes(*shape);
    default:
      return 0;
  }
}

int cp_attn_partial(const cp_shape* shape, const void* q, const void* k, const void* v,
                    const int32_t* q_pos, const int32_t* kv_pos, const int32_t* cu_seqlens_q,
                    const int32_t* cu_seqlens_kv, void* out, float* lse, int32_t out_dtype,
                    void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape);
  if (rc != CP_OK) return rc;
  const cp_shape& s = *shape;
  if (out_dtype != CP_BF16 && out_dtype != CP_FP32) return CP_ERR_UNSUPPORTED;
  if ((cu_seqlens_q == nullptr) != (cu_seqlens_kv == nullptr)) return CP_ERR_NULL;
  if (cu_seqlens_q == nullptr && s.batch != 1) return CP_ERR_SHAPE;
  if (s.total_q > 0 && (q == nullptr || q_pos == nullptr || out == nullptr || lse == nullptr))
    return CP_ERR_NULL;
  if (s.total_q > 0 && s.total_kv > 0 && (k == nullptr || v == nullptr || kv_pos == nullptr))
    return CP_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return CP_ERR_ALIGN;
  if (s.total_q == 0) return CP_OK;
  const float scale = resolve_scale(s.softmax_scale, s.head_dim);
  hipStream_t st = (hipStream_t)stream;
  AttnShape as = single_shape(s);
  as.scale = scale;
  AttnTable t = single_table(s, q, k, v, q_pos, kv_pos, out, lse);
  const AttnOut ao = {out_dtype, 0, 0};
  // (one sequence: the cu_seqlens of a batch of one say nothing new to the MFMA kernel)
  const bool packed = cu_seqlens_q != nullptr && s.batch > 1;
  if (mfma_applies(s) && (cu_seqlens_q == nullptr || s.head_dim == 128)) {
    const size_t enc = packed ? varseq_workspace_bytes(s.batch, s.total_q, s.total_kv) : 0;
    const size_t need = enc + attn_mfma_workspace_bytes(as);
    if (need > 0 && (workspace == nullptr || !aligned256(workspace) || workspace_bytes < need))
      return CP_ERR_WORKSPACE;
    const int32_t* q_lo = nullptr;
    if (packed) {  // shift every sequence into its own position range, then one launch
      rc = launch_varseq_encode(s.batch, s.total_kv, t, &cu_seqlens_q, &cu_seqlens_kv, workspace,
                                &q_lo, st);
      if (rc != CP_OK) return rc;
    }
    return launch_attn_mfma(as, t, ao, q_lo, (char*)workspace + enc,
                            workspace_bytes - enc, nullptr, nullptr, st);
  }
  if (s.dtype == CP_FP32 && cu_seqlens_q == nullptr) return launch_attn_fp32(as, t, ao, st);
  return launch_partial_generic(s, scale, q, k, v, q_pos, kv_pos, cu_seqlens_q, cu_seqlens_kv,
                                out, lse, out_dtype, st);
}

int cp_attn_partial_accumulate(const cp_shape* shape, const void* q, const void* k,
                               const void* v, const int32_t* q_pos, const int32_t* kv_pos,
                               float* acc_out, float* acc_lse, void* final_out,
                               int32_t final_dtype, float* final_lse, void* workspace,
                               size_t workspace_bytes, void* stream) {
  int rc = check_shape(shape);
  if (rc != CP_OK) return rc;
  const cp_shape& s = *shape;
  if (final_out != nullptr && final_dtype != CP_BF16 && final_dtype != CP_FP32)
    return CP_ERR_UNSUPPORTED;
  if (s.batch != 1 || !mfma_applies(s) || !attn_mfma_merging_applies(single_shape(s)))
    return CP_ERR_UNSUPPORTED;
  if (s.total_q > 0 && (q == nullptr || q_pos == nullptr || acc_out == nullptr || acc_lse == nullptr))
    return CP_ERR_NULL;
  if (s.total_q > 0 && s.total_kv > 0 && (k == nullptr || v == nullptr || kv_pos == nullptr))
    return CP_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(acc_out) || !aligned16(final_out))
    return CP_ERR_ALIGN;
  if (s.total_q == 0) return CP_OK;
  AttnShape as = single_shape(s);
  as.scale = resolve_scale(s.softmax_scale, s.head_dim);
  const size_t need = attn_mfma_workspace_bytes(as);
  if (need > 0 && (workspace == nullptr || !aligned256(workspace) || workspace_bytes < need))
    return CP_ERR_WORKSPACE;
  const AttnTable t = single_table(s, q, k, v, q_pos, kv_pos, nullptr, acc_lse);
  const PrefillAccumulate acc = {acc_out, acc_lse, final_out, final_lse, final_dtype};
  return launch_attn_mfma_accumulate(as, t, acc, workspace, workspace_bytes, nullptr,
                                     (hipStream_t)stream);
}

// Argument checks shared by cp_attn_decode and cp_attn_decode_static. Returns CP_OK with
// *launch = false when there is nothing to do.
static int check_decode(const cp_shape* shape, const void* q, const void* k, const void* v,
                        const int32_t* q_pos, const int32_t* kv_pos, const int32_t* cu_seqlens_kv,
                        const int32_t* bid, const void* out, const float* lse, int32_t out_dtype,
                        bool* launch) {
  *launch = false;
  int rc = check_shape(shape);
  if (rc != CP_OK) return rc;
  const cp_shape& s = *shape;
  if (out_dtype != CP_BF16 && out_dtype != CP_FP32) return CP_ERR_UNSUPPORTED;
  if (s.dtype != CP_BF16 || s.head_dim != 128) return CP_ERR_UNSUPPORTED;
  if (s.n_q_heads / s.n_kv_heads > 16) return CP_ERR_UNSUPPORTED;
  if (cu_seqlens_kv == nullptr) return CP_ERR_NULL;
  if (s.total_q > 0 &&
      (q == nullptr || q_pos == nullptr || bid == nullptr || out == nullptr || lse == nullptr))
    return CP_ERR_NULL;
  if (s.total_q > 0 && s.total_kv > 0 && (k == nullptr || v == nullptr || kv_pos == nullptr))
    return CP_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return CP_ERR_ALIGN;
  *launch = s.total_q > 0;
  return CP_OK;
}

int cp_attn_decode(const cp_shape* shape, const void* q, const void* k, const void* v,
                   const int32_t* q_pos, const int32_t* kv_pos, const int32_t* cu_seqlens_kv,
                   const int32_t* bid, void* out, float* lse, int32_t out_dtype,
                   void* workspace, size_t workspace_bytes, void* stream) {
  bool launch = false;
  const int rc = check_decode(shape, q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out, lse,
                              out_dtype, &launch);
  if (rc != CP_OK || !launch) return rc;
  const cp_shape& s = *shape;
  const size_t need = decode_workspace_bytes(s);
  if (need > 0 && (workspace == nullptr || !aligned256(workspace) || workspace_bytes < need))
    return CP_ERR_WORKSPACE;
  const float scale = resolve_scale(s.softmax_scale, s.head_dim);
  return launch_decode(s, scale, q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out, lse, out_dtype,
                       workspace, workspace_bytes, (hipStream_t)stream);
}

int cp_attn_decode_static(const cp_shape* shape, const void* q, const void* k, const void* v,
                          const int32_t* q_pos, const int32_t* kv_pos,
                          const int32_t* cu_seqlens_kv, const int32_t* bid, void* out, float* lse,
                          int32_t out_dtype, void* stream) {
  bool launch = false;
  const int rc = check_decode(shape, q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out, lse,
                              out_dtype, &launch);
  if (rc != CP_OK || !launch) return rc;
  const cp_shape& s = *shape;
  if (decode_workspace_bytes(s) > CP_STATIC_SCRATCH_BYTES) return CP_ERR_WORKSPACE;
  void* ws = nullptr;
  const int rs = static_scratch(&ws);
  if (rs != CP_OK) return rs;
  const float scale = resolve_scale(s.softmax_scale, s.head_dim);
  return launch_decode(s, scale, q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out, lse, out_dtype,
                       ws, CP_STATIC_SCRATCH_BYTES, (hipStream_t)stream);
}

int cp_attn_merge(int64_t rows, int32_t head_dim, int32_t n_parts, const void* const* outs,
                  const float* const* lses, int32_t part_dtype, void* out, int32_t out_dtype,
                  float* lse_out, void* stream) {
  if (rows < 0 || head_dim < 8 || head_dim > 256 || head_dim % 8 != 0) return CP_ERR_SHAPE;
  if (n_parts < 1 || n_parts > CP_MAX_PARTS) return CP_ERR_SHAPE;
  if ((part_dtype != CP_BF16 && part_dtype != CP_FP32) ||
      (out_dtype != CP_BF16 && out_dtype != CP_FP32))
    return CP_ERR_UNSUPPORTED;
  if (outs == nullptr || lses == nullptr) return CP_ERR_NULL;
  if (rows > 0) {
    if (out == nullptr) return CP_ERR_NULL;
    for (int s = 0; s < n_parts; ++s) {
      if (outs[s] == nullptr || lses[s] == nullptr) return CP_ERR_NULL;
      if (!aligned16(outs[s])) return CP_ERR_ALIGN;
    }
    if (!aligned16(out)) return CP_ERR_ALIGN;
  }
  if (rows == 0) return CP_OK;
  return launch_merge(rows, head_dim, n_parts, outs, lses, part_dtype, out, out_dtype, lse_out,
                      (hipStream_t)stream);
}

}  // extern "C"

// ---------------------------------------------------------------------------
// ring drivers
// ---------------------------------------------------------------------------

// Prefill drivers over packed batches (the fused variable-length inputs of Algorithm 2): every
// rank's Q and KV hold `batch` sequences back to back with per-rank cu_seqlens.
static bool ring_is_packed(const cp_ring_desc* d, bool decode) {
  return !decode && d->cu_seqlens_q != nullptr;
}

static int check_ring(const cp_ring_desc* d, bool decode) {
  if (d == nullptr) return CP_ERR_NULL;
  if (d->n_ranks < 1 || d->n_ranks > CP_MAX_PARTS) return CP_ERR_SHAPE;
  if (d->fused_merge < 0 || d->fused_merge > 2) return CP_ERR_SHAPE;
  if (d->message_layout != 0 && d->message_layout != 1) return CP_ERR_SHAPE;
  if (d->gathered_q != 0 && d->gathered_q != 1) return CP_ERR_SHAPE;
  if (d->unique_bid != 0 && d->unique_bid != 1) return CP_ERR_SHAPE;
  if (d->gathered_q && (!d->keep_partials || d->message_layout || d->fused_merge))
    return CP_ERR_UNSUPPORTED;
  if (d->fused_merge && (decode || d->keep_partials || d->part_dtype != CP_FP32))
    return CP_ERR_UNSUPPORTED;
  if (d->n_q == nullptr || d->n_kv == nullptr || d->q == nullptr || d->k == nullptr ||
      d->v == nullptr || d->q_pos == nullptr || d->kv_pos == nullptr || d->out == nullptr)
    return CP_ERR_NULL;
  if (d->fused_merge == 2 && d->arrived != nullptr &&
      (d->ring_error == nullptr || d->spin_limit < 1))
    return CP_ERR_SHAPE;
  if (d->partial_out == nullptr || (d->partial_lse == nullptr && !d->message_layout))
    return CP_ERR_NULL;
  if (d->part_dtype != CP_BF16 && d->part_dtype != CP_FP32) return CP_ERR_UNSUPPORTED;
  if (d->out_dtype != CP_BF16 && d->out_dtype != CP_FP32) return CP_ERR_UNSUPPORTED;
  if (!aligned16(d->partial_out)) return CP_ERR_ALIGN;
  if (decode) {
    if (d->batch < 1 || d->cu_seqlens_kv == nullptr || d->bid == nullptr) return CP_ERR_NULL;
  }
  const bool packed = ring_is_packed(d, decode);
  if (packed) {
    if (d->batch < 1) return CP_ERR_SHAPE;
    if (d->cu_seqlens_kv == nullptr) return CP_ERR_NULL;
    if (d->fused_merge || d->gathered_q || d->aux_stream != nullptr) return CP_ERR_UNSUPPORTED;
  }
  cp_shape s = {};
  s.dtype = d->dtype; s.head_dim = d->head_dim; s.n_q_heads = d->n_q_heads;
  s.n_kv_heads = d->n_kv_heads; s.batch = (decode || packed) ? d->batch : 1;
  s.softmax_scale = d->softmax_scale;
  int rc = check_shape(&s);
  if (rc != CP_OK) return rc;
  for (int r = 0; r < d->n_ranks; ++r) {
    if (d->n_q[r] < 0 || d->n_kv[r] < 0) return CP_ERR_SHAPE;
    if (d->n_q[r] > 0 && (d->q[r] == nullptr || d->q_pos[r] == nullptr || d->out[r] == nullptr))
      return CP_ERR_NULL;
    if (d->n_kv[r] > 0 && (d->k[r] == nullptr || d->v[r] == nullptr || d->kv_pos[r] == nullptr))
      return CP_ERR_NULL;
    if (decode && (d->cu_seqlens_kv[r] == nullptr || (d->n_q[r] > 0 && d->bid[r] == nullptr)))
      return CP_ERR_NULL;
    if (packed && (d->cu_seqlens_q[r] == nullptr || d->cu_seqlens_kv[r] == nullptr))
      return CP_ERR_NULL;
  }
  return CP_OK;
}

static cp_shape ring_shape(const cp_ring_desc* d, int q_rank, int kv_rank, bool decode) {
  cp_shape s = {};
  s.dtype = d->dtype; s.head_dim = d->head_dim; s.n_q_heads = d->n_q_heads;
  s.n_kv_heads = d->n_kv_heads; s.batch = (decode || ring_is_packed(d, decode)) ? d->batch : 1;
  s.total_q = d->n_q[q_rank]; s.total_kv = d->n_kv[kv_rank];
  s.softmax_scale = d->softmax_scale;
  if (decode && d->unique_bid) s.flags = CP_SHAPE_UNIQUE_BID;
  return s;
}

// Prefill drivers: a ring is one attention launch over all its ranks and shards (AttnTable)
// wherever the kernels take it: up to kMaxTable ranks, bf16 in one sequence or packed with
// head_dim 128, fp32 in one sequence. Otherwise it is N x N partial-attention calls into the slots
// (N with gathered queries) and a merge per rank.
static bool ring_is_one_launch(const cp_ring_desc* d) {
  if (d->n_ranks > kMaxTable) return false;
  const bool packed = ring_is_packed(d, false);
  if (d->dtype == CP_FP32) {
    if (packed) return false;
  } else if (!attn_mfma_applies(d->dtype, d->head_dim, d->n_q_heads, d->n_kv_heads) ||
             (packed && d->head_dim != 128)) {
    return false;
  }
  // tokens, rows and tiles of all ranks together are kept in 31 bits
  int64_t tokens = 0, keys = 0;
  for (int r = 0; r < d->n_ranks; ++r) {
    if (d->n_q[r] > INT32_MAX || d->n_kv[r] > INT32_MAX - kAttnBlock) return false;
    tokens += d->n_q[r];
    keys += d->n_kv[r];
  }
  return tokens * (d->n_q_heads / d->n_kv_heads) <= INT32_MAX && tokens <= INT32_MAX &&
         keys <= (int64_t)INT32_MAX * 8;
}

static AttnShape ring_attn_shape(const cp_ring_desc* d) {
  AttnShape s = {};
  s.dtype = d->dtype; s.head_dim = d->head_dim;
  s.n_q_heads = d->n_q_heads; s.n_kv_heads = d->n_kv_heads;
  s.n_shards = d->n_ranks;
  s.batch = ring_is_packed(d, false) ? d->batch : 1;
  for (int r = 0; r < d->n_ranks; ++r) {
    s.total_q += d->n_q[r];
    s.n_blocks += kv_blocks(d->n_kv[r]);
  }
  s.per_shard = d->keep_partials != 0;
  s.scale = resolve_scale(d->softmax_scale, d->head_dim);
  return s;
}

static size_t ring_varseq_bytes(const cp_ring_desc* d) {
  if (!ring_is_packed(d, false)) return 0;
  int64_t tokens = 0, keys = 0;
  for (int r = 0; r < d->n_ranks; ++r) {
    tokens += d->n_q[r];
    keys += d->n_kv[r];
  }
  return varseq_workspace_bytes(d->batch, tokens, keys);
}

// The N x N calls of a ring on the MFMA kernel read every shard N times: its position bounds are
// made once, at the head of the ring's workspace. (Not of a packed batch, whose positions are
// shifted for every call.)
static bool ring_shares_bounds(const cp_ring_desc* d, bool decode) {
  return !decode && !ring_is_packed(d, decode) && mfma_applies(ring_shape(d, 0, 0, false));
}

// One of those calls, to the attention launch.
static AttnShape step_shape(const cp_shape& s) {
  AttnShape a = single_shape(s);
  a.has_bounds = true;
  a.scale = resolve_scale(s.softmax_scale, s.head_dim);
  return a;
}

// Shape of the one call KV holder b answers with when the queries are gathered.
static cp_shape gathered_shape(const cp_ring_desc* d, int b, bool decode) {
  cp_shape s = ring_shape(d, 0, b, decode);
  s.total_q = 0;
  for (int a = 0; a < d->n_ranks; ++a) s.total_q += d->n_q[a];
  return s;
}

extern "C" size_t cp_ring_workspace_bytes(const cp_ring_desc* d, int32_t decode) {
  if (check_ring(d, decode != 0) != CP_OK) return 0;
  if (!decode && ring_is_one_launch(d))
    return d->dtype == CP_FP32 ? 0
           : d->fused_merge == 2 && d->arrived != nullptr
               ? attn_mfma_ring_workspace_bytes(ring_attn_shape(d))
               : attn_mfma_workspace_bytes(ring_attn_shape(d)) + ring_varseq_bytes(d);
  const bool shared = ring_shares_bounds(d, decode != 0);
  auto call_bytes = [&](const cp_shape& s) -> size_t {
    if (!shared) return cp_workspace_bytes(&s, decode ? CP_WS_DECODE : CP_WS_PARTIAL);
    return check_shape(&s) == CP_OK ? attn_mfma_workspace_bytes(step_shape(s)) : 0;
  };
  size_t need = 0;
  for (int a = 0; a < d->n_ranks; ++a)
    for (int b = 0; b < d->n_ranks; ++b)
      need = std::max(need, call_bytes(ring_shape(d, a, b, decode != 0)));
  if (!decode && d->gathered_q)
    for (int b = 0; b < d->n_ranks; ++b) need = std::max(need, call_bytes(gathered_shape(d, b, false)));
  if (shared) need += kv_bounds_ring_bytes(d->n_ranks, d->n_kv);
  if (d->gathered_q && decode) {
    cp_shape shapes[CP_MAX_PARTS];
    bool flat = true;
    for (int b = 0; b < d->n_ranks; ++b) {
      shapes[b] = gathered_shape(d, b, true);
      need = std::max(need, cp_workspace_bytes(&shapes[b], CP_WS_DECODE));
      flat = flat && decode_flat_applies(shapes[b]);
    }
    if (flat) need = std::max(need, decode_flat_bytes(d->n_ranks, shapes));
  }
  return need;
}

namespace {

// Where the partial (O, LSE) of a slot live. Two buffers, or (message_layout) one buffer of
// messages, each the slot's O followed by its LSE: what the All2All of Algorithms 3 and 4
// moves as one piece, written in place by the attention kernel and read in place by the merge.
struct RingSlots {
  int64_t max_q = 0;
  size_t out_slot_bytes = 0;
  size_t lse_slot_elems = 0;
  size_t out_stride = 0;   // bytes between the O of consecutive slots
  bool messages = false;
  char* out_base = nullptr;
  float* lse_base = nullptr;
  void* out(int64_t slot) const { return out_base + slot * out_stride; }
  float* lse(int64_t slot) const {
    return messages ? (float*)(out_base + slot * out_stride + out_slot_bytes)
                    : lse_base + slot * lse_slot_elems;
  }
};

size_t ring_message_bytes(size_t out_slot_bytes, size_t lse_slot_elems) {
  return (out_slot_bytes + lse_slot_elems * sizeof(float) + 255) / 256 * 256;
}

RingSlots make_slots(const cp_ring_desc* d) {
  RingSlots r;
  for (int i = 0; i < d->n_ranks; ++i) r.max_q = std::max<int64_t>(r.max_q, d->n_q[i]);
  r.lse_slot_elems = (size_t)r.max_q * d->n_q_heads;
  r.out_slot_bytes = r.lse_slot_elems * d->head_dim * elem_size(d->part_dtype);
  r.messages = d->message_layout != 0;
  r.out_stride = r.messages ? ring_message_bytes(r.out_slot_bytes, r.lse_slot_elems)
                            : r.out_slot_bytes;
  r.out_base = (char*)d->partial_out;
  r.lse_base = d->partial_lse;
  return r;
}

// Slot of the partial of rank a's queries against rank b's KV: a holder's N slots in destination
// order with gathered queries, a source's N slots otherwise; without keep_partials the slots
// are reused for every rank.
int64_t slot_of(const cp_ring_desc* d, int a, int b) {
  if (!d->keep_partials) return b;
  return d->gathered_q ? (int64_t)b * d->n_ranks + a : (int64_t)a * d->n_ranks + b;
}

int check_ring_workspace(const cp_ring_desc* d, bool decode) {
  const size_t need = cp_ring_workspace_bytes(d, decode ? 1 : 0);
  if (need > 0 && (d->workspace == nullptr || !aligned256(d->workspace) ||
                   d->workspace_bytes < need))
    return CP_ERR_WORKSPACE;
  return CP_OK;
}

// What the options that ask for the merge inside the attention launch require: the MFMA kernel
// with head_dim 128 on one sequence per rank, and calls long enough not to split their KV axis.
int check_fused(const cp_ring_desc* d) {
  const int n = d->n_ranks;
  const bool mfma = attn_mfma_applies(d->dtype, d->head_dim, d->n_q_heads, d->n_kv_heads) &&
                    d->head_dim == 128;
  const bool walk = d->fused_merge == 2;
  if (n == 1 && !walk) return CP_OK;
  if (walk && n > kMaxTable) return CP_ERR_UNSUPPORTED;
  int64_t largest = 0;
  for (int b = 0; b < n; ++b) largest = std::max(largest, d->n_kv[b]);
  for (int a = 0; a < n; ++a) {
    if (!mfma) return CP_ERR_UNSUPPORTED;
    if (d->n_q[a] == 0) continue;
    cp_shape s = ring_shape(d, a, 0, false);
    for (int b = 0; b < n; ++b) {
      s.total_kv = d->n_kv[b];
      if (!attn_mfma_merging_applies(single_shape(s))) return CP_ERR_UNSUPPORTED;
    }
    s.total_kv = largest;
    if (walk && !attn_mfma_merging_applies(single_shape(s))) return CP_ERR_UNSUPPORTED;
  }
  return CP_OK;
}

int ring_merge(const cp_ring_desc* d, const RingSlots& slots, int a, hipStream_t st) {
  const void* outs[CP_MAX_PARTS];
  const float* lses[CP_MAX_PARTS];
  for (int b = 0; b < d->n_ranks; ++b) {
    outs[b] = slots.out(slot_of(d, a, b));
    lses[b] = slots.lse(slot_of(d, a, b));
  }
  float* lse_out = d->lse != nullptr ? d->lse[a] : nullptr;
  return cp_attn_merge(d->n_q[a] * d->n_q_heads, d->head_dim, d->n_ranks, outs, lses,
                       d->part_dtype, d->out[a], d->out_dtype, lse_out, st);
}

// The ranks' outputs lie back to back, as gathered queries do.
bool outputs_are_gathered(const cp_ring_desc* d) {
  const size_t out_row = (size_t)d->n_q_heads * d->head_dim * elem_size(d->out_dtype);
  bool one = true;
  for (int a = 1; a < d->n_ranks && one; ++a) {
    one = (char*)d->out[a] == (char*)d->out[a - 1] + d->n_q[a - 1] * out_row;
    if (d->lse != nullptr)
      one = one && d->lse[a] != nullptr && d->lse[0] != nullptr &&
            d->lse[a] == d->lse[a - 1] + d->n_q[a - 1] * d->n_q_heads;
  }
  return one;
}

// The All2All with gathered queries: source rank a merges slot k * n + a of every holder k. With
// the outputs back to back the N merges are one launch over the holders' whole blocks.
int ring_merge_gathered(const cp_ring_desc* d, const RingSlots& slots, hipStream_t st) {
  const int n = d->n_ranks;
  int rc = CP_OK;
  if (!outputs_are_gathered(d)) {
    for (int a = 0; a < n && rc == CP_OK; ++a) rc = ring_merge(d, slots, a, st);
    return rc;
  }
  const void* outs[CP_MAX_PARTS];
  const float* lses[CP_MAX_PARTS];
  for (int k = 0; k < n; ++k) {
    outs[k] = slots.out(slot_of(d, 0, k));
    lses[k] = slots.lse(slot_of(d, 0, k));
  }
  return cp_attn_merge((int64_t)n * d->n_q[0] * d->n_q_heads, d->head_dim, n, outs, lses,
                       d->part_dtype, d->out[0], d->out_dtype,
                       d->lse != nullptr ? d->lse[0] : nullptr, st);
}

// The whole ring as one attention launch (plus the tile-bound pre-pass and, where the KV axis is
// split or the partials are kept, a merge launch over all ranks).
int ring_one_launch(const cp_ring_desc* d, hipStream_t st) {
  const int n = d->n_ranks;
  AttnTable t = {};
  t.n_ranks = t.n_shards = n;
  const RingSlots slots = make_slots(d);
  for (int r = 0; r < n; ++r) {
    t.q[r] = d->q[r]; t.q_pos[r] = d->q_pos[r];
    t.out[r] = d->keep_partials ? slots.out(slot_of(d, r, 0)) : d->out[r];
    t.lse[r] = d->keep_partials ? slots.lse(slot_of(d, r, 0))
                                : d->lse != nullptr ? d->lse[r] : nullptr;
    t.k[r] = d->k[r]; t.v[r] = d->v[r]; t.kv_pos[r] = d->kv_pos[r];
    t.n_kv[r] = (int32_t)d->n_kv[r];
    t.tok_begin[r + 1] = t.tok_begin[r] + (int32_t)d->n_q[r];
    t.blk_begin[r + 1] = t.blk_begin[r] + kv_blocks(d->n_kv[r]);
    if (!aligned16(d->q[r]) || !aligned16(d->k[r]) || !aligned16(d->v[r]) ||
        (d->n_q[r] > 0 && !aligned16(d->out[r])))
      return CP_ERR_ALIGN;
  }
  const AttnShape s = ring_attn_shape(d);
  if (s.total_q == 0) return CP_OK;
  // (slots of the partials lie slot_step apart along the KV shards)
  const int64_t slot_step = d->gathered_q ? n : 1;
  const int64_t slot_lse = slots.messages ? (int64_t)(slots.out_stride / sizeof(float))
                                          : (int64_t)slots.lse_slot_elems;
  const AttnOut o = {d->keep_partials ? d->part_dtype : d->out_dtype,
                     slot_step * (int64_t)slots.out_stride, slot_step * slot_lse};
  OverShards over = {};
  over.dtype = d->out_dtype;
  for (int a = 0; a < n; ++a) {
    over.out[a] = d->out[a];
    over.lse[a] = d->lse != nullptr ? d->lse[a] : nullptr;
  }
  int rc;
  if (d->dtype == CP_FP32) {
    rc = launch_attn_fp32(s, t, o, st);
  } else {
    char* ws = (char*)d->workspace;
    size_t left = d->workspace_bytes;
    const int32_t* q_lo = nullptr;
    if (ring_is_packed(d, false)) {
      int64_t keys = 0;
      for (int r = 0; r < n; ++r) keys += d->n_kv[r];
      rc = launch_varseq_encode(d->batch, keys, t, d->cu_seqlens_q, d->cu_seqlens_kv, ws, &q_lo,
                                st);
      if (rc != CP_OK) return rc;
      ws += ring_varseq_bytes(d);
      left -= ring_varseq_bytes(d);
    }
    if (d->fused_merge == 2 && d->arrived != nullptr) {
      // every shard behind its arrival flag, walked in ring order
      return launch_attn_mfma_ring(s, t, d->arrived, d->ring_error, d->spin_limit, d->out_dtype,
                                   ws, left, st);
    }
    rc = launch_attn_mfma(s, t, o, q_lo, ws, left, nullptr, d->keep_partials ? &over : nullptr, st);
  }
  if (rc != CP_OK || !d->keep_partials || over.done) return rc;
  MergeTable m = {};
  m.n_ranks = n; m.n_parts = n; m.n_groups = 1;
  m.part_bytes = o.shard_out_bytes;
  m.part_lse_elems = o.shard_lse_elems;
  for (int a = 0; a < n; ++a) {
    m.part[a] = t.out[a]; m.part_lse[a] = t.lse[a];
    m.out[a] = d->out[a]; m.lse[a] = d->lse != nullptr ? d->lse[a] : nullptr;
    m.row_begin[a + 1] = m.row_begin[a] + d->n_q[a] * d->n_q_heads;
  }
  m.rows = m.row_begin[n];
  return launch_merge_table(m, d->head_dim, d->part_dtype, d->out_dtype, st);
}

// What the steps of a ring that is not one launch share.
struct RingSteps {
  bool bounds = false;                  // of every shard, made once
  size_t bounds_off[CP_MAX_PARTS] = {};
  char* call_ws = nullptr;
  size_t call_ws_bytes = 0;
  hipStream_t aux = nullptr;            // the calls of a rank alternate between two streams
  hipEvent_t fork = nullptr, join = nullptr;
  ~RingSteps() {
    if (fork != nullptr) (void)hipEventDestroy(fork);
    if (join != nullptr) (void)hipEventDestroy(join);
  }
};

int prepare_steps(const cp_ring_desc* d, hipStream_t st, RingSteps& w) {
  w.bounds = ring_shares_bounds(d, false);
  const size_t head = w.bounds ? kv_bounds_ring_bytes(d->n_ranks, d->n_kv) : 0;
  w.call_ws = (char*)d->workspace + head;
  w.call_ws_bytes = d->workspace_bytes - head;   // (check_ring_workspace)
  if (!w.bounds) return CP_OK;
  const int rc = launch_kv_bounds_ring(d->n_ranks, d->kv_pos, d->n_kv, d->workspace, w.bounds_off,
                                       st);
  if (rc != CP_OK || d->aux_stream == nullptr || d->fused_merge || d->gathered_q) return rc;
  // Two streams only if no call writes partials to the workspace that all of them share.
  for (int a = 0; a < d->n_ranks; ++a)
    for (int b = 0; b < d->n_ranks; ++b)
      if (d->n_q[a] > 0 && attn_mfma_has_partials(step_shape(ring_shape(d, a, b, false))))
        return CP_OK;
  if (hipEventCreateWithFlags(&w.fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&w.join, hipEventDisableTiming) != hipSuccess)
    return CP_ERR_LAUNCH;
  w.aux = (hipStream_t)d->aux_stream;
  return CP_OK;
}

// Queries of rank a (s.total_q of them) against the KV of rank b; `acc`: merged into a running
// result.
int step_call(const cp_ring_desc* d, const RingSteps& w, const cp_shape& s, int a, int b, void* out,
              float* lse, int32_t dtype, const PrefillAccumulate* acc, hipStream_t st) {
  const bool packed = ring_is_packed(d, false);
  if (!w.bounds)   // (fused_merge is refused there)
    return cp_attn_partial(&s, d->q[a], d->k[b], d->v[b], d->q_pos[a], d->kv_pos[b],
                           packed ? d->cu_seqlens_q[a] : nullptr,
                           packed ? d->cu_seqlens_kv[b] : nullptr, out, lse, dtype, w.call_ws,
                           w.call_ws_bytes, st);
  if (!aligned16(d->q[a]) || !aligned16(d->k[b]) || !aligned16(d->v[b])) return CP_ERR_ALIGN;
  if (s.total_q == 0) return CP_OK;
  if (s.total_q > INT32_MAX) return CP_ERR_SHAPE;
  const AttnShape as = step_shape(s);
  const AttnTable t = single_table(s, d->q[a], d->k[b], d->v[b], d->q_pos[a], d->kv_pos[b], out,
                                   lse);
  const char* const bounds = (const char*)d->workspace + w.bounds_off[b];
  if (acc != nullptr)
    return launch_attn_mfma_accumulate(as, t, *acc, w.call_ws, w.call_ws_bytes, bounds, st);
  return launch_attn_mfma(as, t, AttnOut{dtype, 0, 0}, nullptr, w.call_ws, w.call_ws_bytes, bounds,
                          nullptr, st);
}

// fused_merge of a rank of such a ring, which has one slot for its partials: step 0 writes a
// running (O, LSE) there, the following steps merge into it in their epilogues and the last one
// writes the rank's output.
template <typename KvOf>
int ring_rank_fused(const cp_ring_desc* d, const RingSteps& w, const RingSlots& slots, int a,
                    hipStream_t st, KvOf kv_of_step) {
  float* const acc_out = (float*)slots.out(0);
  float* const acc_lse = slots.lse(0);
  for (int j = 0; j < d->n_ranks; ++j) {
    const int b = kv_of_step(a, j);
    const bool last = j == d->n_ranks - 1;
    const PrefillAccumulate acc = {acc_out, acc_lse, last ? d->out[a] : nullptr,
                                   last && d->lse != nullptr ? d->lse[a] : nullptr, d->out_dtype};
    if (last && d->n_q[a] > 0 && !aligned16(d->out[a])) return CP_ERR_ALIGN;
    const int rc = step_call(d, w, ring_shape(d, a, b, false), a, b, acc_out, acc_lse, CP_FP32,
                             j == 0 ? nullptr : &acc, st);
    if (rc != CP_OK) return rc;
  }
  return CP_OK;
}

// N x N partial-attention calls and a merge per rank, for the rings that are not one launch.
// `kv_of_step(k, j)`: the KV rank of step j of rank k's queries.
template <typename KvOf>
int ring_steps(const cp_ring_desc* d, hipStream_t st, KvOf kv_of_step) {
  const RingSlots slots = make_slots(d);
  const int n = d->n_ranks;
  RingSteps w;
  int rc = prepare_steps(d, st, w);
  if (rc != CP_OK) return rc;
  if (d->gathered_q) {   // one call per KV holder, whose slots are one block
    for (int b = 0; b < n; ++b) {
      const int64_t slot = slot_of(d, 0, b);
      rc = step_call(d, w, gathered_shape(d, b, false), 0, b, slots.out(slot), slots.lse(slot),
                     d->part_dtype, nullptr, st);
      if (rc != CP_OK) return rc;
    }
    return ring_merge_gathered(d, slots, st);
  }
  for (int a = 0; a < n; ++a) {
    if (d->fused_merge && n > 1) {
      rc = ring_rank_fused(d, w, slots, a, st, kv_of_step);
      if (rc != CP_OK) return rc;
      continue;
    }
    // (the aux stream starts behind the previous rank's merge, which reads the slots)
    if (w.aux != nullptr && (hipEventRecord(w.fork, st) != hipSuccess ||
                             hipStreamWaitEvent(w.aux, w.fork, 0) != hipSuccess))
      return CP_ERR_LAUNCH;
    for (int j = 0; j < n && rc == CP_OK; ++j) {
      const int b = kv_of_step(a, j);
      const int64_t slot = slot_of(d, a, b);
      rc = step_call(d, w, ring_shape(d, a, b, false), a, b, slots.out(slot), slots.lse(slot),
                     d->part_dtype, nullptr, w.aux != nullptr && (j & 1) ? w.aux : st);
    }
    if (w.aux != nullptr && (hipEventRecord(w.join, w.aux) != hipSuccess ||
                             hipStreamWaitEvent(st, w.join, 0) != hipSuccess))
      return CP_ERR_LAUNCH;
    if (rc == CP_OK) rc = ring_merge(d, slots, a, st);
    if (rc != CP_OK) return rc;
  }
  return CP_OK;
}

// Prefill in either ring order: the same N x N partials and the same merge.
template <typename KvOf>
int ring_prefill(const cp_ring_desc* d, hipStream_t st, KvOf kv_of_step) {
  int rc = check_ring_workspace(d, false);
  if (rc != CP_OK) return rc;
  if (d->fused_merge) {
    rc = check_fused(d);
    if (rc != CP_OK) return rc;
  }
  return ring_is_one_launch(d) ? ring_one_launch(d, st) : ring_steps(d, st, kv_of_step);
}

}  // namespace

extern "C" {

size_t cp_ring_message_bytes(const cp_ring_desc* d) {
  if (d == nullptr || d->n_q == nullptr || d->n_ranks < 1 || d->n_ranks > CP_MAX_PARTS) return 0;
  if (d->part_dtype != CP_BF16 && d->part_dtype != CP_FP32) return 0;
  if (d->n_q_heads < 1 || d->head_dim < 1) return 0;
  for (int i = 0; i < d->n_ranks; ++i)
    if (d->n_q[i] < 0) return 0;
  const RingSlots r = make_slots(d);
  return ring_message_bytes(r.out_slot_bytes, r.lse_slot_elems);
}

int cp_ring_passkv(const cp_ring_desc* d, void* stream) {
  const int rc = check_ring(d, false);
  if (rc != CP_OK) return rc;
  if (d->gathered_q) return CP_ERR_UNSUPPORTED;  // pass-Q only
  const int n = d->n_ranks;
  // Algorithm 2: at step j rank k holds the KV of rank (k - j) mod N.
  return ring_prefill(d, (hipStream_t)stream, [n](int k, int j) { return ((k - j) % n + n) % n; });
}

// gathered_q: the query shards of all source ranks lie back to back in one buffer (an
// all-gather of the small Q instead of passing it round), so a KV holder answers all N ring
// steps of Algorithms 3 / 4 with one call over the gathered queries. Its output block, N slots
// of equal size, is the holder's All2All send buffer in destination order.
static bool queries_are_gathered(const cp_ring_desc* d, bool decode) {
  const size_t row = (size_t)d->n_q_heads * d->head_dim * elem_size(d->dtype);
  for (int s = 0; s < d->n_ranks; ++s) {
    if (d->n_q[s] != d->n_q[0] || d->n_q[s] == 0) return false;
    if (s == 0) continue;
    if ((const char*)d->q[s] != (const char*)d->q[s - 1] + d->n_q[s - 1] * row) return false;
    if (d->q_pos[s] != d->q_pos[s - 1] + d->n_q[s - 1]) return false;
    if (decode && d->bid[s] != d->bid[s - 1] + d->n_q[s - 1]) return false;
  }
  return true;
}

// Algorithm 4 with gathered queries: one decode call per KV holder.
static int ring_decode_gathered(const cp_ring_desc* d, hipStream_t st) {
  const RingSlots slots = make_slots(d);
  const int n = d->n_ranks;
  int rc = CP_OK;
  cp_shape shapes[CP_MAX_PARTS];
  bool flat = true;
  for (int k = 0; k < n; ++k) {
    shapes[k] = gathered_shape(d, k, true);
    flat = flat && decode_flat_applies(shapes[k]);
    if (!aligned16(d->k[k]) || !aligned16(d->v[k])) return CP_ERR_ALIGN;
  }
  if (!aligned16(d->q[0])) return CP_ERR_ALIGN;
  if (flat) {
    // every holder's split-KV partials in one launch, one merge over splits x holders
    const int64_t all = (int64_t)n * d->n_q[0];
    const bool one = outputs_are_gathered(d);
    return launch_decode_flat(n, shapes, resolve_scale(d->softmax_scale, d->head_dim), d->q[0],
                              d->k, d->v, d->q_pos[0], d->kv_pos, d->cu_seqlens_kv, d->bid[0],
                              one ? 1 : n, one ? &all : d->n_q, d->out, d->out_dtype, d->lse,
                              d->workspace, d->workspace_bytes, st);
  }
  for (int k = 0; k < n; ++k) {
    const int64_t slot = slot_of(d, 0, k);
    rc = cp_attn_decode(&shapes[k], d->q[0], d->k[k], d->v[k], d->q_pos[0], d->kv_pos[k],
                        d->cu_seqlens_kv[k], d->bid[0], slots.out(slot), slots.lse(slot),
                        d->part_dtype, d->workspace, d->workspace_bytes, st);
    if (rc != CP_OK) return rc;
  }
  return ring_merge_gathered(d, slots, st);
}

// Algorithm 4: N x N decode calls, grouped by source rank, and a merge per source.
static int ring_decode(const cp_ring_desc* d, hipStream_t st) {
  int rc = check_ring_workspace(d, true);
  if (rc != CP_OK) return rc;
  if (d->gathered_q) return ring_decode_gathered(d, st);
  const RingSlots slots = make_slots(d);
  const int n = d->n_ranks;
  for (int s = 0; s < n && rc == CP_OK; ++s) {
    for (int j = 0; j < n && rc == CP_OK; ++j) {
      const int k = (s + j) % n;
      const cp_shape sh = ring_shape(d, s, k, true);
      const int64_t slot = slot_of(d, s, k);
      rc = cp_attn_decode(&sh, d->q[s], d->k[k], d->v[k], d->q_pos[s], d->kv_pos[k],
                          d->cu_seqlens_kv[k], d->bid[s], slots.out(slot), slots.lse(slot),
                          d->part_dtype, d->workspace, d->workspace_bytes, st);
    }
    if (rc == CP_OK) rc = ring_merge(d, slots, s, st);
  }
  return rc;
}

int cp_ring_passq(const cp_ring_desc* d, void* stream) {
  const int rc = check_ring(d, false);
  if (rc != CP_OK) return rc;
  if (d->fused_merge == 2) return CP_ERR_UNSUPPORTED;  // pass-KV only: the queries stay put
  if (d->gathered_q && !queries_are_gathered(d, false)) return CP_ERR_UNSUPPORTED;
  const int n = d->n_ranks;
  // Algorithm 3: at step j rank k answers the queries of rank (k - j) mod N, so rank s's
  // queries meet the KV of rank (s + j) mod N; writing the result to the slot of (s, k) is the
  // permute + All2All.
  return ring_prefill(d, (hipStream_t)stream, [n](int s, int j) { return (s + j) % n; });
}

int cp_ring_passq_decode(const cp_ring_desc* d, void* stream) {
  const int rc = check_ring(d, true);
  if (rc != CP_OK) return rc;
  if (d->fused_merge == 2) return CP_ERR_UNSUPPORTED;
  if (d->gathered_q && !queries_are_gathered(d, true)) return CP_ERR_UNSUPPORTED;
  return ring_decode(d, (hipStream_t)stream);
}

int cp_ring_prefill(const cp_ring_desc* d, const cp_select_params* params, int64_t p_cached,
                    int32_t rule, int32_t* order_out, void* stream) {
  if (d == nullptr || params == nullptr) return CP_ERR_NULL;
  if (d->n_ranks < 1 || d->n_ranks > CP_MAX_PARTS || d->n_q == nullptr) return CP_ERR_SHAPE;
  if (params->n_ranks != d->n_ranks) return CP_ERR_SHAPE;
  int64_t t_new = 0;
  for (int r = 0; r < d->n_ranks; ++r) {
    if (d->n_q[r] < 0) return CP_ERR_SHAPE;
    t_new += d->n_q[r];
  }
  int32_t order = CP_ORDER_PASS_KV;
  const int rc = cp_select_order(params, t_new, p_cached, rule, &order);
  if (rc != CP_OK) return rc;
  if (order_out != nullptr) *order_out = order;
  return order == CP_ORDER_PASS_Q ? cp_ring_passq(d, stream) : cp_ring_passkv(d, stream);
}

}  // extern "C"
