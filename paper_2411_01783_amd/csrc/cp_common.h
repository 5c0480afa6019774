// Internal declarations shared by the HIP translation units of libcp_attn.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "cp_attn.h"

namespace cp {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float to_float(float x) { return x; }
__device__ __forceinline__ float to_float(bf16_t x) { return static_cast<float>(x); }

template <typename T>
__device__ __forceinline__ T from_float(float x);
template <>
__device__ __forceinline__ float from_float<float>(float x) {
  return x;
}
template <>
__device__ __forceinline__ bf16_t from_float<bf16_t>(float x) {
  return static_cast<bf16_t>(x);
}

// Workgroup barrier that orders LDS traffic only: global loads issued before it stay in flight
// across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Asks for all lines of the kernel's one argument (a struct P) at once, and returns something that has
// to be used, once the first loads are waited for anyway. As scalar loads, a few lines at a time, they are
// one cold memory latency after the other: 128 queries of 16 heads on 16 of 8192 keys 9.7 -> 6.9 us
// from the start to the first tile's requests.
template <typename P>
__device__ __forceinline__ int touch_arguments() {
  int x = 0;
  if (threadIdx.x < (sizeof(P) + 63) / 64)
    x = ((const __attribute__((address_space(4))) int*)
             __builtin_amdgcn_kernarg_segment_ptr())[threadIdx.x * 16];
  return x;
}

// ---- launchers (each returns a cp_status; enqueue on `stream` only) ----

// fp32 vector kernel: any supported dtype / head_dim, packed batches.
int launch_partial_generic(const cp_shape& s, float scale, const void* q, const void* k,
                           const void* v, const int32_t* q_pos, const int32_t* kv_pos,
                           const int32_t* cu_q, const int32_t* cu_kv, void* out, float* lse,
                           int32_t out_dtype, hipStream_t stream);

// What one attention launch works on: the queries (and outputs) of n_ranks ranks back to back,
// against n_shards KV shards, any query against any key that its position lets it see. A single
// call is one rank and one shard; a ring whose ranks all live on this GPU is one launch. Passed
// by value (kernel argument segment).
constexpr int kMaxTable = 32;
constexpr int kAttnBlock = 32;  // keys per block of the MFMA kernel
struct AttnTable {
  const void* q[kMaxTable];
  const int32_t* q_pos[kMaxTable];
  void* out[kMaxTable];
  float* lse[kMaxTable];  // entries may be NULL
  const void* k[kMaxTable];
  const void* v[kMaxTable];
  const int32_t* kv_pos[kMaxTable];
  int32_t n_kv[kMaxTable];
  int32_t tok_begin[kMaxTable + 1];   // first token of every rank, and the total
  int32_t blk_begin[kMaxTable + 1];   // first block (kAttnBlock keys) of every shard, and the total
  int32_t n_ranks, n_shards;
};
// Its sizes, from which a launch is planned (no pointers: also the workspace query's argument).
struct AttnShape {
  int32_t dtype, head_dim, n_q_heads, n_kv_heads;
  int64_t total_q;      // tokens of all ranks
  int32_t n_blocks;     // blocks of all shards
  int32_t n_shards;
  int32_t batch;        // packed sequences
  bool has_bounds;      // one rank, one shard: its position bounds are there already
  bool per_shard;       // keep the shards' results apart: one (O, LSE) per rank and shard
  float scale;
};
// Where the results go: t.out / t.lse in `dtype`; with per_shard the result against shard b is
// b * shard_out_bytes (and b * shard_lse_elems) further on.
struct AttnOut {
  int32_t dtype;
  int64_t shard_out_bytes;
  int64_t shard_lse_elems;
};
// Equation 4 over the shards' results (per_shard), rank by rank: where it goes. A launch whose own
// merge can do it along the way does, and says so in `done`.
struct OverShards {
  int32_t dtype;
  void* out[kMaxTable];
  float* lse[kMaxTable];   // entries may be NULL
  bool done;
};

// bf16 MFMA kernel, head_dim 128 and 64, groups of at most 64 heads.
// `q_lo`: packed batches (head_dim 128), smallest visible key position per token, all ranks back
// to back.
bool attn_mfma_applies(int dtype, int head_dim, int n_q_heads, int n_kv_heads);
// `bounds`: the shard's position bounds, if they are there already (kv_bounds_ring; one rank, one
// shard), else NULL.
size_t attn_mfma_workspace_bytes(const AttnShape& s);
bool attn_mfma_has_partials(const AttnShape& s);   // writes to the workspace besides the bounds
int launch_attn_mfma(const AttnShape& s, const AttnTable& t, const AttnOut& o,
                     const int32_t* q_lo, void* workspace, size_t workspace_bytes,
                     const void* bounds, OverShards* over, hipStream_t stream);   // over: or NULL

// Position bounds of n_shards shards for the calls that each take one of them, in at most two
// launches. offset[b]: where those of shard b begin in the region of kv_bounds_ring_bytes.
size_t kv_bounds_ring_bytes(int n_shards, const int64_t* n_kv);
int launch_kv_bounds_ring(int n_shards, const int32_t* const* kv_pos, const int64_t* n_kv,
                          void* region, size_t* offset, hipStream_t stream);

// "Merge into a running result": (out, lse) are read and updated (Equation 4), and if final_out
// is not NULL the merged O goes there in final_dtype instead of back to out. One rank, one
// shard, no split of the KV axis (attn_mfma_merging_applies), head_dim 128.
struct PrefillAccumulate {
  float* out;        // fp32 [total_q, n_q_heads, head_dim]
  float* lse;        // fp32 [total_q, n_q_heads]; also t.lse[0]
  void* final_out;   // or NULL
  float* final_lse;  // or NULL
  int32_t final_dtype;
};
bool attn_mfma_merging_applies(const AttnShape& s);
int launch_attn_mfma_accumulate(const AttnShape& s, const AttnTable& t,
                                const PrefillAccumulate& acc, void* workspace,
                                size_t workspace_bytes, const void* bounds, hipStream_t stream);

// One launch for all ring steps of all ranks (pass-KV), rank k walking the shards in the order
// k, k - 1, ... (mod n_ranks) with one running softmax state per row, each shard behind its
// arrival flag. arrived[k] (device): int32 per step of rank k; the kernel waits (at most
// spin_limit polls) for a nonzero value before it reads step j's shard; a wait that gives up
// sets bit j of error[k] and leaves the shard out.
size_t attn_mfma_ring_workspace_bytes(const AttnShape& s);
int launch_attn_mfma_ring(const AttnShape& s, const AttnTable& t, const int32_t* const* arrived,
                          int32_t* error, int32_t spin_limit, int32_t out_dtype, void* workspace,
                          size_t workspace_bytes, hipStream_t stream);

// fp32 MFMA kernel, head_dim 64 and 128: the same table, no workspace.
int launch_attn_fp32(const AttnShape& s, const AttnTable& t, const AttnOut& o,
                     hipStream_t stream);

// Packed batches on the MFMA path: per-sequence position ranges for the queries and keys of all
// ranks of the table (see cp_varseq.hip). cu_q[a], cu_kv[b]: boundaries of rank a's queries and
// of shard b's keys. Replaces t.q_pos and t.kv_pos by the shifted positions in the workspace;
// *q_lo receives the lower bounds of the queries.
size_t varseq_workspace_bytes(int32_t batch, int64_t total_q, int64_t total_kv);
int launch_varseq_encode(int32_t batch, int64_t total_kv, AttnTable& t, const int32_t* const* cu_q,
                         const int32_t* const* cu_kv, void* workspace, const int32_t** q_lo,
                         hipStream_t stream);

// split-KV decode, bf16, head_dim 128.
size_t decode_workspace_bytes(const cp_shape& s);
int launch_decode(const cp_shape& s, float scale, const void* q, const void* k, const void* v,
                  const int32_t* q_pos, const int32_t* kv_pos, const int32_t* cu_kv,
                  const int32_t* bid, void* out, float* lse, int32_t out_dtype, void* workspace,
                  size_t workspace_bytes, hipStream_t stream);

// Flat split-KV decode (cp_shape.flags has CP_SHAPE_UNIQUE_BID): one launch over the packed KV of
// n_holders holders (shapes[h], k[h], ...; all share the queries, their bid and the head counts)
// leaves split-KV partials in the workspace, one merge launch per run of outputs (normally one:
// n_q[a] queries into out[a], lse[a]; lse or its entries may be NULL) applies Equation 4 over
// splits and holders.
bool decode_flat_applies(const cp_shape& s);
size_t decode_flat_bytes(int n_holders, const cp_shape* shapes);
int launch_decode_flat(int n_holders, const cp_shape* shapes, float scale, const void* q,
                       const void* const* k, const void* const* v, const int32_t* q_pos,
                       const int32_t* const* kv_pos, const int32_t* const* cu_kv,
                       const int32_t* bid, int n_outs, const int64_t* n_q, void* const* out,
                       int32_t out_dtype, float* const* lse, void* workspace,
                       size_t workspace_bytes, hipStream_t stream);

// Equation 4 over n_parts partials given as device pointers.
int launch_merge(int64_t rows, int32_t head_dim, int32_t n_parts, const void* const* outs,
                 const float* const* lses, int32_t part_dtype, void* out, int32_t out_dtype,
                 float* lse_out, hipStream_t stream);

// Equation 4 over partials at a constant stride, for the rows of several ranks (row_begin: rows
// are (token, head) pairs) and, in grid.y, for n_groups runs of n_parts partials each.
struct MergeTable {
  int32_t n_ranks, n_parts, n_groups;
  int64_t rows;                      // of all ranks
  int64_t part_bytes;                // bytes from one part to the next
  int64_t part_lse_elems;
  int64_t group_out_bytes;           // bytes between the outputs of two groups
  int64_t group_lse_elems;
  const void* part[kMaxTable];       // part 0 of the rank's rows
  const float* part_lse[kMaxTable];
  void* out[kMaxTable];
  float* lse[kMaxTable];             // entries may be NULL
  int64_t row_begin[kMaxTable + 1];
};
int launch_merge_table(const MergeTable& m, int32_t head_dim, int32_t part_dtype,
                       int32_t out_dtype, hipStream_t stream);
// The same over fp32 partials, and Equation 4 over the groups in the same launch.
bool merge_over_groups_applies(const MergeTable& m);
int launch_merge_over_groups(const MergeTable& m, int32_t head_dim, int32_t out_dtype,
                             const OverShards& over, hipStream_t stream);

inline int check_launch() {
  return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_LAUNCH;
}

}  // namespace cp
