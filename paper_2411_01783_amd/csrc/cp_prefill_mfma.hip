// bf16 MFMA attention for gfx950, head_dim 128 and 64: host side (launch plan, tile-bound
// pre-pass) and the definitions shared with the kernel in cp_prefill_pipe.h.
//
// Computes O, LSE = Attn(Q, KV) (Algorithms 2 and 3; O and LSE as in Appendix B) for the
// queries of one or more ranks against one or more KV shards, per KV head and its group of
// G = N_H / N_KV query heads.
//
// Work decomposition
//   - The (token, head-in-group) pairs of a KV head form R = total_q * G rows, token-major, the
//     ranks' tokens back to back. The causal mask depends on the token only, so all G heads of
//     a token share mask and K/V tile: GQA turns into a taller M dimension.
//   - A workgroup of 8 wavefronts owns 256 consecutive rows, 32 per wavefront, and walks the
//     128-key tiles of the KV shards, brought straight into LDS (double buffered) and consumed
//     in blocks of 32 keys by a three-stage software pipeline per wavefront (see
//     cp_prefill_pipe.h).
//   - Scores are produced transposed, S^T = K Q^T with v_mfma_f32_32x32x16_bf16:
//     a lane then holds 16 keys of ONE query per 32-key block, so the softmax
//     row statistics are per-lane scalars (one cross-lane exchange with lane^32)
//     and the exponentiated block is already in the B-operand layout of the
//     second product O^T += V^T P^T. No register shuffle between the products.
//   - Tile skipping (load-balanced sharding leaves half of every off-diagonal
//     step fully masked): a pre-pass records min/max kv_pos of every KV tile;
//     each workgroup compacts the tiles any of its queries can see into a list
//     in LDS and walks only those; only tiles that straddle a query position
//     pay for the mask.
//   - A ring whose ranks all live here is one launch: every rank's rows against the tiles of all
//     shards, so that Equation 4 over the ring steps happens inside the online softmax. (A
//     launch per ring step costs 12 to 17 us at small query shards whatever its work: 256
//     launches and 256 split merges for 16 ranks, 6.06 ms at 1024 new tokens on 131072 cached
//     ones, where the arithmetic is 0.85 ms at the rate of a large matrix product.)
//   - Where the row blocks alone leave compute units idle the KV axis is split over grid.z,
//     every part taking an equal share of the tiles its rows can see; the parts' fp32 results
//     go to the workspace and are combined with Eq. 4.
//   - The epilogue transposes the accumulators through LDS so that every output
//     row leaves as one contiguous 4 D byte (fp32) or 2 D byte (bf16) run.
//   - The same body also merges into a running (O, LSE) in its epilogue (ACC), and walks the
//     shards of one rank's ring steps in ring order, each behind an arrival flag (RING,
//     prefill_ring_walk_kernel).
#include "cp_common.h"
#include "cp_table.h"

namespace cp {
namespace {

constexpr int BM = 256;         // rows per workgroup
constexpr int TILE = kAttnTile; // keys per LDS tile
constexpr int NWAVE = 8;        // wavefronts per workgroup
constexpr int NTHREADS = NWAVE * 64;
constexpr int POS_BYTES = TILE * 4;
constexpr int MAX_LIVE = 512;   // visible-tile list entries per chunk (8 wavefronts x 64 tiles)
constexpr float kRescaleSlack = 8.f;               // log2 units
constexpr float kOverflowSum = 1099511627776.f;    // 2^40: a block sum beyond it is redone
constexpr float kDeadRowRef = 1e30f;               // reference of a row that sees no key

struct Params {
  AttnTable t;            // queries and outputs per rank, KV per shard
  const int2* bounds;     // [n_tiles] (min, max) of kv_pos per tile, shard after shard
  const int32_t* q_lo;    // BAND only: smallest visible key position per query token
  float* part_out;        // SPLIT: [grid.z][rows_all_heads][D] fp32
  float* part_lse;        // SPLIT: [grid.z][rows_all_heads]
  float* acc;             // ACC: running O, fp32 [rows_all_heads][D] (running LSE: t.lse[0])
  void* final_out;        // ACC: where the merged O goes on the last step (else NULL)
  float* final_lse;       // ACC: optional copy of the merged LSE
  const int32_t* arrived; // RING: or NULL: [n_shards], nonzero once step j's shard may be read
  int32_t* ring_error;    // RING: bit j is set when the wait of step j gave up
  int64_t rows;           // R = total_q * G
  int64_t rows_all_heads; // total_q * n_q_heads
  int64_t out_shard_stride;  // per_shard, not SPLIT: bytes between the outputs of two shards
  int64_t lse_shard_stride;  // and elements between their LSE
  int32_t group;          // G
  int32_t n_kv_heads;
  int32_t n_tiles;        // of all shards
  int32_t n_sub;          // parts of the KV axis (of every shard's, if per_shard)
  int32_t per_shard;      // the shards' results are kept apart
  int32_t ring_start;     // RING: shard of step 0
  int32_t spin_limit;     // RING: polls per shard before giving up
  float scale_log2;       // softmax scale * log2(e)
};

// (min, max) of kv_pos per tile, for the shards of a whole call in one launch (a launch per
// shard costs more than the work: a shard of 8K keys is 64 tiles). One wavefront per tile.
__global__ __launch_bounds__(256) void kv_tile_bounds_kernel(const AttnTable t, int32_t n_tiles,
                                                              int2* __restrict__ bounds) {
  const int gt = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (gt >= n_tiles) return;
  int j = 0;
  for (int i = 1; i < t.n_shards; ++i) j += gt >= t.tile_begin[i];  // (wave-uniform)
  const int tile = gt - t.tile_begin[j];
  const int32_t* __restrict__ kv_pos = t.kv_pos[j];
  const int32_t total_kv = t.n_kv[j];
  const int lane = threadIdx.x & 63;
  int lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
  for (int h = 0; h < TILE / 64; ++h) {
    const int idx = tile * TILE + h * 64 + lane;
    if (idx < total_kv) {
      const int32_t x = kv_pos[idx];
      lo = min(lo, x);
      hi = max(hi, x);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, 64));
    hi = max(hi, __shfl_xor(hi, o, 64));
  }
  if (lane == 0) bounds[gt] = make_int2(lo, hi);
}

__device__ __forceinline__ floatx16_t mfma32(bf16x8_t a, bf16x8_t b, floatx16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Value of lane ^ 32 (v_permlane32_swap: no LDS round trip).
__device__ __forceinline__ float xor32(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

#include "cp_prefill_pipe.h"

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// Split count of the KV axis for `wgs` workgroups of 256 rows over `tiles` tiles.
// Splitting starts below 256 workgroups, one per CU. Cost of a split count, in units of one
// tile step of a workgroup: the workgroups run in rounds of 256, each round walks its tiles plus
// about three tile steps of start-up and epilogue, and every split adds one fp32 partial of
// the `rows` output rows to write and to merge. (129 .. 255 workgroups mostly stay whole: two
// splits would need a second round.)
int choose_splits(int64_t wgs, int tiles, double rows, int head_dim, int max_splits) {
  if (wgs <= 0 || wgs >= 256 || tiles < 2) return 1;
  max_splits = std::min(max_splits, tiles);
  const double partial_cost = rows * head_dim * (4.8e-5 / 128);
  int splits = 1;
  double best = 0.0;
  for (int c = 1; c <= max_splits; ++c) {
    const int tps = (tiles + c - 1) / c;
    const int64_t rounds = (wgs * c + 255) / 256;
    const double cost = (double)rounds * (tps + 3) + partial_cost * c;
    if (c == 1 || cost < best) {
      best = cost;
      splits = c;
    }
  }
  return splits;
}

struct Plan {
  int n_row_blocks, n_sub, n_z;   // n_z = grid.z
  bool split;                     // fp32 partials in the workspace
  size_t bounds_bytes, part_out_bytes, part_lse_bytes;
  size_t total() const { return bounds_bytes + part_out_bytes + part_lse_bytes; }
};

Plan make_plan(const AttnShape& s) {
  Plan pl;
  const int group = s.n_q_heads / s.n_kv_heads;
  pl.n_row_blocks = (int)((s.total_q * group + BM - 1) / BM);
  const int64_t wgs = (int64_t)pl.n_row_blocks * s.n_kv_heads;
  const double rows = (double)s.total_q * s.n_q_heads;
  if (s.per_shard) {
    // one part per shard at least: the parts of a shard are chosen for the average shard
    const int avg = (s.n_tiles + s.n_shards - 1) / s.n_shards;
    pl.n_sub = choose_splits(wgs * s.n_shards, avg, rows * s.n_shards, s.head_dim,
                             16);
    pl.n_z = s.n_shards * pl.n_sub;
    pl.split = pl.n_sub > 1;
  } else {
    pl.n_sub = choose_splits(wgs, s.n_tiles, rows, s.head_dim, CP_MAX_PARTS);
    pl.n_z = pl.n_sub;
    pl.split = pl.n_sub > 1;
  }
  pl.bounds_bytes = round256((size_t)std::max(s.n_tiles, 1) * sizeof(int2));
  const size_t rows_all = (size_t)s.total_q * s.n_q_heads;
  pl.part_out_bytes = pl.split ? round256((size_t)pl.n_z * rows_all * s.head_dim * 4) : 0;
  pl.part_lse_bytes = pl.split ? round256((size_t)pl.n_z * rows_all * 4) : 0;
  return pl;
}

template <int D>
using Kern = void (*)(Params);

template <int D>
Kern<D> pick_kernel(bool split, bool band, bool bf16_out) {
  if constexpr (D == 128) {
    if (band)
      return split ? prefill_mfma_kernel<128, float, true, true>
             : bf16_out ? prefill_mfma_kernel<128, bf16_t, true, false>
                        : prefill_mfma_kernel<128, float, true, false>;
  }
  return split ? prefill_mfma_kernel<D, float, false, true>
         : bf16_out ? prefill_mfma_kernel<D, bf16_t, false, false>
                    : prefill_mfma_kernel<D, float, false, false>;
}

int launch_body(void (*kern)(Params), int smem, const dim3& grid, const Params& p,
                hipStream_t stream) {
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem) !=
      hipSuccess)
    return CP_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, grid, dim3(NTHREADS), smem, stream, p);
  return check_launch();
}

int check_rows(const AttnShape& s) {
  if (s.n_kv_heads > 65535) return CP_ERR_SHAPE;
  if (s.total_q * (s.n_q_heads / s.n_kv_heads) > 0x7fffffffLL) return CP_ERR_SHAPE;  // 31-bit rows
  return CP_OK;
}

void fill_params(const AttnShape& s, const AttnTable& t, const void* bounds, Params& p) {
  p.t = t;
  p.bounds = (const int2*)bounds;
  p.group = s.n_q_heads / s.n_kv_heads;
  p.rows = s.total_q * p.group;
  p.rows_all_heads = s.total_q * s.n_q_heads;
  p.n_kv_heads = s.n_kv_heads;
  p.n_tiles = s.n_tiles;
  p.n_sub = 1;
  p.scale_log2 = s.scale * kLog2e;
}

}  // namespace

bool attn_mfma_applies(int dtype, int head_dim, int n_q_heads, int n_kv_heads) {
  return dtype == CP_BF16 && (head_dim == 128 || head_dim == 64) &&
         n_q_heads / n_kv_heads <= 64;
}

size_t attn_mfma_workspace_bytes(const AttnShape& s) { return make_plan(s).total(); }

bool attn_mfma_merging_applies(const AttnShape& s) {
  const int64_t rows = s.total_q * (s.n_q_heads / s.n_kv_heads);
  const int64_t wgs = (rows + BM - 1) / BM * s.n_kv_heads;
  if (s.head_dim != 128) return false;
  if (wgs >= 128 || wgs == 0) return true;
  return choose_splits(wgs, s.n_tiles, (double)s.total_q * s.n_q_heads, s.head_dim,
                       CP_MAX_PARTS) == 1;
}

int launch_kv_tile_bounds(const AttnTable& t, int n_tiles, void* bounds_out, hipStream_t stream) {
  if (n_tiles == 0) return CP_OK;
  hipLaunchKernelGGL(kv_tile_bounds_kernel, dim3((n_tiles + 3) / 4), dim3(256), 0, stream, t,
                     n_tiles, (int2*)bounds_out);
  return check_launch();
}

int launch_attn_mfma(const AttnShape& s, const AttnTable& t, const AttnOut& o,
                     const int32_t* q_lo, const void* tile_bounds, void* workspace,
                     size_t workspace_bytes, hipStream_t stream) {
  const Plan pl = make_plan(s);
  if (workspace_bytes < pl.total()) return CP_ERR_WORKSPACE;
  if (pl.n_row_blocks == 0) return CP_OK;
  const int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  char* ws = (char*)workspace;
  if (tile_bounds == nullptr && launch_kv_tile_bounds(t, s.n_tiles, ws, stream) != CP_OK)
    return CP_ERR_LAUNCH;
  Params p = {};
  fill_params(s, t, tile_bounds != nullptr ? tile_bounds : ws, p);
  p.q_lo = q_lo;
  p.n_sub = pl.n_sub;
  p.per_shard = s.per_shard ? 1 : 0;
  p.part_out = (float*)(ws + pl.bounds_bytes);
  p.part_lse = (float*)(ws + pl.bounds_bytes + pl.part_out_bytes);
  p.out_shard_stride = o.shard_out_bytes;
  p.lse_shard_stride = o.shard_lse_elems;
  const bool bf16_out = o.dtype == CP_BF16, band = q_lo != nullptr;
  if (band && s.head_dim != 128) return CP_ERR_UNSUPPORTED;
  const dim3 grid(pl.n_row_blocks, s.n_kv_heads, pl.n_z);
  const int rl = s.head_dim == 128
                     ? launch_body(pick_kernel<128>(pl.split, band, bf16_out), Geo<128>::SMEM, grid,
                                   p, stream)
                     : launch_body(pick_kernel<64>(pl.split, band, bf16_out), Geo<64>::SMEM, grid,
                                   p, stream);
  if (rl != CP_OK || !pl.split) return rl;

  // Equation 4 over the parts: of the whole KV axis, or of every shard into the shard's output
  MergeTable m = {};
  m.n_ranks = t.n_ranks;
  m.n_parts = pl.n_sub;
  m.part_bytes = p.rows_all_heads * s.head_dim * 4;
  m.part_lse_elems = p.rows_all_heads;
  m.n_groups = s.per_shard ? s.n_shards : 1;
  m.group_out_bytes = o.shard_out_bytes;
  m.group_lse_elems = o.shard_lse_elems;
  for (int a = 0; a < t.n_ranks; ++a) {
    const int64_t row0 = (int64_t)t.tok_begin[a] * s.n_q_heads;
    m.row_begin[a] = row0;
    m.part[a] = p.part_out + row0 * s.head_dim;
    m.part_lse[a] = p.part_lse + row0;
    m.out[a] = t.out[a];
    m.lse[a] = t.lse[a];
  }
  m.row_begin[t.n_ranks] = p.rows_all_heads;
  return launch_merge_table(m, s.head_dim, CP_FP32, o.dtype, stream);
}

int launch_attn_mfma_accumulate(const AttnShape& s, const AttnTable& t,
                                const PrefillAccumulate& acc, void* workspace,
                                size_t workspace_bytes, hipStream_t stream) {
  if (!attn_mfma_merging_applies(s)) return CP_ERR_UNSUPPORTED;
  const size_t bounds_bytes = round256((size_t)std::max(s.n_tiles, 1) * sizeof(int2));
  if (workspace_bytes < bounds_bytes) return CP_ERR_WORKSPACE;
  const int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  if (launch_kv_tile_bounds(t, s.n_tiles, workspace, stream) != CP_OK) return CP_ERR_LAUNCH;
  Params p = {};
  fill_params(s, t, workspace, p);
  p.acc = acc.out;
  p.final_out = acc.final_out;
  p.final_lse = acc.final_lse;
  const int64_t blocks = (p.rows + BM - 1) / BM;
  const dim3 grid((unsigned)blocks, s.n_kv_heads, 1);
  return launch_body(acc.final_out != nullptr && acc.final_dtype == CP_BF16
                         ? prefill_mfma_kernel<128, bf16_t, false, false, true>
                         : prefill_mfma_kernel<128, float, false, false, true>,
                     Geo<128>::SMEM, grid, p, stream);
}

int launch_attn_mfma_ring(const AttnShape& s, const AttnTable& t, int ring_start,
                          const int32_t* arrived, int32_t* error, int32_t spin_limit,
                          int32_t out_dtype, const void* tile_bounds, hipStream_t stream) {
  if (t.n_ranks != 1 || ring_start < 0 || ring_start >= t.n_shards) return CP_ERR_SHAPE;
  if (arrived != nullptr && (error == nullptr || spin_limit < 1)) return CP_ERR_SHAPE;
  const int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  Params p = {};
  fill_params(s, t, tile_bounds, p);
  p.arrived = arrived; p.ring_error = error; p.spin_limit = spin_limit;
  p.ring_start = ring_start;
  const int64_t blocks = (p.rows + BM - 1) / BM;
  if (blocks == 0) return CP_OK;
  const dim3 grid((unsigned)blocks, s.n_kv_heads, 1);
  return launch_body(out_dtype == CP_BF16 ? prefill_ring_walk_kernel<bf16_t>
                                          : prefill_ring_walk_kernel<float>,
                     Geo<128>::SMEM, grid, p, stream);
}

}  // namespace cp
