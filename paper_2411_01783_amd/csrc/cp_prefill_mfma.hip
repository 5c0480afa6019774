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
//     keys of the KV shards in tiles of four 32-key blocks, brought straight into LDS (double
//     buffered) and consumed block by block by a three-stage software pipeline per wavefront
//     (see cp_prefill_pipe.h).
//   - Scores are produced transposed, S^T = K Q^T with v_mfma_f32_32x32x16_bf16:
//     a lane then holds 16 keys of ONE query per 32-key block, so the softmax
//     row statistics are per-lane scalars (one cross-lane exchange with lane^32)
//     and the exponentiated block is already in the B-operand layout of the
//     second product O^T += V^T P^T. No register shuffle between the products.
//   - Block skipping (load-balanced sharding leaves half of every off-diagonal step fully
//     masked): from the min/max kv_pos of every block a workgroup compacts the blocks that any of
//     its queries can see into a list in LDS and walks only those, four to a tile wherever they
//     lie; only blocks that straddle a query position pay for the mask.
//   - A ring whose ranks all live here is one launch: every rank's rows against the tiles of all
//     shards, so that Equation 4 over the ring steps happens inside the online softmax. (A
//     launch per ring step costs 12 to 17 us at small query shards whatever its work: 256
//     launches and 256 split merges for 16 ranks, 6.08 ms at 1024 new tokens on 131072 cached
//     ones, where one launch takes 0.94 ms; 4096 tokens of head_dim 64 over 4 ranks 3.8 ms
//     on the vector pipe, 55 to 60 us here.)
//   - Small and middling calls, whose row blocks would leave compute units idle or with very
//     different walks, plan in the workgroups themselves (PLAN), if their positions fit LDS: a
//     workgroup per row block where walks are short, equal shares of all the work elsewhere. Where
//     positions do not fit, and in single calls with few row blocks, the KV axis is split over
//     grid.z (SPLIT). What is cut goes to the workspace as fp32 partials, which a second launch
//     merges with Eq. 4.
//   - The epilogue transposes the accumulators through LDS so that every output
//     row leaves as one contiguous 4 D byte (fp32) or 2 D byte (bf16) run.
//   - The same body also merges into a running (O, LSE) in its epilogue (ACC), and walks the
//     shards of every rank's ring steps in ring order, each behind an arrival flag (RING,
//     prefill_ring_walk_kernel).
#include "cp_common.h"
#include "cp_launch_rules.h"
#include "cp_table.h"

namespace cp {
namespace {

constexpr int BM = 256;         // rows per workgroup
constexpr int BLOCK = kAttnBlock;  // keys per block: what is listed, masked and pipelined
constexpr int TILE = 4 * BLOCK;    // keys per LDS tile
constexpr int NWAVE = 8;           // wavefronts per workgroup
constexpr int NTHREADS = NWAVE * 64;
constexpr int POS_BYTES = TILE * 4;
constexpr int MAX_LIVE = NTHREADS;        // blocks looked at (and listed) per chunk
constexpr int PLAN_MAX_BLOCKS = 960;      // PLAN: block bounds kept in LDS (30K keys; what fits)
constexpr int PLAN_MAX_UNITS = 1024;      // PLAN: units per KV head
constexpr int kPlanWorkgroups = 256;      // one per CU
constexpr int kUnitCost = 3;              // start-up and epilogue of a unit, in steps (Geo::STEP_BLOCKS)
constexpr int kCutCost = 12;              // partials of a cut at head_dim 128, in tile steps
constexpr int kUncutTiles = 6;            // units up to this long are not worth a cut
constexpr float kRescaleSlack = 8.f;               // log2 units
constexpr float kOverflowSum = 1099511627776.f;    // 2^40: a block sum beyond it is redone
constexpr float kDeadRowRef = INFINITY;            // reference of a row that sees no key

struct Params {
  // The first rank and shard of the table, beside the sizes: a single call reads its arguments from
  // a few cache lines, in one go. (Spread over the table they were eight latencies one after the
  // other, 2 us of every call.)
  const void* q;
  const int32_t* q_pos;
  void* out;
  float* lse;
  const void* k;
  const void* v;
  const int32_t* kv_pos;
  const int2* bounds;     // (min, max) of kv_pos per block, shard after shard (not PLAN)
  const int32_t* q_lo;    // BAND only: smallest visible key position per query token
  float* part_out;        // SPLIT: [grid.z][rows_all_heads][D] fp32; PLAN: [2 slots per wg][BM][D]
  float* part_lse;        // likewise, without D
  int64_t rows_all_heads; // total_q * n_q_heads
  int64_t out_shard_stride;  // per_shard: bytes between the outputs of two shards
  int64_t lse_shard_stride;  // and elements between their LSE
  int32_t n_ranks, n_shards;
  int32_t n_kv;           // of the first shard
  int32_t rows;           // R = total_q * G
  int32_t group;          // G
  int32_t n_kv_heads;
  int32_t n_row_blocks;
  int32_t n_z;            // shards whose results are kept apart (1 if not per_shard)
  int32_t n_blocks;       // of all shards
  int32_t bounds_shift;   // blocks per entry of `bounds`: 1 << bounds_shift
  int32_t n_sub;          // SPLIT: parts of the KV axis (of every shard's, if per_shard)
  int32_t sub_blocks;     // SPLIT: blocks per part, by their index; 0: equal parts of the visible ones
  int32_t per_shard;      // the shards' results are kept apart
  ChunkRule chunks;       // of ordered_row_block, in rows (RING: in row blocks)
  int32_t xcd_slice;      // WHOLE, SPLIT: workgroups are placed by xcd_slice
  int32_t cut_units;      // PLAN: equal shares (else a workgroup per unit)
  int32_t spin_limit;     // RING: polls per shard before giving up
  float scale_log2;       // softmax scale * log2(e)
  int2* plan_rec;         // PLAN: (unit, begin in it) of every share, for plan_merge_kernel
  float* acc;             // ACC: running O, fp32 [rows_all_heads][D] (running LSE: lse)
  void* final_out;        // ACC: where the merged O goes on the last step (else NULL)
  float* final_lse;       // ACC: optional copy of the merged LSE
  int32_t* ring_error;    // RING: per rank; bit j is set when the wait of step j gave up
  AttnTable t;            // queries and outputs per rank, KV per shard
  const int32_t* arrived[kMaxTable];  // RING: per rank [n_shards], nonzero once step j's shard
                                      // may be read
  int32_t rb_begin[kMaxTable + 1];    // RING: first row block of every rank
};

// (min, max) of kv_pos per 32-key block (or, coarse, per four), for the shards of a whole call
// in one launch (a launch per shard costs more than the work: a shard of 8K keys is 256
// blocks). A wavefront takes four blocks.
template <bool COARSE>
__global__ __launch_bounds__(256) void kv_bounds_kernel(const AttnTable t, int32_t n_blocks,
                                                         int2* __restrict__ bounds) {
  const int lane = threadIdx.x & 63;
  const int b = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 4 + (lane >> 4);
  int lo = INT32_MAX, hi = INT32_MIN;
  if (b < n_blocks) {
    // (one shard: scalar loads)
    int first = 0, total_kv = t.n_kv[0];
    const int32_t* __restrict__ kv_pos = t.kv_pos[0];
    if (t.n_shards > 1) {
      int j = 0;
      for (int i = 1; i < t.n_shards; ++i) j += b >= t.blk_begin[i];
      kv_pos = t.kv_pos[j];
      total_kv = t.n_kv[j];
      first = t.blk_begin[j];
    }
#pragma unroll
    for (int h = 0; h < BLOCK; h += 16) {
      const int idx = (b - first) * BLOCK + h + (lane & 15);
      if (idx < total_kv) {
        const int32_t x = kv_pos[idx];
        lo = min(lo, x);
        hi = max(hi, x);
      }
    }
  }
#pragma unroll
  for (int o = COARSE ? 32 : 8; o > 0; o >>= 1) {
    lo = min(lo, __shfl_xor(lo, o, 64));
    hi = max(hi, __shfl_xor(hi, o, 64));
  }
  if (COARSE) {
    if (lane == 0 && b < n_blocks) bounds[b >> 2] = make_int2(lo, hi);
  } else {
    if ((lane & 15) == 0 && b < n_blocks) bounds[b] = make_int2(lo, hi);
  }
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

// The most parts that a launch of `wgs` workgroups cuts `tiles` tiles into: three rounds of
// workgroups, beyond which there is 2 % to gain and the partials grow without end.
int max_parts(int64_t wgs, int tiles, bool per_shard) {
  const int64_t three_rounds = wgs > 0 && wgs < 256 ? 768 / wgs : 1;
  return (int)std::min<int64_t>({three_rounds, tiles, per_shard ? 16 : CP_MAX_PARTS});
}

struct Plan {
  Mode mode;
  int n_row_blocks, n_blocks, n_sub, n_z;  // n_z: shards kept apart
  int sub_blocks;                          // see Params
  bool cut, coarse;
  size_t bounds_bytes, part_out_bytes, part_lse_bytes, rec_bytes;
  size_t total() const { return bounds_bytes + part_out_bytes + part_lse_bytes + rec_bytes; }
};

Plan make_plan(const AttnShape& s) {
  Plan pl = {};
  const int group = s.n_q_heads / s.n_kv_heads;
  pl.n_row_blocks = (int)((s.total_q * group + BM - 1) / BM);
  pl.n_blocks = s.n_blocks;
  pl.n_z = s.per_shard ? s.n_shards : 1;
  pl.n_sub = 1;
  const int64_t units = (int64_t)pl.n_row_blocks * pl.n_z;   // per KV head
  const int64_t wgs = units * s.n_kv_heads;
  // A single call of 256 row blocks and more has no workspace but its position bounds, one
  // entry per 128 keys.
  const bool single_large = s.n_shards == 1 && !s.per_shard && wgs >= 256;
  const size_t rows_all = (size_t)s.total_q * s.n_q_heads;
  pl.coarse = s.n_shards == 1;
  const size_t entries = pl.coarse ? (s.n_blocks + 3) / 4 : s.n_blocks;
  // (the planned launch has its bounds in LDS, but cp_attn_partial_accumulate, which shares the
  // workspace query, does not)
  pl.bounds_bytes = round256(std::max<size_t>(entries, 1) * sizeof(int2));
  // tiles of the average walk, if every query saw everything
  const int tiles = (int)((s.n_blocks / pl.n_z + 3) / 4);
  const bool one_call = s.n_shards == 1 && !s.per_shard;
  bool plan = !single_large && s.n_blocks <= PLAN_MAX_BLOCKS && units <= PLAN_MAX_UNITS &&
              wgs <= 8 * PLAN_MAX_UNITS &&
              // (the line of all units, in half tiles, times 256, and token rows, within 32 bits)
              wgs * (24 + s.n_blocks / 4) < (1ll << 23);
  if (one_call) {
    // A call of one rank against one shard, as a rank of a real ring makes it. Up to two tiles, or
    // up to six with three times as many row blocks: a workgroup per row block in one launch (400
    // queries of 16 heads on 500 keys 22 us, with the KV axis split in three launches 25; 200
    // queries, 13 row blocks on 4 tiles, 22.7 and 22.3; 64 queries 22 against 18). Equal shares from 128 row blocks on: with fewer, parts of the KV axis
    // fill the CUs as well and write a smaller partial (1000 queries on their own 1000 keys 28 us
    // against 40). From 86 row blocks on two parts are all that fits one round, and equal shares
    // are better if the walks are long (3100 queries of 8 heads on 2 KV heads, later half of them
    // seeing all keys: 53 us against 64). At head_dim 64 a partial is half as large and parts win
    // earlier (700 queries of 16 heads on 2 25 us against 31).
    const int seen = tiles / s.batch;
    const bool uncut = seen <= 2 || (seen <= kUncutTiles &&
                                     wgs >= (s.head_dim == 64 ? 128 : 3 * seen));
    const bool cut = seen > kUncutTiles && (wgs >= 128 || (3 * wgs > 256 && seen >= 16));
    // (With the position bounds there already, planning costs more than it saves: 33 ranks of 60
    // tokens 14.4 us a call against 12.3; and equal shares leave no room for a second stream.)
    plan = plan && (uncut || cut) && !s.has_bounds;
  }
  if (plan) {
    pl.mode = PLAN;
    // Up to six tiles a unit there is nothing worth cutting (the plan and the merge launch take
    // as long as three tile steps).
    pl.cut = (one_call ? tiles / s.batch : tiles) > kUncutTiles;
    if (pl.cut) {
      pl.part_out_bytes = (size_t)2 * kPlanWorkgroups * BM * s.head_dim * 4;
      pl.part_lse_bytes = (size_t)2 * kPlanWorkgroups * BM * 4;
      pl.rec_bytes = (kPlanWorkgroups + 2) * sizeof(int2);
    }
    return pl;
  }
  // Otherwise the KV axis is split where the workgroups alone leave CUs idle: for every shard
  // kept apart by the size of the average shard.
  pl.n_sub = choose_splits(wgs, tiles, (double)rows_all * pl.n_z, s.head_dim,
                           max_parts(wgs, tiles, s.per_shard));
  pl.mode = pl.n_sub > 1 ? SPLIT : WHOLE;
  if (pl.mode == SPLIT) {
    // One shard of more blocks than a workgroup lists at once: parts by index, since counting and
    // passing over the blocks of the others takes longer than equal parts gain.
    if (one_call && s.n_blocks > MAX_LIVE) {
      const int per = (tiles + pl.n_sub - 1) / pl.n_sub;
      pl.n_sub = (tiles + per - 1) / per;
      pl.sub_blocks = 4 * per;
    }
    pl.part_out_bytes = round256((size_t)pl.n_z * pl.n_sub * rows_all * s.head_dim * 4);
    pl.part_lse_bytes = round256((size_t)pl.n_z * pl.n_sub * rows_all * 4);
  }
  return pl;
}

using Kern = void (*)(Params);

template <int D, bool BAND>
Kern pick_kernel(Mode mode, bool bf16_out) {
  if (mode == SPLIT) return prefill_mfma_kernel<D, float, BAND, SPLIT>;
  if (mode == PLAN)
    return bf16_out ? prefill_mfma_kernel<D, bf16_t, BAND, PLAN>
                    : prefill_mfma_kernel<D, float, BAND, PLAN>;
  return bf16_out ? prefill_mfma_kernel<D, bf16_t, BAND, WHOLE>
                  : prefill_mfma_kernel<D, float, BAND, WHOLE>;
}

int launch_body(Kern kern, int smem, const dim3& grid, const Params& p, hipStream_t stream) {
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem) !=
      hipSuccess)
    return CP_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, grid, dim3(NTHREADS), smem, stream, p);
  return check_launch();
}

int launch_kv_bounds(const AttnTable& t, int n_blocks, bool coarse, void* out, hipStream_t stream) {
  if (n_blocks == 0) return CP_OK;
  hipLaunchKernelGGL(coarse ? kv_bounds_kernel<true> : kv_bounds_kernel<false>,
                     dim3((n_blocks + 15) / 16), dim3(256), 0, stream, t, n_blocks, (int2*)out);
  return check_launch();
}

int check_rows(const AttnShape& s) {
  if (s.n_kv_heads > 65535) return CP_ERR_SHAPE;
  const int64_t rows = s.total_q * (s.n_q_heads / s.n_kv_heads);
  if (rows > 0x7fffffffLL) return CP_ERR_SHAPE;  // 31-bit rows
  if ((rows + BM) / BM * s.n_kv_heads > 0x7fffffffLL) return CP_ERR_SHAPE;
  return CP_OK;
}

void fill_params(const AttnShape& s, const AttnTable& t, Params& p) {
  p.t = t;
  p.q = t.q[0]; p.q_pos = t.q_pos[0]; p.out = t.out[0]; p.lse = t.lse[0];
  p.k = t.k[0]; p.v = t.v[0]; p.kv_pos = t.kv_pos[0];
  p.n_kv = t.n_kv[0];
  p.n_ranks = t.n_ranks; p.n_shards = t.n_shards;
  p.group = s.n_q_heads / s.n_kv_heads;
  p.rows = (int32_t)(s.total_q * p.group);   // (check_rows)
  p.rows_all_heads = s.total_q * s.n_q_heads;
  p.n_row_blocks = (int32_t)(((int64_t)p.rows + BM - 1) / BM);
  p.n_kv_heads = s.n_kv_heads;
  p.chunks = chunk_rule(t.n_ranks, t.tok_begin, (uint32_t)p.group);
  p.n_blocks = s.n_blocks;
  p.n_sub = p.n_z = 1;
  p.scale_log2 = s.scale * kLog2e;
}

}  // namespace

bool attn_mfma_applies(int dtype, int head_dim, int n_q_heads, int n_kv_heads) {
  return dtype == CP_BF16 && (head_dim == 128 || head_dim == 64) &&
         n_q_heads / n_kv_heads <= 64;
}

// A program may keep one workspace, sized for its largest KV, and call with less. Fewer keys can
// need more (other part counts, equal shares), so the size covers every smaller KV: the shares if
// any of them is cut into shares, and the most parts that any of them is split into.
size_t attn_mfma_workspace_bytes(const AttnShape& s) {
  const Plan pl = make_plan(s);
  if (pl.mode == PLAN && !pl.cut) return pl.total();   // and so is every smaller KV
  size_t need = pl.total() - pl.bounds_bytes;
  AttnShape fewer = s;
  fewer.n_blocks = std::min(s.n_blocks, PLAN_MAX_BLOCKS);
  const Plan shares = make_plan(fewer);
  if (shares.cut) need = std::max(need, shares.total() - shares.bounds_bytes);
  // (Short walks one by one, longer ones by the bound. Where equal shares take over, from 16 tiles
  // per sequence on at the latest, there are none of those up to the plan's limit.)
  const int kShort = s.batch <= 8 ? 16 * std::max(s.batch, 1) : 0;
  const int tiles = (int)((s.n_blocks / pl.n_z + 3) / 4);
  const int64_t wgs = (int64_t)pl.n_row_blocks * pl.n_z * s.n_kv_heads;
  const size_t rows = (size_t)pl.n_z * s.total_q * s.n_q_heads;
  int parts = 1;
  for (int t = 2; t <= std::min(tiles, kShort); ++t)
    parts = std::max(parts, choose_splits(wgs, t, (double)rows, s.head_dim,
                                          max_parts(wgs, t, s.per_shard)));
  if (tiles > kShort && !(s.n_blocks <= PLAN_MAX_BLOCKS && shares.cut))
    parts = std::max(parts, max_parts(wgs, tiles, s.per_shard));
  if (parts > 1)
    need = std::max(need, round256(parts * rows * s.head_dim * 4) + round256(parts * rows * 4));
  return pl.bounds_bytes + need;
}

size_t attn_mfma_ring_workspace_bytes(const AttnShape& s) {
  return round256((size_t)std::max(s.n_blocks, 1) * sizeof(int2));
}

bool attn_mfma_merging_applies(const AttnShape& s) {
  const int64_t rows = s.total_q * (s.n_q_heads / s.n_kv_heads);
  const int64_t wgs = (rows + BM - 1) / BM * s.n_kv_heads;
  if (s.head_dim != 128) return false;
  if (wgs >= 128 || wgs == 0) return true;
  return choose_splits(wgs, (s.n_blocks + 3) / 4, (double)s.total_q * s.n_q_heads, s.head_dim,
                       CP_MAX_PARTS) == 1;
}

bool attn_mfma_has_partials(const AttnShape& s) { return make_plan(s).part_out_bytes > 0; }

size_t kv_bounds_ring_bytes(int n_shards, const int64_t* n_kv) {
  size_t entries = 0;
  for (int b = 0; b < n_shards; ++b) entries += (size_t)((n_kv[b] + TILE - 1) / TILE);
  return round256(std::max<size_t>(entries, 1) * sizeof(int2));
}

int launch_kv_bounds_ring(int n_shards, const int32_t* const* kv_pos, const int64_t* n_kv,
                          void* region, size_t* offset, hipStream_t stream) {
  int2* out = (int2*)region;
  for (int first = 0; first < n_shards; first += kMaxTable) {
    AttnTable t = {};
    t.n_shards = std::min(n_shards - first, kMaxTable);
    int64_t blocks = 0;
    for (int j = 0; j < t.n_shards; ++j) {   // (a shard begins with a new entry, of four blocks)
      const int b = first + j;
      if (n_kv[b] > INT32_MAX - TILE) return CP_ERR_SHAPE;
      t.kv_pos[j] = kv_pos[b];
      t.n_kv[j] = (int32_t)n_kv[b];
      t.blk_begin[j] = (int32_t)blocks;
      offset[b] = (size_t)(out + blocks / 4 - (int2*)region) * sizeof(int2);
      blocks += (n_kv[b] + TILE - 1) / TILE * 4;
      if (blocks > INT32_MAX - 16) return CP_ERR_SHAPE;
    }
    t.blk_begin[t.n_shards] = (int32_t)blocks;
    const int rc = launch_kv_bounds(t, (int)blocks, true, out, stream);
    if (rc != CP_OK) return rc;
    out += blocks / 4;
  }
  return CP_OK;
}

int launch_attn_mfma(const AttnShape& s, const AttnTable& t, const AttnOut& o,
                     const int32_t* q_lo, void* workspace, size_t workspace_bytes,
                     const void* bounds, OverShards* over, hipStream_t stream) {
  const Plan pl = make_plan(s);
  if (workspace_bytes < pl.total()) return CP_ERR_WORKSPACE;
  if (pl.n_row_blocks == 0) return CP_OK;
  int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  const bool bf16_out = o.dtype == CP_BF16, band = q_lo != nullptr;
  if (band && s.head_dim != 128) return CP_ERR_UNSUPPORTED;
  char* ws = (char*)workspace;
  Params p = {};
  fill_params(s, t, p);
  p.bounds = (const int2*)(bounds != nullptr ? bounds : ws);
  p.bounds_shift = pl.coarse ? 2 : 0;
  p.part_out = (float*)(ws + pl.bounds_bytes);
  p.part_lse = (float*)(ws + pl.bounds_bytes + pl.part_out_bytes);
  p.plan_rec = (int2*)(ws + pl.bounds_bytes + pl.part_out_bytes + pl.part_lse_bytes);
  p.q_lo = q_lo;
  p.n_sub = pl.n_sub;
  p.sub_blocks = pl.sub_blocks;
  p.n_z = pl.n_z;
  p.per_shard = s.per_shard ? 1 : 0;
  p.cut_units = pl.cut ? 1 : 0;
  p.out_shard_stride = o.shard_out_bytes;
  p.lse_shard_stride = o.shard_lse_elems;
  if (pl.mode != PLAN && bounds == nullptr) {
    rc = launch_kv_bounds(t, s.n_blocks, pl.coarse, ws, stream);
    if (rc != CP_OK) return rc;
  }
  const Kern kern = s.head_dim == 64 ? pick_kernel<64, false>(pl.mode, bf16_out)
                    : band           ? pick_kernel<128, true>(pl.mode, bf16_out)
                                     : pick_kernel<128, false>(pl.mode, bf16_out);
  const int smem = s.head_dim == 64 ? (pl.mode == PLAN ? Geo<64>::SMEM_PLAN : Geo<64>::SMEM)
                                    : (pl.mode == PLAN ? Geo<128>::SMEM_PLAN : Geo<128>::SMEM);
  const unsigned wgs = (unsigned)(pl.n_row_blocks * s.n_kv_heads);
  const dim3 grid = pl.mode == PLAN ? dim3(pl.cut ? kPlanWorkgroups : wgs * pl.n_z)
                                    : dim3(wgs, 1, pl.n_z * pl.n_sub);
  const GridParts parts = s.per_shard ? shards_alike(t.n_shards, t.n_kv, s.total_q) ? kShardsAlike
                                                                                    : kShardsOther
                          : s.n_shards > 1 ? kPartsOfVisible
                                           : kPartsByIndex;
  p.xcd_slice = xcd_slice_applies(parts, pl.n_row_blocks, s.n_kv_heads, grid.z, s.n_blocks) ? 1 : 0;
  rc = launch_body(kern, smem, grid, p, stream);
  if (rc != CP_OK) return rc;

  if (pl.cut) {
    const dim3 mgrid(kPlanWorkgroups - 1, kMergeParts);
    auto mk = s.head_dim == 64 ? (bf16_out ? plan_merge_kernel<64, bf16_t> : plan_merge_kernel<64, float>)
                               : (bf16_out ? plan_merge_kernel<128, bf16_t> : plan_merge_kernel<128, float>);
    hipLaunchKernelGGL(mk, mgrid, dim3(256), 0, stream, p);
    return check_launch();
  }
  if (pl.mode != SPLIT) return CP_OK;
  // Equation 4 over the parts: of the whole KV axis, or of every shard into the shard's output
  MergeTable m = {};
  m.n_ranks = t.n_ranks;
  m.n_parts = pl.n_sub;
  m.part_bytes = p.rows_all_heads * s.head_dim * 4;
  m.part_lse_elems = p.rows_all_heads;
  m.n_groups = pl.n_z;
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
  m.rows = m.row_begin[t.n_ranks] = p.rows_all_heads;
  if (over != nullptr && merge_over_groups_applies(m)) {
    over->done = true;
    return launch_merge_over_groups(m, s.head_dim, o.dtype, *over, stream);
  }
  return launch_merge_table(m, s.head_dim, CP_FP32, o.dtype, stream);
}

int launch_attn_mfma_accumulate(const AttnShape& s, const AttnTable& t,
                                const PrefillAccumulate& acc, void* workspace,
                                size_t workspace_bytes, const void* bounds, hipStream_t stream) {
  if (!attn_mfma_merging_applies(s)) return CP_ERR_UNSUPPORTED;
  const size_t need = round256((size_t)std::max((s.n_blocks + 3) / 4, 1) * sizeof(int2));
  if (bounds == nullptr && workspace_bytes < need) return CP_ERR_WORKSPACE;
  int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  if (bounds == nullptr) {
    rc = launch_kv_bounds(t, s.n_blocks, true, workspace, stream);
    if (rc != CP_OK) return rc;
  }
  Params p = {};
  fill_params(s, t, p);
  p.bounds = (const int2*)(bounds != nullptr ? bounds : workspace);
  p.bounds_shift = 2;
  p.acc = acc.out;
  p.final_out = acc.final_out;
  p.final_lse = acc.final_lse;
  return launch_body(acc.final_out != nullptr && acc.final_dtype == CP_BF16
                         ? prefill_mfma_kernel<128, bf16_t, false, ACC>
                         : prefill_mfma_kernel<128, float, false, ACC>,
                     Geo<128>::SMEM, dim3((unsigned)(p.n_row_blocks * p.n_kv_heads)), p, stream);
}

int launch_attn_mfma_ring(const AttnShape& s, const AttnTable& t, const int32_t* const* arrived,
                          int32_t* error, int32_t spin_limit, int32_t out_dtype, void* workspace,
                          size_t workspace_bytes, hipStream_t stream) {
  if (arrived == nullptr || error == nullptr || spin_limit < 1) return CP_ERR_SHAPE;
  if (t.n_ranks != t.n_shards) return CP_ERR_SHAPE;
  if (workspace_bytes < attn_mfma_ring_workspace_bytes(s)) return CP_ERR_WORKSPACE;
  int rc = check_rows(s);
  if (rc != CP_OK) return rc;
  rc = launch_kv_bounds(t, s.n_blocks, false, workspace, stream);
  if (rc != CP_OK) return rc;
  Params p = {};
  fill_params(s, t, p);
  p.bounds = (const int2*)workspace;
  p.ring_error = error;
  p.spin_limit = spin_limit;
  int64_t blocks = 0;
  for (int a = 0; a < t.n_ranks; ++a) {
    p.arrived[a] = arrived[a];
    p.rb_begin[a] = (int32_t)blocks;
    blocks += ((int64_t)(t.tok_begin[a + 1] - t.tok_begin[a]) * p.group + BM - 1) / BM;
  }
  p.rb_begin[t.n_ranks] = (int32_t)blocks;
  if (blocks == 0) return CP_OK;
  if (blocks * p.n_kv_heads > 0x7fffffffLL) return CP_ERR_SHAPE;
  p.n_row_blocks = (int32_t)blocks;
  p.chunks = chunk_rule_in_blocks(t.n_ranks, p.chunks, BM, blocks);
  return launch_body(out_dtype == CP_BF16 ? prefill_ring_walk_kernel<bf16_t>
                                          : prefill_ring_walk_kernel<float>,
                     Geo<128>::SMEM, dim3((unsigned)(blocks * p.n_kv_heads)), p, stream);
}

}  // namespace cp
