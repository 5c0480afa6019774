// Device helpers for kernels that work on an AttnTable (queries of several ranks back to back).
#pragma once

#include "cp_common.h"
#include "cp_launch_rules.h"

namespace cp {
namespace {

// Row block that workgroup i of B takes: the longest walks first, so that what runs last is
// short. In one rank's shard (chunk r of the sequence, then chunk 2N-1-r) later rows see more
// keys. Over N ranks back to back the late chunks of all ranks go first, rank 0's (the last of
// the sequence) at their head, then the early chunks, rank 0's (the first of the sequence) last.
// `rows`: of a row block, in the units of the rule.
__device__ __forceinline__ int ordered_row_block(int i, int B, int n_ranks, int lane, ChunkRule rule,
                                                 uint32_t rows) {
  if (n_ranks == 1) return B - 1 - i;
  // lane l < N: late chunk of rank l; N <= l < 2N: early chunk of rank 2N-1-l  (N <= 32)
  const bool late = lane < n_ranks;
  const int r = late ? lane : 2 * n_ranks - 1 - lane;
  int lo = 0, hi = 0;
  if (r >= 0) {   // (in 32 bits: 64-bit divisions took 1000 cycles of every start)
    const int middle = chunk_begin(2 * r + 1, B, n_ranks, rule, rows);
    const int side = chunk_begin(late ? 2 * r + 2 : 2 * r, B, n_ranks, rule, rows);
    lo = late ? middle : side;
    hi = late ? side : middle;
  }
  int end = hi - lo;  // inclusive prefix sum of the lengths
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int x = __shfl_up(end, o, 64);
    if (lane >= o) end += x;
  }
  const int seg = __builtin_ctzll(__builtin_amdgcn_ballot_w64(end > i));
  return __builtin_amdgcn_readlane(hi, seg) - 1 -
         (i - (__builtin_amdgcn_readlane(end, seg) - (__builtin_amdgcn_readlane(hi, seg) -
                                                     __builtin_amdgcn_readlane(lo, seg))));
}

// Rank whose queries global token `tok` belongs to.
__device__ __forceinline__ int rank_of_token(const AttnTable& t, int tok) {
  int a = 0;
#pragma unroll 8
  for (int i = 1; i < t.n_ranks; ++i) a += tok >= t.tok_begin[i];
  return a;
}

// One query row on the vector pipe, a wavefront for it, reading V of the visible keys only. The
// matrix pipe multiplies the V of a hidden key by a probability of zero, which is no zero if that
// V is infinite or NaN: the kernels look at their finished rows (one test per row and walk) and
// compute again, with this, those whose sum of probabilities is finite and whose O is not.
template <typename T, int D>
struct VectorRow {
  const T* q;
  float scale_log2;
  int32_t qp, ql;   // visible: ql <= kv_pos <= qp
  float m = -INFINITY, l = 0.f;
  float acc[D / 64] = {};   // channels lane * (D / 64) ..

  // `count` <= 64 keys; `stride`: elements between keys
  __device__ void keys(const T* k, const T* v, const int32_t* pos, int count, uint32_t stride,
                       int lane) {
    const int32_t x = pos[min(lane, count - 1)];
    const bool vis = lane < count && x <= qp && x >= ql;
    float s = -INFINITY;
    if (vis) {
      const T* const kj = k + (int64_t)lane * stride;
      float dot = 0.f;
#pragma unroll 4
      for (int c = 0; c < D; ++c) dot = fmaf(to_float(q[c]), to_float(kj[c]), dot);
      s = dot * scale_log2;
    }
    float bm = s;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bm = fmaxf(bm, __shfl_xor(bm, o, 64));
    const float m_new = fmaxf(m, bm);
    if (m_new == -INFINITY) return;
    const float old = __builtin_amdgcn_exp2f(m - m_new);
    const float pr = vis ? __builtin_amdgcn_exp2f(s - m_new) : 0.f;
    float sum = pr;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    l = fmaf(l, old, sum);
    m = m_new;
#pragma unroll
    for (int c = 0; c < D / 64; ++c) acc[c] *= old;
    for (int t = 0; t < count; ++t) {
      const float pt = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pr), t));
      if (pt == 0.f) continue;
      const T* const vj = v + (int64_t)t * stride + lane * (D / 64);
#pragma unroll
      for (int c = 0; c < D / 64; ++c) acc[c] = fmaf(pt, to_float(vj[c]), acc[c]);
    }
  }
};

}  // namespace
}  // namespace cp
