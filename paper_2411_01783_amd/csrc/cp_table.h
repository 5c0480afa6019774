// Device helpers for kernels that work on an AttnTable (queries of several ranks back to back).
#pragma once

#include "cp_common.h"

namespace cp {
namespace {

// Row block that workgroup i of B takes: the longest walks first, so that what runs last is
// short. In one rank's shard (chunk r of the sequence, then chunk 2N-1-r) later rows see more
// keys. Over N ranks back to back the late chunks of all ranks go first, rank 0's (the last of
// the sequence) at their head, then the early chunks, rank 0's (the first of the sequence) last.
// The boundaries are those of equal shards; shards of other sizes only lose some of the order.
__device__ __forceinline__ int ordered_row_block(int i, int B, int n_ranks, int lane) {
  if (n_ranks == 1) return B - 1 - i;
  // lane l < N: second half of rank l; N <= l < 2N: first half of rank 2N-1-l  (N <= 32)
  const bool late = lane < n_ranks;
  const int r = late ? lane : 2 * n_ranks - 1 - lane;
  int lo = 0, hi = 0;
  if (r >= 0) {
    const int h = late ? 2 * r + 1 : 2 * r;
    lo = (int)((uint64_t)(uint32_t)h * (uint32_t)B / (uint32_t)(2 * n_ranks));
    hi = (int)((uint64_t)(uint32_t)(h + 1) * (uint32_t)B / (uint32_t)(2 * n_ranks));
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

}  // namespace
}  // namespace cp
