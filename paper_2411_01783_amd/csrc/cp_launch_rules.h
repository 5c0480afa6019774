// Rules of the launches that are arithmetic on sizes alone. No HIP types: the same functions are
// compiled for the host and checked there over whole ranges of sizes.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define CP_RULE __host__ __device__ inline
#else
#define CP_RULE inline
#endif

namespace cp {

constexpr int kXcds = 8;   // workgroups go to them in turn, in the order of x + nx * z
constexpr int kCus = 256;

// ---- bf16 prefill: which workgroup of a grid nx * nz, whose z are different keys, runs where ----

struct GridPos {
  int x, z;
};

// The workgroups of one z on one XCD, whose L2 then fetches a tile of keys once for all that walk
// it; as dispatched, 8 row blocks against 16 holders in two parts each put every key on every XCD.
// z in turn over the XCDs; the order of x (longest walks first) is kept. (nz: a multiple of 8.)
CP_RULE GridPos xcd_slice(int x, int z, int nx, int nz) {
  const uint32_t line = (uint32_t)x + (uint32_t)nx * (uint32_t)z;
  const uint32_t xcd = line % kXcds, idx = line / kXcds, per = (uint32_t)nz / kXcds, k = idx / per;
  return {(int)k, (int)(xcd + kXcds * (idx - k * per))};
}

// Where that is done: one full round of workgroups, in which each has a compute unit to itself; few
// row blocks, so that the traffic of the keys counts; and keys enough (4096 blocks: 131072) for it to
// be seen. 128 queries of 16 heads, us, placed and as dispatched: 131072 keys in 16 shards kept apart
// 145.3 and 149.8, in one 133.0 and 137.0 (the queries spread over its positions: 114 and 137).
// Elsewhere it costs:
//   more row blocks: an XCD has 32 compute units for its z, and those may be the long ones. 16
//     holders of 8192 keys, one of them of 16384, 1024 queries 1506 and 1111; 32768 causal tokens in 8
//     contiguous shards 7144 and 4663; 49152 tokens of one head against themselves 899 and 601. Of one
//     round, too: 1024 queries on 2 shards of 32768 of which they see one 474 and 349.
//   part of a round: 96 queries that see 8 of 16 shards of 16384 182 and 136
//   few keys: 48 queries on 16384 33.3 and 28.3, 128 on 31744 in 16 shards (half seen) 56 and 54
CP_RULE bool xcd_slice_applies(int64_t nx, int64_t nz, int64_t n_blocks) {
  return nx * nz == kCus && nx <= 8 && n_blocks >= 4096;
}

}  // namespace cp
