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

// The workgroups of one z onto as few XCDs as there are to share out: an XCD's L2 fetches a tile of
// keys once for all that walk it there; as dispatched, 8 row blocks against 16 holders in two parts
// each put every key on every XCD. g = gcd(nz, 8) classes of z, an eighth of the workgroups for each
// XCD: class xcd % g, and every (8 / g)-th x. The order of x (longest walks first) is kept.
CP_RULE GridPos xcd_slice(int x, int z, int nx, int nz) {
  const int g = (nz & -nz & (kXcds - 1)) ? (nz & -nz) : kXcds, s = kXcds / g;
  if (g == 1 || nx % s != 0) return {x, z};
  const uint32_t line = (uint32_t)x + (uint32_t)nx * (uint32_t)z;
  const uint32_t xcd = line % kXcds, idx = line / kXcds, per = (uint32_t)nz / (uint32_t)g;
  const uint32_t k = idx / per;
  return {(int)(k * s + xcd / g), (int)(xcd % g + g * (idx - k * per))};
}

// What the z of a grid are.
enum GridParts {
  kPartsOfVisible,  // equal parts of what every row block sees
  kPartsByIndex,    // of one shard, by the index of the keys
  kShardsAlike,     // shards kept apart, of one length, and few queries (new ones on cached keys)
  kShardsOther      // shards kept apart
};
CP_RULE bool shards_alike(int n, const int32_t* n_kv, int64_t total_q) {
  int64_t longest = 0, total = 0;
  for (int i = 0; i < n; ++i) {
    longest = n_kv[i] > longest ? n_kv[i] : longest;
    total += n_kv[i];
  }
  return 20 * longest * n <= 21 * total && 8 * total_q <= total;
}

// Where xcd_slice is used: row blocks that share keys (2 of a KV head at least), few enough that the
// traffic of the keys counts, and z of the same work, since a class of z has its XCDs' compute units
// and no others. us, as dispatched and sliced:
//   rings merged in the launch, 4 to 32 row blocks, one round: 65 queries of 8 heads on 2 KV heads on 40401 keys of
//     8 ranks 43.1 and 39.9, 106 of 16 on 4 on 106961 of 16 126.9 and 119.5, 588 of 8 on 2 122.6 and 117.7
//   one shard by index, 4 to 8, one round, in 32 parts or more (under a causal mask the first are the
//     long walks): 128 queries of 16 heads on 131072 keys 137 and 133, 64 81 and 78; 128 on 16384 keys
//     37.4 and 40.4
//   shards kept apart, alike, 3 to 16, of three quarters of a round to two: 128 queries of 16 heads on
//     16 of 8192 keys 149.8 and 145.3, 160 of 16 on 16 of 5733 155.0 and 149.7, 96 of 8 on 2 on 16 of
//     1970 45.3 and 42.2; but 64 of 16 on 2 of 15872 44.4 and 47.5, half a round
// and where not:
//   shards that are not alike: 1024 queries of 16 heads on 16 of 8192 keys, one of them of 16384, 1111
//     and 1506; 32768 causal tokens in 8 contiguous shards 4663 and 7144; 49152 tokens of one head on
//     themselves, by index, 601 and 899; of one round, too: 1024 queries on 49152 and 16384 keys 558
//     and 696
//   one row block a KV head: 32 queries of 16 heads on 4 KV heads on 32768 keys 31.8 and 32.9
//   more row blocks, more rounds: no difference where the z are alike
// (Fewer keys than some 30000 are planned in equal shares.)
// (Shards alike whose keys the queries do not see alike, contiguous ones in the middle of which the
// queries stand, lose up to 40 %; with load-balanced shards there is no such thing.)
CP_RULE bool xcd_slice_applies(GridParts parts, int64_t row_blocks, int64_t n_kv_heads, int64_t nz,
                               int64_t n_blocks) {
  const int64_t nx = row_blocks * n_kv_heads;
  if (nz < 2 || row_blocks < 2 || parts == kShardsOther) return false;
  if (parts == kShardsAlike)
    return nx >= 3 && nx <= 16 && nx * nz >= kCus * 3 / 4 && nx * nz <= 2 * kCus;
  if (nx < 4 || nx * nz > kCus) return false;
  return parts == kPartsOfVisible ? nx <= 32 : nx <= 8 && nz >= 32 && n_blocks >= 2048;
}

// Equal shares of a planned call (256 of `units` row blocks, per KV head and shard kept apart): whether
// neighbouring shares go to one XCD, as they walk the same keys. With few units neighbours are mostly
// parts of one unit, that is other keys, and at head_dim 128 that costs. As dispatched and grouped, us:
// 104 queries of 16 heads on 4 KV heads, 8 units, on 24208 keys 74.0 and 75.6, 12 units on 12649 62.3 and
// 64.5, 20 on 20628 90.9 and 94.2; 28 on 12047 76.2 and 73.7 (28 to 100 are 0.95 to 1.05 of the time, 1.00
// on average); packed prompts 111.5 and 110.7. Head_dim 64: 16 to 48 units 0.93 to 1.01 of the time, a
// ring of 4096 tokens 62.4 and 61.3.
CP_RULE bool shares_grouped(int head_dim, int units) { return head_dim == 64 || units >= 28; }

// ---- packed batches: spans found and positions encoded in one launch, or in two ----

// `lists`: of positions, the queries of every rank and the keys of every shard. In one launch the 16
// wavefronts of a workgroup walk batch * lists / 16 pieces each, one after the other; in two, every
// sequence has a workgroup of its own, which walks the lists, and the second launch costs as much as
// 3 to 4 pieces. The line is where the two take the same, by the sweep of 1 to 64 sequences over 1 to
// 32 ranks (whole call, us, one launch and two): over 1 rank 28 sequences of 256 tokens 28.6 and
// 29.2, 40 46.0 and 44.7; over 4 ranks 8 33.3 and 34.8, 12 37.2 and 37.0, 64 104 and 82; over 16 ranks
// 5 63.2 and 64.4, 8 56.1 and 52.9, 64 236 and 144; over 32 ranks 4 73.1 and 75.6, 8 87 and 78.
// Every workgroup reads all positions, up to 65536 tokens: that is as far as it was measured (one
// sequence of 32768 1869 and 1889, 8 of 4096 over 4 ranks 352.5 and 355.5).
CP_RULE bool encode_in_one_launch(int64_t batch, int64_t lists, int64_t tokens) {
  return (batch - 5) * lists <= 48 && tokens <= 65536;
}

// ---- the chunks of a ring's ranks among the row blocks, for ordered_row_block ----

// Where the chunks lie, in rows: a rank's early chunk, then its late one. Sharding deals chunks of one length, and what the last ones lack is missing from the late chunks
// of the first ranks (the whole of it, then the next rank's). Sizes dealt otherwise only lose some of
// the order.
struct ChunkRule {
  uint32_t rank, early, missing;
};
// `begin`: of every rank, and the end, in tokens of `rows` rows.
CP_RULE ChunkRule chunk_rule(int N, const int32_t* begin, uint32_t rows) {
  const int64_t all = (int64_t)begin[N] * rows;
  int64_t longest = 0;
  for (int r = 0; r < N; ++r)
    longest = longest < begin[r + 1] - begin[r] ? begin[r + 1] - begin[r] : longest;
  int64_t rank = longest * rows, early = longest / 2 * rows;
  if (rank * N > 0xffff0000ll) {   // (no sharding: 31 bits of rows and 2N tokens of a group are fewer)
    rank = (all + N - 1) / N;
    early = rank / 2;
  }
  return {(uint32_t)rank, (uint32_t)early, (uint32_t)(rank * N - all)};
}
// The same in row blocks of `rows` rows, `blocks` in all, none of which holds rows of two ranks.
CP_RULE ChunkRule chunk_rule_in_blocks(int N, ChunkRule c, uint32_t rows, int64_t blocks) {
  const int64_t rank = ((int64_t)c.rank + rows - 1) / rows, missing = rank * N - blocks;
  return {(uint32_t)rank, c.early / rows, missing > 0 ? (uint32_t)missing : 0};
}
// First of the B row blocks of `rows` rows (over the queries of N ranks back to back) of chunk j: rank
// j / 2's early chunk (j even) or late chunk (j odd). A block with rows of two chunks is the late one's,
// on either side of it, since its longest walk is a late row's: taken for early, such a block is
// dispatched last and the call waits for it alone. So it does for those that lie between the boundaries
// of equal chunks and the real ones, up to 2N - 1 tokens apart, almost two row blocks of 16 heads over 16
// ranks. us, with a block the chunk's that ends in it, the late one's between equal chunks, and here:
//   bf16: 33348 tokens of 8 heads over 16 ranks 2704, 2645 and 2028, 41111 of 16 over 16 6852, 6527 and
//     6031, 65050 of 16 over 16 15961, 16181 and 14955, 49873 of 8 on 2 over 8 5543, 5368 and 4441, 33001
//     of 8 at head_dim 64 over 16 3261, 3043 and 2258, 50723 of 8 over 4 5502, 4519 and 4536, 31744 of 16
//     over 16 3573, 3547 and 3548; none of 28 slower
//   fp32, between equal chunks and here: 1763 tokens of 4 heads over 4 ranks 45.5 and 35.8, 1761 over 3
//     41.9 and 35.9, 1320 over 4 25.2 and 25.2, 1345 of 8 on 2 over 4 49.3 and 44.6; none of 27 slower
//   the walk behind flags, whose row blocks do not straddle ranks, a block the chunk's that ends in it
//     and here: 44444 of 8 over 8 4491 and 3471, 90001 of 8 on 2 over 8 16364 and 13821, 77777 of 16 over
//     16 21774 and 20737, 65536 over 16 the same order; none of 16 slower
CP_RULE int chunk_begin(int j, int B, int N, ChunkRule c, uint32_t rows) {
  const uint32_t r = (uint32_t)j >> 1;
  const uint32_t lack = r * c.early < c.missing ? r * c.early : c.missing;
  const uint32_t x = r * c.rank - lack, first = (x + rows - 1) / rows, late = (x + c.early) / rows;
  const uint32_t b = j % 2 && late > first ? late : first;
  return j >= 2 * N || b > (uint32_t)B ? B : (int)b;
}

// ---- fp32 attention: rows and wavefronts of a workgroup ----

struct Fp32Form {
  int rows, waves;
};

// A workgroup's wavefronts share its keys, 16 at a time, and their results are combined in LDS. How
// many workgroups a CU holds is the registers' doing: at head_dim 64 two of 4 wavefronts (175
// registers) and one of 8, at head_dim 128 likewise. So the same wavefronts are at work either way, and
// 8 a workgroup halve the longest walk where there is one workgroup a CU or less; beyond that they
// run in two rounds, longest walks first, and win where walks differ in length (a whole prefill: as
// many queries as keys), and lose a start and an end where they do not. `keys`: of a walk on average,
// all of them or (kept_apart shards) those of a shard. us, 4 and 8 wavefronts:
//   up to 128 keys: a block of 16 for each of 8 or none. head_dim 64: 512 tokens of 4 heads on 16
//     6.0 and 6.6, 2048 6.8 and 11.1; head_dim 128, 8 shards of 64 kept apart, 2048 queries 87 and 137
//   one workgroup of 16 rows a CU (256): 512 tokens of 4 heads over 2 ranks 17.5 and 14.2, at
//     head_dim 128 26 and 21; 512 queries on 512 keys 17.4 and 13.6, 26 and 21
//   head_dim 64, up to 512 workgroups: 1320 tokens of 4 heads over 4 ranks 37 and 25, 2048 54 and 43,
//     1500 queries on 3000 cached and new keys 78 and 67; but 2048 queries that all see 512 keys 21.4
//     and 25.5, 1024 over 2 ranks, their partials kept apart, 25.6 and 26.8, 512 over 4 14.9 and 18.3.
//     Sizes do not say who sees what, and 8 lose where all rows see as much: 2048 queries on 1024 keys
//     36.9 and 39.5, the step of a ring in which a later rank's 1200 queries meet an earlier rank's keys
//     24.9 and 28.7 (the step the other way round 33 and 23), a shard that no query sees 5.8 and 9.2.
//   up to 768: 16 rows by 4: 2400 tokens of 4 heads 63.8 and 63.1, 3040 80 and 89, 700 workgroups of
//     8 heads on 2 KV heads 44.4 and 49
//   up to 1024: 32 rows, half the K/V traffic and half the workgroups: by 8, 3600 tokens of 4 heads
//     over 2 ranks 93 (16 rows by 4: 113), 4096 queries on 512 keys 38 (41); by 4 up to 256 keys, which
//     are one round: 4096 queries on 256 20.3 (16 rows by 4: 26.1, 32 by 8: 27.3), on 16 9.4 (11.2, 17)
//   beyond: 32 rows by 4 (5000 tokens of 4 heads 203, by 8 224), 16 rows where it is the kept-apart
//     shards that make the workgroups
//   head_dim 128 (16 rows): beyond 256 workgroups 4 up to 256 keys: 2048 queries on 8 shards of 256
//     kept apart 233 and 357; 2048 on 256 22 and 28. (On more, two workgroups of 4 a CU mostly win, 2048
//     queries on 8 shards of 512 272 and 325, but a whole prefill of 1100 tokens of 4 heads 51 and 36.)
CP_RULE Fp32Form fp32_form(int head_dim, int64_t rows, int64_t n_kv_heads, int64_t shards,
                           bool kept_apart, int64_t total_q, int64_t total_keys) {
  const int64_t apart = kept_apart ? shards : 1, keys = total_keys / apart;
  const int64_t wgs = (rows + 15) / 16 * n_kv_heads, all = wgs * apart;   // of 16 rows
  if (head_dim == 128) return {16, keys <= 128 || (keys <= 256 && all > kCus) ? 4 : 8};
  if (wgs > 4 * kCus) return {32, 4};
  if (all > 3 * kCus && all <= 4 * kCus) return {32, keys > 256 ? 8 : 4};
  if (all > 2 * kCus || keys <= 128) return {16, 4};
  if (all <= kCus) return {16, 8};
  return {16, !kept_apart && (keys > 512 || total_q == total_keys) ? 8 : 4};
}

}  // namespace cp
