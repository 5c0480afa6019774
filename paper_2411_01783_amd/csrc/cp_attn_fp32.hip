// fp32 attention on the matrix pipe, head_dim 64 and 128: the queries of one or more ranks
// against one or more KV shards in one launch (AttnTable), fp32 throughout.
//
// v_mfma_f32_16x16x4_f32 for both products, operands straight from global memory to registers:
// S^T = K Q^T leaves a lane with four keys of one query, so the softmax statistics are per-lane
// scalars (two lane exchanges) and exp(S^T) is the B operand of O^T += V^T P^T as it stands. The
// contraction order of the first product is free, so a lane takes four consecutive channels
// per 16-byte load of K; the channel order of the second is free as well, so a lane's 16-byte
// load of V serves four channel blocks.
//
// A workgroup of 4 or 8 wavefronts owns 16 * NR rows (token, head-in-group) of one KV head; the
// 16-key blocks that any of its queries can see are listed in LDS and dealt out over the
// wavefronts, whose results are combined in LDS at the end. Splitting the keys and not the rows
// over the wavefronts keeps small problems (the 512-token configuration has 2048 rows) on many
// CUs with a short serial chain each. NR = 2 (head_dim 64, many rows) halves the K/V traffic
// from L2.
//
// Bound: the matrix pipe's fp32 rate (157 TFLOP/s) for long shards, launch and the chain positions ->
// list -> K -> V for short ones. A ring of 512 tokens over 2 ranks (4 heads of 64) takes 13.5 us: 128
// workgroups, of whose 13 us the matrix pipe needs 3.4. It took 17.5 with 4 wavefronts a workgroup,
// 18.1 with the key positions asked for after the queries' had come as well, and 14.2 with the shard of
// a block and the rank of a row looked up by lane, two latencies of arguments ahead of the positions.
#include "cp_common.h"
#include "cp_launch_rules.h"
#include "cp_table.h"

namespace cp {
namespace {

constexpr int BLK = 16;                     // keys per block
constexpr int PER = kAttnBlock / BLK;       // blocks here per block of the table
constexpr int kMaxList = 512;               // blocks looked at per chunk: a thread each, at most

struct Params {
  AttnTable t;
  int64_t rows;              // total_q * group
  int32_t group;
  int32_t n_kv_heads;
  int32_t n_blocks;          // of the table
  int32_t per_shard;
  ChunkRule chunks;          // of ordered_row_block
  float scale_log2;          // (up to here one line: what the start asks for)
  int64_t out_shard_bytes;   // per_shard: distance between the results of two shards
  int64_t lse_shard_elems;
};

__device__ __forceinline__ floatx4_t mfma4(float a, float b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D>
struct BlockRegs {
  floatx4_t k[D / 16];      // key lane % 16, channels 16 j + (lane / 16) * 4 .. +3
  floatx4_t v[4][D / 64];   // key (lane / 16) * 4 + i, channels 64 h + (lane % 16) * 4 .. +3
  int32_t pos[4];           // of the keys (lane / 16) * 4 + i
  // Last key of the block that exists. Tested where pos is used: in load_block the test waits for the
  // positions just asked for before the block in hand is computed, for as long as the compiler's
  // order has it (2500 tokens of 4 heads of 64 67 to 74 us; 64.6 here).
  int last;
};

// (head_dim 128: two wavefronts a SIMD asked for; left to itself the compiler takes 278 registers for
// workgroups of 4, and one runs. Two at most: with a third, which 168 registers allow, whole prefills of
// 513 to 768 workgroups take their longest walks slower, 2500 tokens of 4 heads on 2 74 -> 79.6.)
template <int D, int NR, int NWAVE, typename TO>
__global__ __launch_bounds__(NWAVE * 64) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 1, 2)))
void attn_fp32_kernel(const Params p) {
  constexpr int NTHREADS = NWAVE * 64;
  constexpr int MAX_LIST = NTHREADS;                    // blocks looked at per chunk
  constexpr int ROWS = 16 * NR;
  constexpr int STRIDE = D + 4;
  __shared__ int2 list[MAX_LIST];                       // (shard, first key)
  __shared__ int wg_scratch[NWAVE];
  __shared__ __align__(16) float comb[NWAVE][ROWS][STRIDE];
  __shared__ float comb_m[NWAVE][ROWS], comb_l[NWAVE][ROWS];
  const int touched = touch_arguments<Params>();
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kg = lane >> 4;
  const int row_block = ordered_row_block(blockIdx.x, gridDim.x, p.t.n_ranks, lane, p.chunks, ROWS);
  const int kvh = blockIdx.y;
  const int z_shard = p.per_shard ? blockIdx.z : 0;

  // This thread's block of the chunk at b0 and its smallest position (none: above every query's).
  // The first chunk's positions are asked for before the queries, so that the two travel together.
  const int b_begin = (p.per_shard ? p.t.blk_begin[z_shard] : 0) * PER;
  const int b_end = (p.per_shard ? p.t.blk_begin[z_shard + 1] : p.n_blocks) * PER;
  int sh = z_shard, key0 = 0;
  int64_t lo = INT64_MAX;
  auto look = [&](int b0) {
    const int b = b0 + tid;
    sh = z_shard;
    lo = INT64_MAX;
    if (b < b_end) {
      const int blk = b / PER;
      // (scalar loads and selects: looked up by lane, the shard's arguments are another latency)
      int begin = p.t.blk_begin[z_shard], count = p.t.n_kv[z_shard];
      const int32_t* pos = p.t.kv_pos[z_shard];
      if (!p.per_shard) {
#pragma unroll 4
        for (int i = 1; i < p.t.n_shards; ++i) {
          const int x = p.t.blk_begin[i], c = p.t.n_kv[i];
          const int32_t* const y = p.t.kv_pos[i];
          const bool in = blk >= x;
          sh = in ? i : sh;
          begin = in ? x : begin;
          count = in ? c : count;
          pos = in ? y : pos;
        }
      }
      key0 = (blk - begin) * kAttnBlock + (b % PER) * BLK;
      const int last = count - 1 - key0;
      if (last >= 0) {
        const int32_t* pt = pos + key0;
        int m = INT32_MAX;
#pragma unroll
        for (int i = 0; i < BLK; ++i) m = min(m, pt[min(i, last)]);
        lo = m;
      }
    }
  };
  look(b_begin);

  const uint32_t stride = (uint32_t)p.n_kv_heads * D;
  auto load_block = [&](int sh, int key0, BlockRegs<D>& x) {
    const int last = p.t.n_kv[sh] - 1 - key0;   // >= 0
    const float* kt = (const float*)p.t.k[sh] + (int64_t)key0 * stride + kvh * D;
    const float* vt = (const float*)p.t.v[sh] + (int64_t)key0 * stride + kvh * D;
    const int32_t* pt = p.t.kv_pos[sh] + key0;
    x.last = last;
    const uint32_t krow = (uint32_t)min(n, last) * stride + kg * 4;
#pragma unroll
    for (int j = 0; j < D / 16; ++j) x.k[j] = *(const floatx4_t*)(kt + krow + j * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = kg * 4 + i, kc = min(key, last);
      x.pos[i] = pt[kc];
#pragma unroll
      for (int h = 0; h < D / 64; ++h)
        x.v[i][h] = *(const floatx4_t*)(vt + (uint32_t)kc * stride + h * 64 + n * 4);
    }
  };
  auto load_listed = [&](int e, BlockRegs<D>& x) {
    const int2 le = list[e];
    load_block(__builtin_amdgcn_readfirstlane(le.x), __builtin_amdgcn_readfirstlane(le.y), x);
  };
  // ---- queries: row r of column group c is this lane's column n ----
  // (The rank of the first row, in scalar registers, is mostly that of all.)
  const int t0 = (int)((uint32_t)(row_block * ROWS) / (uint32_t)p.group);
  const int a0 = rank_of_token(p.t, t0);
  const bool one_rank = (int64_t)row_block * ROWS + ROWS <= (int64_t)p.t.tok_begin[a0 + 1] * p.group ||
                        a0 == p.t.n_ranks - 1;
  floatx4_t qf[NR][D / 16];
  int32_t qp[NR];
  int qmax = INT32_MIN;
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    const int64_t r = (int64_t)row_block * ROWS + c * 16 + n;
    const bool ok = r < p.rows;
    const int token = ok ? (int)((uint32_t)r / (uint32_t)p.group) : 0;
    const int hg = ok ? (int)(r - (int64_t)token * p.group) : 0;
    const float* q = (const float*)p.t.q[a0];
    const int32_t* q_pos = p.t.q_pos[a0];
    int first = p.t.tok_begin[a0];
    if (!one_rank) {
      const int a = rank_of_token(p.t, token);
      q = (const float*)p.t.q[a];
      q_pos = p.t.q_pos[a];
      first = p.t.tok_begin[a];
    }
    const int local = ok ? token - first : 0;
    q += (((int64_t)local * p.n_kv_heads + kvh) * p.group + hg) * D + kg * 4;
    qp[c] = ok ? q_pos[local] : CP_POS_PAD_Q;
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
      qf[c][j] = ok ? *(const floatx4_t*)(q + j * 16) : floatx4_t{0.f, 0.f, 0.f, 0.f};
    qmax = max(qmax, qp[c]);
  }
  // The first block this wavefront takes if all of the first are visible, as they mostly are (else it
  // is not used): it travels with the queries, not behind the list. (head_dim 128, where a block is
  // longest on its way: 512 tokens of 4 heads 23.0 -> 21.3 us, 4096 of 8 heads 488 -> 464. A call that
  // sees none of its keys waits for it in vain: 512 queries on 512 6.3 -> 8.3. At head_dim 64 it gains
  // nothing: 14.1 and 14.3, 2048 tokens of 4 heads 42.9 and 45.0.)
  BlockRegs<D> cur, nxt;
  const int guess = wave * BLK;   // of the first shard
  const bool guessed = D == 128 && guess < p.t.n_kv[z_shard];
  if (guessed) load_block(z_shard, guess, cur);
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) qmax = max(qmax, __shfl_xor(qmax, o, 64));
  qmax = __builtin_amdgcn_readfirstlane(qmax);  // (the wavefronts hold the same rows)

  asm volatile("" ::"v"(touched));
  float m_run[NR], l_run[NR];
  floatx4_t acc[NR][D / 16];
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    m_run[c] = -INFINITY;
    l_run[c] = 0.f;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) acc[c][i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }

  auto compute = [&](const BlockRegs<D>& x) {
#pragma unroll
    for (int c = 0; c < NR; ++c) {
      floatx4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < D / 16; ++j)
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          s0 = mfma4(x.k[j][i], qf[c][j][i], s0);
          s1 = mfma4(x.k[j][i + 1], qf[c][j][i + 1], s1);
        }
      float s[4], mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[i] = x.pos[i] <= qp[c] && kg * 4 + i <= x.last ? (s0[i] + s1[i]) * p.scale_log2
                                                         : -INFINITY;
        mx = fmaxf(mx, s[i]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run[c], mx);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run[c] - m_use);
      m_run[c] = m_new;
      float ls = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[i] = __builtin_amdgcn_exp2f(s[i] - m_use);
        ls += s[i];
      }
      l_run[c] = fmaf(l_run[c], alpha, ls);
      if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
        for (int i = 0; i < D / 16; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[c][i][e] *= alpha;
      }
      // block h * 4 + e of O^T holds the channels 64 h + 4 m + e, m its row
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < D / 64; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[c][h * 4 + e] = mfma4(x.v[i][h][e], s[i], acc[c][h * 4 + e]);
    }
  };

  for (int b0 = b_begin; b0 < b_end; b0 += MAX_LIST) {
    // list of the blocks some query of the workgroup can see
    if (b0 != b_begin) look(b0);
    const bool live = lo <= qmax;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(live);
    lds_barrier();  // the previous list is no longer read
    if (lane == 0) wg_scratch[wave] = __builtin_popcountll(mask);
    lds_barrier();
    int base = 0, n_live = 0;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) {
      const int c = wg_scratch[w];
      if (w < wave) base += c;
      n_live += c;
    }
    n_live = __builtin_amdgcn_readfirstlane(n_live);
    if (live)
      list[base + __builtin_popcountll(mask & ((1ull << lane) - 1ull))] = make_int2(sh, key0);
    lds_barrier();

    // the next block's operands travel while the current one is used
    int e = wave;
    if (e < n_live) {
      const int2 le = list[e];
      if (b0 != b_begin || !guessed || __builtin_amdgcn_readfirstlane(le.x) != z_shard ||
          __builtin_amdgcn_readfirstlane(le.y) != guess)
        load_listed(e, cur);
    }
    while (e < n_live) {
      const int en = e + NWAVE;
      if (en < n_live) load_listed(en, nxt);
      compute(cur);
      cur = nxt;
      e = en;
    }
  }

  // ---- combine the wavefronts (disjoint keys) ----
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    float l = l_run[c];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    float* const o = comb[wave][c * 16 + n];
#pragma unroll
    for (int h = 0; h < D / 64; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const floatx4_t w = {acc[c][h * 4][i], acc[c][h * 4 + 1][i], acc[c][h * 4 + 2][i],
                             acc[c][h * 4 + 3][i]};
        *(floatx4_t*)(o + h * 64 + (kg * 4 + i) * 4) = w;
      }
    if (kg == 0) {
      comb_m[wave][c * 16 + n] = m_run[c];
      comb_l[wave][c * 16 + n] = l;
    }
  }
  __syncthreads();
  constexpr int TPR = NTHREADS / 16, CPT = D / TPR;   // threads per row, channels per thread
  static_assert(TPR <= 64 && CPT >= 1, "a row is in one wavefront");
#pragma unroll
  for (int c = 0; c < NR; ++c) {
    const int row = c * 16 + tid / TPR, ch = (tid % TPR) * CPT;
    const int64_t r = (int64_t)row_block * ROWS + row;
    const bool row_ok = r < p.rows;
    float mw[NWAVE], mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) {
      mw[w] = comb_m[w][row];
      mmax = fmaxf(mmax, mw[w]);
    }
    float x[CPT], den = 0.f;
#pragma unroll
    for (int i = 0; i < CPT; ++i) x[i] = 0.f;
    if (mmax != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NWAVE; ++w) {
        const float f = __builtin_amdgcn_exp2f(mw[w] - mmax);
        den = fmaf(comb_l[w][row], f, den);
#pragma unroll
        for (int i = 0; i < CPT; ++i) x[i] = fmaf(comb[w][row][ch + i], f, x[i]);
      }
    }
    const float inv = den > 0.f ? 1.f / den : 0.f;
    const int token = row_ok ? (int)((uint32_t)r / (uint32_t)p.group) : 0;
    const int hg = row_ok ? (int)(r - (int64_t)token * p.group) : 0;
    int a = a0, first = p.t.tok_begin[a0];
    char* out0 = (char*)p.t.out[a0];
    float* lse = p.t.lse[a0];
    if (!one_rank) {
      a = rank_of_token(p.t, token);
      first = p.t.tok_begin[a];
      out0 = (char*)p.t.out[a];
      lse = p.t.lse[a];
    }
    const int64_t lin = ((int64_t)(token - first) * p.n_kv_heads + kvh) * p.group + hg;
    out0 += z_shard * p.out_shard_bytes;
    // Rows that a V they do not see has spoiled (see VectorRow).
    float spoil = 0.f;   // stays zero if O is finite
#pragma unroll
    for (int i = 0; i < CPT; ++i) spoil = fmaf(x[i], 0.f, spoil);
    uint64_t spoiled = __builtin_amdgcn_ballot_w64(row_ok && den > 0.f && den < INFINITY &&
                                                   !(spoil == 0.f));
    constexpr uint64_t kRowLanes = TPR == 64 ? ~0ull : (1ull << (TPR & 63)) - 1;
    const bool mine = (spoiled >> (lane & ~(TPR - 1)) & kRowLanes) != 0;
    while (__builtin_expect(spoiled != 0, 0)) {
      const int rl = __builtin_ctzll(spoiled) & ~(TPR - 1);   // first lane of the row
      spoiled &= ~(kRowLanes << rl);
      const int ra = __builtin_amdgcn_readlane(a, rl);
      const int64_t rlin = (int64_t)(
          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)lin, rl) |
          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(lin >> 32), rl) << 32);
      VectorRow<float, D> vr;
      vr.q = (const float*)p.t.q[ra] + rlin * D;
      vr.scale_log2 = p.scale_log2;
      vr.qp = p.t.q_pos[ra][__builtin_amdgcn_readlane(token, rl) - p.t.tok_begin[ra]];
      vr.ql = INT32_MIN;
      for (int sh = z_shard; sh < (p.per_shard ? z_shard + 1 : p.t.n_shards); ++sh)
        for (int key0 = 0; key0 < p.t.n_kv[sh]; key0 += 64) {
          const int64_t off = (int64_t)key0 * stride + kvh * D;
          vr.keys((const float*)p.t.k[sh] + off, (const float*)p.t.v[sh] + off,
                  p.t.kv_pos[sh] + key0, min(64, p.t.n_kv[sh] - key0), stride, lane);
        }
      TO* const o = (TO*)((char*)p.t.out[ra] + z_shard * p.out_shard_bytes) + rlin * D;
#pragma unroll
      for (int i = 0; i < D / 64; ++i)
        o[lane * (D / 64) + i] = from_float<TO>(vr.acc[i] * (1.f / vr.l));
    }
    if (!row_ok) continue;
    if (!mine) {
      TO* const o = (TO*)out0 + lin * D + ch;
#pragma unroll
      for (int i = 0; i < CPT; ++i) o[i] = from_float<TO>(den > 0.f ? x[i] * inv : 0.f);
    }
    if (tid % TPR == 0 && lse != nullptr)
      lse[z_shard * p.lse_shard_elems + lin] =
          den > 0.f ? (mmax + __builtin_amdgcn_logf(den)) * kLn2 : -INFINITY;
  }
}

template <int D, int NR, int NWAVE, typename TO>
int launch_t(const AttnShape& s, Params& p, hipStream_t stream) {
  const int64_t blocks = (p.rows + 16 * NR - 1) / (16 * NR);
  if (blocks > 0x7fffffffLL) return CP_ERR_SHAPE;
  p.chunks = chunk_rule(p.t.n_ranks, p.t.tok_begin, (uint32_t)p.group);
  hipLaunchKernelGGL((attn_fp32_kernel<D, NR, NWAVE, TO>),
                     dim3((unsigned)blocks, s.n_kv_heads, s.per_shard ? s.n_shards : 1),
                     dim3(NWAVE * 64), 0, stream, p);
  return check_launch();
}

template <typename TO>
int launch_o(const AttnShape& s, Params& p, hipStream_t stream) {
  int64_t keys = 0;
  for (int b = 0; b < s.n_shards; ++b) keys += p.t.n_kv[b];
  const Fp32Form f = fp32_form(s.head_dim, p.rows, s.n_kv_heads, s.n_shards, s.per_shard, s.total_q,
                               keys);
  if (s.head_dim == 128)
    return f.waves == 4 ? launch_t<128, 1, 4, TO>(s, p, stream) : launch_t<128, 1, 8, TO>(s, p, stream);
  if (f.rows == 32)
    return f.waves == 4 ? launch_t<64, 2, 4, TO>(s, p, stream) : launch_t<64, 2, 8, TO>(s, p, stream);
  return f.waves == 4 ? launch_t<64, 1, 4, TO>(s, p, stream) : launch_t<64, 1, 8, TO>(s, p, stream);
}

}  // namespace

int launch_attn_fp32(const AttnShape& s, const AttnTable& t, const AttnOut& o,
                     hipStream_t stream) {
  if (s.head_dim != 64 && s.head_dim != 128) return CP_ERR_UNSUPPORTED;
  if (s.n_kv_heads > 65535) return CP_ERR_SHAPE;
  // block indices are kept in 31 bits; so are row indices
  if (s.n_blocks > 0x7fffffff / PER - kMaxList) return CP_ERR_SHAPE;
  Params p = {};
  p.t = t;
  p.group = s.n_q_heads / s.n_kv_heads;
  p.rows = s.total_q * p.group;
  if (p.rows > 0x7fffffffLL) return CP_ERR_SHAPE;
  if (p.rows == 0) return CP_OK;
  p.out_shard_bytes = o.shard_out_bytes;
  p.lse_shard_elems = o.shard_lse_elems;
  p.n_kv_heads = s.n_kv_heads;
  p.n_blocks = s.n_blocks;
  p.per_shard = s.per_shard ? 1 : 0;
  p.scale_log2 = s.scale * kLog2e;
  return o.dtype == CP_BF16 ? launch_o<bf16_t>(s, p, stream) : launch_o<float>(s, p, stream);
}

}  // namespace cp
