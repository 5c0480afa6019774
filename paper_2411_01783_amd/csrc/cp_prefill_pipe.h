// Software-pipelined bf16 MFMA attention kernel (included by cp_prefill_mfma.hip, which
// defines Params and the tile constants used here), for head_dim D = 128 and 64.
//
// K and V tiles travel HBM/L2 -> LDS with global_load_lds (16 bytes per lane, no register
// staging): both are stored row-major [key][2 D bytes]; bank conflicts are avoided by
// permuting the 16-byte chunks of a row on the GLOBAL side (k_perm / v_perm below). K
// fragments (rows = keys) are read with ds_read_b128, V^T fragments (rows = channels) with
// ds_read_b64_tr_b16.
//
// The KV axis is consumed in blocks of 32 keys and each wavefront runs three stages at
// once, one block apart:
//     P(i-1):  O^T += V^T P^T of the previous block        (D / 16 MFMA, matrix pipe; 12 at D = 64)
//     SM(i):   mask, row maximum, exponentials of block i   (vector pipe)
//     Q(i+1):  S^T = K Q^T of the next block                (D / 16 MFMA, matrix pipe)
// The three are independent, so the vector work is issued between the MFMAs of its
// neighbours, one slice per MFMA, in source order (scheduling fences keep that order). LDS
// fragment reads are inline assembly with hand-counted lgkmcnt waits, issued D / 16 MFMAs (of one
// term) before their use: the compiler would otherwise wait for the tile prefetch
// (vmcnt(0)) in front of every LDS read that follows a direct-to-LDS load, and would not
// keep reads in flight across its own waits.
//
// Synchronisation per 128-key tile, two buffers: barrier Y before the last block of a tile
// (the next tile has landed; that block's Q stage reads its first 32 keys), barrier X after
// it (every read of the current tile has completed; the tile after the next is requested
// into its buffer).
#pragma once

#define CP_LDS_AS __attribute__((address_space(3)))
#define CP_GLB_AS __attribute__((address_space(1)))

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

// Sizes and LDS layout for head_dim D. The list of visible 32-key blocks holds, per block, the
// addresses of its K and V rows (this KV head) and of its positions; four consecutive entries
// make a tile, wherever their keys lie, so that a workgroup walks any number of KV shards with
// one loop and spends nothing on blocks it cannot see.
template <int D>
struct Geo {
  static constexpr int ROW = D * 2;              // one K or V row in bytes
  static constexpr int KD = TILE * ROW;          // one tile buffer of K or of V
  static constexpr int BLK = 32 * ROW;           // one 32-key block of a tile
  static constexpr int NKS = D / 16;             // MFMAs of S^T per block, K fragments
  static constexpr int NDB = D / 32;             // 32-channel blocks of O^T
  static constexpr int NVF = 2 * NDB;            // MFMAs of O^T per block, V^T fragments
  // bf16 terms of a probability. head_dim 64: three, which hold all 24 bits of the fp32 value (the
  // products with V are exact and summed in fp32: nothing is rounded to 16 bits). head_dim 128: one.
  static constexpr int TERMS = D == 64 ? 3 : 1;
  // Blocks of a step: lists are cut between two of them (SPLIT, PLAN), and the line of units is counted
  // in them. Head_dim 128: a tile. Results depend on where a list is cut there (a probability is rounded
  // relative to the first block of its piece), and half tiles gain nothing (us, tiles and halves: 12
  // packed prompts of 40 to 1200 tokens over 4 ranks 91.9 and 92.3, 2 of 1700 to 2100 66.9 and 63.4, 6 of
  // 200 to 3000 97.6 and 99.1; 25 packed calls 1.00 of the time on average, 24 of pass-Q, too). Head_dim
  // 64, where all 24 bits are kept: half a tile. 7.5 us lie between the last tile of one unit and the
  // first of the next, and a tile takes 3.7 (987 tokens of 8 heads over 2 ranks 36.2 and 30.9, 4096 of 8
  // on 2 over 4 59.6 and 57.7; 61 calls 0.96 of the time on average, the worst 1.03).
  static constexpr int STEP_BLOCKS = D == 64 ? 2 : 4;
  static constexpr int CHUNKS = ROW / 16;        // 16-byte chunks of a row
  static constexpr int LOAD_ROWS = 64 / CHUNKS;  // rows one 1 KiB load instruction brings
  static constexpr int PARTS = 16 / LOAD_ROWS;   // load instructions per wavefront for K (or V)
  static constexpr int OFF_V = 2 * KD;
  static constexpr int OFF_POS = OFF_V + 2 * KD;
  static constexpr int OFF_SCRATCH = OFF_POS + 2 * POS_BYTES;
  static constexpr int OFF_LIVE = OFF_SCRATCH + 256;
  static constexpr int OFF_LIVE_POS = OFF_LIVE + MAX_LIVE * 16;
  static constexpr int OFF_LIVE_RANGE = OFF_LIVE_POS + MAX_LIVE * 8;
  static constexpr int OFF_BOUNDS = OFF_LIVE_RANGE + MAX_LIVE * 8;
  static constexpr int SMEM = OFF_BOUNDS;                        // bounds from global memory
  static constexpr int OFF_WEIGHT = OFF_BOUNDS + PLAN_MAX_BLOCKS * 8;  // PLAN: bounds kept in LDS
  static constexpr int OFF_SHARDS = OFF_WEIGHT + PLAN_MAX_UNITS * 2;   // units' weights,
  static constexpr int OFF_RANKS = OFF_SHARDS + kMaxTable * 32;        // the shards
  static constexpr int OFF_RANK_TOK = OFF_RANKS + kMaxTable * 32;      // and ranks, first token of each,
  static constexpr int OFF_BLOCK_SHARD = OFF_RANK_TOK + 144;           // shard of every block
  static constexpr int OFF_INDEX = OFF_BLOCK_SHARD + PLAN_MAX_BLOCKS;
  static constexpr int SMEM_PLAN = OFF_INDEX + 16;                     // which share this is
  static_assert(NWAVE * 32 * (D * 4 + 16) <= OFF_INDEX, "the epilogue's staging leaves it alone");
  static constexpr int OUT_STRIDE = D * 4 + 16;  // epilogue staging: one fp32 output row + pad
  static_assert(NWAVE * 32 * OUT_STRIDE <= SMEM, "epilogue staging fits in the allocation");
  static_assert(SMEM_PLAN <= 160 * 1024, "LDS budget of one CU");
  static_assert(2 * KD <= 65536, "K fragment offsets fit the 16-bit LDS offset field");
  static_assert(NKS == NVF, "the two halves of a pipeline step have the same length");
  // Chunk c of K row r lands at position c ^ k_perm(r): 16 lanes that read the same chunk of
  // 16 consecutive rows then touch all 64 banks. Chunk c of V row r lands at c ^ v_perm(r):
  // the four rows a transposed read covers lie in different 64-byte quarters of the banks.
  __host__ __device__ static constexpr int k_perm(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
  __host__ __device__ static constexpr int v_perm(int r) { return D == 128 ? (r & 3) * 4 : ((r >> 1) & 1) * 4; }
};

__device__ __forceinline__ void load_lds16(const void* src, char* lds_dst_wave_uniform) {
  __builtin_amdgcn_global_load_lds((const CP_GLB_AS void*)src, (CP_LDS_AS void*)lds_dst_wave_uniform,
                                   16, 0, 0);
}

template <int OFF>
__device__ __forceinline__ u32x4_t lds_read_b128(uint32_t addr) {
  u32x4_t r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// Lane i of a 16-lane group receives element i % 4 of the 8 bytes addressed by each of the
// lanes 4j + i / 4 (j = 0..3) of the group: four lanes address four consecutive keys of a
// 16-channel strip and every lane receives one channel of those four keys.
template <int OFF>
__device__ __forceinline__ u32x2_t lds_read_tr(uint32_t addr) {
  u32x2_t r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// Wait until at most N LDS operations issued after the one that fills the operands are
// outstanding. The operands are tied to the statement so that their consumer cannot be
// scheduled above the wait.
template <int N>
__device__ __forceinline__ void lgkm_wait(u32x4_t& x) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N < 15 ? N : 15));
}
template <int N>
__device__ __forceinline__ void lgkm_wait(u32x2_t& x, u32x2_t& y) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x), "+v"(y) : "n"(N < 15 ? N : 15));
}
template <int N>
__device__ __forceinline__ void lgkm_wait(u32x4_t& a, u32x4_t& b, u32x4_t& c, u32x4_t& d) {
  asm volatile("s_waitcnt lgkmcnt(%4)"
               : "+v"(a), "+v"(b), "+v"(c), "+v"(d)
               : "n"(N < 15 ? N : 15));
}
// A V^T fragment is two transposed reads into the halves of one 128-bit register tuple.
template <int OFF, int ROW>
__device__ __forceinline__ u32x4_t lds_read_vt_frag(uint32_t addr) {
  const u32x2_t lo = lds_read_tr<OFF>(addr), hi = lds_read_tr<OFF + 8 * ROW>(addr);
  const u32x4_t v = {lo[0], lo[1], hi[0], hi[1]};
  return v;
}
// Keeps the computation of x at this point of the instruction stream (the optimiser would
// otherwise sink the softmax arithmetic to its first use, one pipeline step later).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(unsigned& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  bf16x2_t t;
  t[0] = static_cast<bf16_t>(a);
  t[1] = static_cast<bf16_t>(b);
  return __builtin_bit_cast(unsigned, t);
}

// Everything a wavefront carries from block to block. All indices are compile-time.
template <int D>
struct PipeRegs {
  floatx16_t o[D / 32];    // O^T accumulators, blocks of 32 channels
  floatx16_t s[2];         // scores of block i (index: parity of i) and of block i+1
  // probabilities (bf16 pairs, per term) of block i (parity of i) / i-1, two 16-key slices
  u32x4_t pb[2][Geo<D>::TERMS][2];
  u32x4_t kf[D / 16];      // K fragments of block i+1
  u32x4_t vf[D / 16];      // V^T fragments of block i-1
  float m_run, l_run;
};


template <int J>
struct IntC {
  static constexpr int value = J;
};

// One pipeline step for block BLK of the current tile. kaddr / vaddr / paddr are this
// lane's LDS byte addresses into the K buffer that holds block BLK+1, the V buffer of the
// current tile and its kv_pos.
// Accumulator idx of S^T in lane (n, g) is key (idx/4)*8 + g*4 + idx%4 of the block and query
// n; slot jj of the lane's slice of P^T in MFMA kk is key kk*16 + (jj/4)*8 + g*4 + jj%4,
// which is the order in which the V^T fragments are fetched.
// `hook(IntC<M>)` runs after MFMA M (0 .. D/8 - 1) of the step: the caller spreads the requests
// for the next tile over these points.
template <int D, int BLK, bool BAND, typename Hook>
__device__ __forceinline__ void pipe_body(PipeRegs<D>& R, const bf16x8_t (&qf)[D / 16],
                                          const uint32_t (&kaddr)[D / 16],
                                          const uint32_t (&vaddr)[D / 32],
                                          uint32_t paddr, int32_t qp, int32_t ql,
                                          float scale_log2, bool need_mask, bool dead, bool& have_ref,
                                          Hook hook) {
  using G = Geo<D>;
  constexpr int CUR = BLK & 1, NXT = CUR ^ 1;
  constexpr int KOFF = ((BLK + 1) & 3) * G::BLK;
  constexpr int VOFF = BLK * G::BLK;
  constexpr int H = G::NKS;          // MFMAs per half step
  constexpr int POFF = BLK * 32 * 4;
  // exponentials started by vector slice 1 + k: values [kBound[k], kBound[k + 1]); they are
  // summed and packed one slice later (a transcendental result has a wait state)
  constexpr int kBound[15] = {0, 1, 2, 3, 5, 6, 7, 8, 9, 10, 11, 13, 14, 15, 16};

  floatx16_t& s = R.s[CUR];
  float e[16];
  float m_use = 0.f, alpha = 1.f;
  float lsum0 = 0.f, lsum1 = 0.f;
  bool raise = false;

  // Online softmax in the log2 domain, reference maximum m_run per row.
  // Fast form (nearly every block): no maximum at all. The exponentials are taken against the
  // standing reference, whatever the block holds; the reference is never above a score the row
  // has seen, so nothing underflows that should not, and a block whose exponentials sum to more
  // than kOverflowSum (a score 40 log2 units above the reference) is detected from its sum and
  // redone in the full form, for the rows concerned. A block that straddles a query position is
  // masked first (need_mask). One that no row of this wavefront can see (dead: the workgroup's
  // other wavefronts can) is taken against an infinite reference, i.e. as zeros; if that gives a NaN
  // (a score that is not finite) it is redone like the others, and masked there: in no form does a
  // score enter that its row must not see. (Masking it at once, 16 moves and a maximum a block, made
  // a wavefront of blind rows hold its workgroup back: 5000 queries, the later half seeing all of
  // 5000 keys, 114.5 -> 127 us.)
  // Full form (until every row of the wavefront has a reference): block maximum, and the
  // reference is raised when the maximum exceeds it by more than kRescaleSlack. O and l are
  // rescaled at the end of the step, after the MFMAs that still belong to the old reference. The
  // denominator sums the unrounded exponentials: LSE must be good to 1e-3 even on rows with a
  // handful of keys, which bf16 rounding of P would not give.
  auto block_max = [&]() __attribute__((always_inline)) -> float {
    float a = fmaxf(fmaxf(s[0], s[1]), s[2]);
    float b = fmaxf(fmaxf(s[3], s[4]), s[5]);
    float c = fmaxf(fmaxf(s[6], s[7]), s[8]);
    float d = fmaxf(fmaxf(s[9], s[10]), s[11]);
    a = fmaxf(fmaxf(a, s[12]), s[13]);
    b = fmaxf(fmaxf(b, s[14]), s[15]);
    const float mx = fmaxf(fmaxf(a, b), fmaxf(c, d));
    return fmaxf(mx, xor32(mx));
  };
  auto finish = [&](int v) __attribute__((always_inline)) {
    if (v & 1) {
      lsum1 += e[v];
      float a = e[v - 1], b = e[v];
#pragma unroll
      for (int t = 0; t < G::TERMS; ++t) {
        unsigned pk = pack_bf16(a, b);
        pin(pk);   // (here: the compiler otherwise converts a once more for its half of pk)
        if (t + 1 < G::TERMS) {   // what the term leaves over (exact)
          a -= __builtin_bit_cast(float, pk << 16);
          b -= __builtin_bit_cast(float, pk & 0xffff0000u);
        }
        R.pb[CUR][t][v >> 3][(v & 7) >> 1] = pk;
      }
      pin(lsum1);
    } else {
      lsum0 += e[v];
      pin(lsum0);
    }
  };

  auto valu = [&](auto jc) __attribute__((always_inline)) {
    constexpr int J = decltype(jc)::value;
    if constexpr (J == 0) {
      m_use = R.m_run;
      if (__builtin_expect(need_mask | !have_ref, 0)) {  // wave-uniform, rare: off the hot path
        if (dead) {
          m_use = INFINITY;
        } else {
          if (need_mask) {
            // The kv_pos reads are simply waited for (which also completes every older LDS read,
            // so the counted waits hold).
            u32x4_t kp0 = lds_read_b128<POFF + 0>(paddr), kp1 = lds_read_b128<POFF + 32>(paddr);
            u32x4_t kp2 = lds_read_b128<POFF + 64>(paddr), kp3 = lds_read_b128<POFF + 96>(paddr);
            lgkm_wait<0>(kp0, kp1, kp2, kp3);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int32_t k0 = (int32_t)kp0[r], k1 = (int32_t)kp1[r];
              const int32_t k2 = (int32_t)kp2[r], k3 = (int32_t)kp3[r];
              if (k0 > qp || (BAND && k0 < ql)) s[0 + r] = -INFINITY;
              if (k1 > qp || (BAND && k1 < ql)) s[4 + r] = -INFINITY;
              if (k2 > qp || (BAND && k2 < ql)) s[8 + r] = -INFINITY;
              if (k3 > qp || (BAND && k3 < ql)) s[12 + r] = -INFINITY;
            }
          }
          if (!have_ref) {
            const float m_step = block_max() * scale_log2;
            // true on the first visible block, also if its scores are NaN: such a row is lost, and
            // must not keep the others of its wavefront on the full form
            raise = !(m_step <= R.m_run + kRescaleSlack);
            const float m_new = raise ? m_step : R.m_run;
            alpha = __builtin_amdgcn_exp2f(R.m_run - (m_new == -INFINITY ? 0.f : m_new));
            R.l_run *= alpha;
            R.m_run = m_new;
            m_use = m_new == -INFINITY ? 0.f : m_new;
            have_ref = __builtin_amdgcn_ballot_w64(m_new == -INFINITY) == 0;
          }
        }
      }
      pin(m_use);
    } else {
      if constexpr (J <= 14) {
#pragma unroll
        for (int v = kBound[J - 1]; v < kBound[J]; ++v) {
          e[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale_log2, -m_use));
          pin(e[v]);
        }
      }
      if constexpr (J >= 2) {
#pragma unroll
        for (int v = kBound[J - 2]; v < kBound[J - 1]; ++v) finish(v);
      }
    }
  };

  // ---- first half: P(i-1) on the matrix pipe, K fragments of block i+1 requested ----
  auto first = [&](auto mc) __attribute__((always_inline)) {
    constexpr int M = decltype(mc)::value;
    if constexpr (M < H) {
      // LDS operations issued after V fragment M: H - 1 - M later V fragments (two reads each)
      // and M K fragments
      lgkm_wait<2 * (H - 1 - M) + M>(R.vf[M]);
      auto term = [&](auto tc) __attribute__((always_inline)) {
        constexpr int T = decltype(tc)::value;
        if constexpr (T < G::TERMS) {
          R.o[M % G::NDB] = mfma32(__builtin_bit_cast(bf16x8_t, R.vf[M]),
                                   __builtin_bit_cast(bf16x8_t, R.pb[NXT][T][M / G::NDB]),
                                   R.o[M % G::NDB]);
          if constexpr (T + 1 == G::TERMS) {
            R.kf[M] = lds_read_b128<KOFF>(kaddr[M]);
            hook(IntC<M>{});
          }
          valu(IntC<M * G::TERMS + T>{});
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      term(IntC<0>{}); term(IntC<1>{}); term(IntC<2>{});
    }
  };
  first(IntC<0>{}); first(IntC<1>{}); first(IntC<2>{}); first(IntC<3>{});
  first(IntC<4>{}); first(IntC<5>{}); first(IntC<6>{}); first(IntC<7>{});

  // ---- second half: Q(i+1) on the matrix pipe, V fragments of block i requested ----
  auto second = [&](auto mc) __attribute__((always_inline)) {
    constexpr int M = decltype(mc)::value;
    if constexpr (M < H) {
      // after K fragment M: H - 1 - M later K fragments and 2 M reads of V fragments
      lgkm_wait<H - 1 - M + 2 * M>(R.kf[M]);
      if constexpr (M == 0) {
        floatx16_t z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        R.s[NXT] = mfma32(__builtin_bit_cast(bf16x8_t, R.kf[M]), qf[M], z);
      } else {
        R.s[NXT] = mfma32(__builtin_bit_cast(bf16x8_t, R.kf[M]), qf[M], R.s[NXT]);
      }
      R.vf[M] = lds_read_vt_frag<VOFF + (M / G::NDB) * 16 * G::ROW, G::ROW>(vaddr[M % G::NDB]);
      hook(IntC<H + M>{});
      valu(IntC<H * G::TERMS + M>{});
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  second(IntC<0>{}); second(IntC<1>{}); second(IntC<2>{}); second(IntC<3>{});
  second(IntC<4>{}); second(IntC<5>{}); second(IntC<6>{}); second(IntC<7>{});

  // A block of the fast form whose exponentials ran away from the reference (rare): redo
  // its softmax in the full form, with a new reference for the rows that did and the same result
  // for the others. No row's sum can pass the test with an infinity or a NaN; a row whose
  // reference has become one is lost, and is not looked at again.
  float blk = lsum0 + lsum1;
  const bool over = !(blk <= kOverflowSum) && R.m_run < INFINITY;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(over) != 0, 0)) {
    const float over_f = over ? 1.f : 0.f;
    const bool row_over = over_f + xor32(over_f) > 0.f;   // in either half of the row's keys
    if (dead) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = -INFINITY;
    }
    const float m_step = block_max() * scale_log2;
    const float m_new = row_over ? fmaxf(R.m_run, m_step) : R.m_run;
    m_use = m_new == -INFINITY ? 0.f : m_new;
    const float a2 = __builtin_amdgcn_exp2f(R.m_run - m_use);
    R.l_run *= a2;
    alpha *= a2;
    R.m_run = m_new;
    raise = true;
    lsum0 = lsum1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      e[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale_log2, -m_use));
      finish(v);
    }
    blk = lsum0 + lsum1;
  }
  R.l_run += blk;
  // rows whose reference maximum moved: bring O to the new reference (rare)
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
#pragma unroll
    for (int db = 0; db < G::NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) R.o[db][i] *= alpha;
  }
  __builtin_amdgcn_sched_barrier(0);
}

// ---- arrival flags of the ring walk (RING): the bounded wait for a shard ----
__device__ __forceinline__ int ring_flag(const Params& p, int rank, int step) {
  return __hip_atomic_load(p.arrived[rank] + step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Makes sure that the shard of ring step `step` of rank `rank` may be read: `peek` is what thread
// 0 read of the step's flag while the previous shard was being walked (so a shard that arrived in
// time costs no round trip here); if that was zero it polls (uncached loads, a short sleep between
// them, at most p.spin_limit of them). The whole workgroup learns the outcome through LDS; false =
// the flag never came up: bit `step` of the rank's error word is set and the caller leaves the shard
// out. Every wait ends.
__device__ __forceinline__ bool ring_enter(const Params& p, int rank, int step, int tid,
                                           int* wg_scratch, int& peek) {
  int* const slot = wg_scratch + 20 + (step & 1);  // two slots: a wavefront may lag one step
  if (tid == 0) {
    int ok = 1;
    if (peek == 0) {
      int budget = p.spin_limit;
      while (ring_flag(p, rank, step) == 0) {
        if (--budget <= 0) {
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(32);
      }
    }
    if (!ok) atomicOr(p.ring_error + rank, 1 << step);  // which step gave up (n_shards <= 32)
    *slot = ok;
    // a look at the next step's flag, used when the walk gets there
    peek = step + 1 < p.n_shards ? ring_flag(p, rank, step + 1) : 0;
  }
  lds_barrier();
  const int ok = __builtin_amdgcn_readfirstlane(*slot);
  // The shard's K and V are read after its flag (its positions before: those are complete when the
  // call is enqueued, and the blocks to walk are chosen from them): every load is issued after this
  // barrier, which thread 0 reaches only with the flag's value in hand. No cache invalidation: the
  // caller gives every step a buffer of its own that is complete before its flag is set and
  // is not written again while the kernel runs, so no line of its K and V can be in a cache
  // before the flag is seen. (An agent-scope acquire here invalidates the XCD's L2 once per workgroup
  // and shard and costs 3.5 % of the walk.)
  return ok != 0;
}

// ---------------------------------------------------------------------------
// PLAN: equal shares for the workgroups.
//
// A causal prefill gives its row blocks walks of very different lengths (one tile to all of
// them), a packed batch even more so; with a workgroup per row block, or an equal number of
// splits for each, the longest walk sets the time (6229 tokens, 8 heads, 195 row blocks of up
// to 49 tiles: 204 us where the work is 70 us of all compute units). So the launch is 256
// workgroups (one per CU) that take equal shares of the whole work, cutting row blocks where a
// share ends. A unit is a row block of one KV head (against one shard, where shards are kept
// apart); its weight is an estimate of its visible steps plus kUnitCost for start-up and
// epilogue. Every workgroup works the plan out for itself, from kv_pos and q_pos, in LDS: that
// costs it 3 to 6 us (10 for packed prompts), less than the launches that would hand it over, and
// replaces the position-bound pre-pass. (Counting a unit's visible blocks exactly took up to 45 us at 700
// units and 350 blocks, so the weight comes from its first and last query and from at most 32
// blocks, 128 in a packed batch; a cut is made at the same fraction of the unit's true list of
// tiles.) What a share cuts goes to the workspace as fp32 partials (at most two per
// workgroup) and is merged by plan_merge_kernel. Those partials are up to 67 MB each way, as much
// time as 12 tile steps (6 at head_dim 64), so units of nearly equal length that fit one round are
// left whole (2100 queries of 16 heads that all see the same 1050 keys: 53 us cut, 41 whole; where
// half of them see 2100 and half none: 53 cut, 67 whole). Only for calls whose positions and unit list
// fit LDS; larger ones have row blocks enough to keep every CU busy. What bounds a share of short
// units are the latencies between the last tile of a unit and the first of the next, 9.9 us of packed
// prompts' 91: with the next rows asked for behind the epilogue, tables in LDS and the blocks counted
// and listed in one go 7.9, the call 109.4 -> 102.3 us, 4096 tokens at head_dim 64 59.3 -> 57.9.
// Six packed prompts of 200 to 3000 tokens over 4 ranks: 241 us with a workgroup per row block and
// 128-key tiles, 97 us in equal shares of 32-key blocks.
// ---------------------------------------------------------------------------

// Shares: workgroup i of W takes [share_begin(i), share_begin(i + 1)) of the line of all units
// (the host keeps total * 256 within 32 bits).
__device__ inline int plan_workgroups(uint32_t total, int own_start, int max_wgs) {
  const uint32_t w = total / (uint32_t)own_start;   // a share is worth its own start-up
  return (int)(w < 1 ? 1 : w > (uint32_t)max_wgs ? (uint32_t)max_wgs : w);
}
__device__ inline int share_begin(int i, uint32_t total, int n_wgs) {
  return (int)((uint32_t)i * total / (uint32_t)n_wgs);
}

// A pointer to global memory, said so: chosen in a branch or looked up in LDS it loses what the
// compiler knows of a kernel argument, and is accessed with flat instructions. Those count as LDS
// operations too, so that every later LDS read waits for memory (2000 cycles of an epilogue).
template <typename T>
using Glb = CP_GLB_AS T*;
// A kernel argument as a value of its own: where it is one of two that a branch chooses from, the
// compiler otherwise chooses between their addresses, and copies the arguments to scratch for it.
template <typename T>
__device__ __forceinline__ Glb<T> argument(T* x) {
  Glb<T> y = (Glb<T>)x;
  asm volatile("" : "+s"(y));
  return y;
}

struct Share {
  int unit;     // first unit
  int begin;    // begin of the share, counted from the begin of that unit
  int length;
};

// Shards, ranks and the shard of every block, as PLAN looks them up (in LDS: per lane, and of every
// unit, they would be chains of argument loads, 2 us of every start). Not filled for one rank or one
// shard.
struct LdsShard {
  const void* k;
  const void* v;
  const int32_t* kv_pos;
  int32_t n_kv, blk_begin;
};
struct LdsRank {
  const void* q;
  const int32_t* q_pos;
  void* out;
  float* lse;
};
struct PlanLds {
  LdsShard* shards;
  LdsRank* ranks;
  int32_t* tok_begin;     // kMaxTable + 1
  uint8_t* block_shard;
};

// x rotated by N within each row of 16 lanes.
template <int N>
__device__ __forceinline__ int row_ror(int x) {
  return __builtin_amdgcn_update_dpp(x, x, 0x120 + N, 0xf, 0xf, false);
}
__device__ __forceinline__ int row_max(int x) {  // over 16 lanes
  x = max(x, row_ror<8>(x));
  x = max(x, row_ror<4>(x));
  x = max(x, row_ror<2>(x));
  return max(x, row_ror<1>(x));
}
__device__ __forceinline__ int row_min(int x) {
  x = min(x, row_ror<8>(x));
  x = min(x, row_ror<4>(x));
  x = min(x, row_ror<2>(x));
  return min(x, row_ror<1>(x));
}
__device__ __forceinline__ int row_sum(int x) {
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  return x + row_ror<1>(x);
}
// Over the wavefront; the results are wave-uniform (scalar).
__device__ __forceinline__ int wave_max(int x) {
  x = row_max(x);
  return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ int wave_min(int x) {
  x = row_min(x);
  return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ int wave_sum(int x) {
  x = row_sum(x);
  return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) +
         __builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48);
}

// (min, max) of the positions of every 32-key block into LDS. Loads are issued many at a time:
// this is a chain of memory latencies, nothing else.
__device__ __forceinline__ void plan_bounds(const Params& p, int2* lds_bounds, const PlanLds& L,
                                            int tid) {
  // 8 threads per block, 4 positions per thread, up to 8 blocks per thread at a time
  constexpr int PER = 8, STEP = NTHREADS / 8;
  for (int b0 = 0; b0 < p.n_blocks; b0 += PER * STEP) {
    int32_t x[PER][4];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (b0 + u * STEP < p.n_blocks) {   // uniform
        const int b = min(b0 + u * STEP + (tid >> 3), p.n_blocks - 1);
        int first = 0, n_kv = p.n_kv;
        Glb<const int32_t> pos = argument(p.kv_pos);
        if (p.n_shards > 1) {
          const LdsShard& e = L.shards[L.block_shard[b]];
          first = e.blk_begin;
          n_kv = e.n_kv;
          pos = (Glb<const int32_t>)e.kv_pos;
        }
        const int key0 = (b - first) * BLOCK + (tid & 7);
#pragma unroll
        for (int i = 0; i < 4; ++i)   // (past the end: the last key again, same bounds)
          x[u][i] = pos[min(key0 + i * 8, n_kv - 1)];
      }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (b0 + u * STEP < p.n_blocks) {
        const int b = b0 + u * STEP + (tid >> 3);
        int lo = min(min(x[u][0], x[u][1]), min(x[u][2], x[u][3]));
        int hi = max(max(x[u][0], x[u][1]), max(x[u][2], x[u][3]));
#pragma unroll
        for (int o = 4; o > 0; o >>= 1) {
          lo = min(lo, __shfl_xor(lo, o, 64));
          hi = max(hi, __shfl_xor(hi, o, 64));
        }
        if ((tid & 7) == 0 && b < p.n_blocks) lds_bounds[b] = make_int2(lo, hi);
      }
    }
  }
}

// Bounds of all blocks, and this workgroup's share. `weight`: the units' planned tiles, `index`: which
// share this is (LDS).
template <int D, bool BAND>
__device__ __forceinline__ Share plan_share(const Params& p, int2* lds_bounds, uint16_t* weight,
                                            const PlanLds& L, int* index, int* wg_scratch,
                                            int tid) {
  // (in steps of kStep blocks)
  constexpr int kStep = Geo<D>::STEP_BLOCKS, kTile = 4 / kStep;
  const int lane = tid & 63, wave = tid >> 6;
  Share sh = {0, 0, 0};
  const int n_rb = p.n_row_blocks, n_units = n_rb * p.n_z;
  // Units of this thread (PER of them): their first and last query, and whose those are.
  constexpr int PER = PLAN_MAX_UNITS / NTHREADS;
  int tok[PER][2], of[PER][2] = {};
  if (p.n_ranks > 1 || p.n_shards > 1) {
    if (tid >= 64 && tid < 64 + p.n_shards) {
      const int i = tid - 64;
      L.shards[i] = {p.t.k[i], p.t.v[i], p.t.kv_pos[i], p.t.n_kv[i], p.t.blk_begin[i]};
    }
    if (tid >= 128 && tid < 128 + p.n_ranks) {
      const int i = tid - 128;
      L.ranks[i] = {p.t.q[i], p.t.q_pos[i], p.t.out[i], p.t.lse[i]};
    }
    if (tid >= 192 && tid <= 192 + p.n_ranks) L.tok_begin[tid - 192] = p.t.tok_begin[tid - 192];
    if (p.n_shards > 1) {
      for (int b = tid; b < p.n_blocks; b += NTHREADS) {
        int sh = 0;
#pragma unroll 8
        for (int i = 1; i < p.n_shards; ++i) sh += b >= p.t.blk_begin[i];
        L.block_shard[b] = (uint8_t)sh;
      }
    }
  }
  if (p.cut_units) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int u = min(k * NTHREADS + tid, n_units - 1);
      const int rb = u - (p.n_z > 1 ? u / n_rb : 0) * n_rb;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t row = (uint32_t)rb * BM;
        tok[k][e] = (int)((e == 0 ? row : min(row + BM, (uint32_t)p.rows) - 1) / (uint32_t)p.group);
      }
    }
#pragma unroll 8
    for (int i = 1; i < p.n_ranks; ++i) {
      const int begin = p.t.tok_begin[i];
#pragma unroll
      for (int k = 0; k < PER; ++k)
#pragma unroll
        for (int e = 0; e < 2; ++e) of[k][e] += tok[k][e] >= begin;
    }
  }
  if (p.n_ranks > 1 || p.n_shards > 1) __syncthreads();
  if (!p.cut_units) {  // a workgroup per unit
    plan_bounds(p, lds_bounds, L, tid);
    __syncthreads();
    const int i = blockIdx.x / p.n_kv_heads, kvh = blockIdx.x - i * p.n_kv_heads;
    const int z = p.n_z > 1 ? i / p.n_row_blocks : 0;
    const int rb = ordered_row_block(i - z * p.n_row_blocks, p.n_row_blocks, p.n_ranks, lane,
                                     p.chunks, BM);
    sh.unit = (kvh * p.n_z + z) * p.n_row_blocks + rb;
    return sh;
  }
  // Position range of every row block as its first and its last query have it, requested before the
  // key positions.
  int mx[PER], lo[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    mx[k] = INT32_MIN;
    lo[k] = INT32_MAX;
    if (k * NTHREADS < n_units) {  // uniform
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int t = tok[k][e], a = of[k][e];
        const int32_t x = p.n_ranks > 1 ? ((Glb<const int32_t>)L.ranks[a].q_pos)[t - L.tok_begin[a]]
                                        : ((Glb<const int32_t>)p.q_pos)[t];
        mx[k] = max(mx[k], x);
        if (BAND) lo[k] = min(lo[k], x >= 0 ? p.q_lo[t] : INT32_MAX);
      }
    }
  }
  // A row block that can hold a whole chunk, a late one between two early ones, has its longest walk at
  // neither end: two more queries of it. (Taken for short, such units were one share's, which walked them
  // whole, and a cut at half tiles made some longer still. 8 heads on 8 KV heads over 8 ranks, us, in whole
  // tiles, half tiles and so: 1660 tokens 74.1, 82.9 and 40.7, 2843 110.8, 114.7 and 57.7, 900 51.0, 49.3
  // and 37.7. At head_dim 64 only: it keeps all bits wherever units are cut.)
  if (D == 64 && p.n_ranks > 1 && p.chunks.early < BM) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (k * NTHREADS < n_units) {
        int t[2], a[2] = {0, 0};
#pragma unroll
        for (int e = 0; e < 2; ++e) t[e] = tok[k][0] + (tok[k][1] - tok[k][0]) * (e + 1) / 3;
#pragma unroll 8
        for (int i = 1; i < p.n_ranks; ++i) {
          const int begin = p.t.tok_begin[i];
          a[0] += t[0] >= begin;
          a[1] += t[1] >= begin;
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
          mx[k] = max(mx[k], ((Glb<const int32_t>)L.ranks[a[e]].q_pos)[t[e] - L.tok_begin[a[e]]]);
      }
    }
  }
  plan_bounds(p, lds_bounds, L, tid);
  __syncthreads();
  // Planned tiles: every stride-th block of the range looked at (more of them in a packed batch,
  // where a row block sees few).
  constexpr int SAMPLES = BAND ? 128 : 32;
  const int avg = (p.n_blocks + p.n_z - 1) / p.n_z, stride = (avg + SAMPLES - 1) / SAMPLES;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NTHREADS < n_units) {
      const int u = min(k * NTHREADS + tid, n_units - 1);
      const int z = p.n_z > 1 ? u / n_rb : 0;
      const int b0 = p.n_z > 1 ? L.shards[z].blk_begin : 0;
      const int b1 = p.n_z > 1 ? (z + 1 < p.n_z ? L.shards[z + 1].blk_begin : p.n_blocks) : p.n_blocks;
      int cnt = 0, b = b0;
      // (no test of the range in the groups that lie in it: 10 vector instructions a sample were 4.4 us
      // of a packed call's start, for 98 samples)
      for (; b + 7 * stride < b1; b += 8 * stride) {
        int2 x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = lds_bounds[b + i * stride];
#pragma unroll
        for (int i = 0; i < 8; ++i) cnt += x[i].x <= mx[k] && (!BAND || x[i].y >= lo[k]) ? 1 : 0;
      }
      for (; b < b1; b += stride) {
        const int2 x = lds_bounds[b];
        cnt += x.x <= mx[k] && (!BAND || x.y >= lo[k]) ? 1 : 0;
      }
      weight[u] = (uint16_t)max(1, (cnt * stride + kStep - 1) / kStep);
    }
  }
  __syncthreads();
  // prefix sums
  int x[PER], sum = 0, most = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = tid * PER + i;
    const int c = u < n_units ? kUnitCost + (int)weight[u] : 0;
    most = max(most, c);
    sum += c;
    x[i] = sum;
  }
  most = wave_max(most);
  int scan = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(scan, o, 64);
    if (lane >= o) scan += y;
  }
  if (lane == 63) {
    wg_scratch[wave] = scan;
    wg_scratch[NWAVE + wave] = most;
  }
  __syncthreads();
  int before = scan - sum, total1 = 0, longest = 0;
#pragma unroll
  for (int w = 0; w < NWAVE; ++w) {
    const int c = wg_scratch[w];
    if (w < wave) before += c;
    total1 += c;
    longest = max(longest, wg_scratch[NWAVE + w]);
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) x[i] += before;
  total1 = __builtin_amdgcn_readfirstlane(total1);
  longest = __builtin_amdgcn_readfirstlane(longest);
  // the line of units, KV head after KV head
  const uint32_t total = (uint32_t)total1 * (uint32_t)p.n_kv_heads;
  const int all = n_units * p.n_kv_heads;
  // Whole units where a cut gains less than its partials cost: one round of workgroups, and the
  // longest unit not much longer than a share.
  const bool keep_whole = all <= (int)gridDim.x &&
                          longest <= (int)(total / gridDim.x) + kCutCost * (D / 64) * kTile / 2;
  const int n_wgs = keep_whole ? all : plan_workgroups(total, kUnitCost + 2 * kTile, gridDim.x);
  // (workgroups go to the 8 XCDs in turn; only if every XCD gets its part of the shares)
  const int i = n_wgs == kPlanWorkgroups && shares_grouped(D, all)
                    ? (int)(blockIdx.x & 7) * (kPlanWorkgroups / 8) + (int)(blockIdx.x >> 3)
                    : (int)blockIdx.x;
  if (tid == 0) *index = i;
  if (i >= n_wgs) {
    if (tid == 0) p.plan_rec[i + 1] = make_int2(-1, 0);
    return sh;
  }
  if (keep_whole) {
    sh.unit = i;
    sh.length = kUnitCost + __builtin_amdgcn_readfirstlane((int)weight[i % n_units]);
    if (tid == 0) {
      p.plan_rec[i] = make_int2(i, 0);
      if (i == n_wgs - 1) p.plan_rec[n_wgs] = make_int2(-1, 0);
    }
    return sh;
  }
  // A boundary in the start-up of a unit moves to its begin: nothing is cut there. (Moving those
  // near an end as well, to save the cut, made the calls of short units up to 30 % slower: the
  // shares are short, too.)
  const int s_end[2] = {share_begin(i, total, n_wgs), share_begin(i + 1, total, n_wgs)};
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int kvh = min((int)((uint32_t)s_end[e] / (uint32_t)total1), p.n_kv_heads - 1);
    const int in_head = s_end[e] - kvh * total1;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int u = tid * PER + k;
      const int first = k == 0 ? before : x[k - 1];
      // (the end of the line belongs to the last unit)
      if (u < n_units && first <= in_head &&
          (in_head < x[k] || (u == n_units - 1 && in_head == x[k]))) {
        int unit = kvh * n_units + u, off = in_head - first;
        if (off <= kUnitCost) off = 0;
        else if (in_head == x[k]) { unit += 1; off = 0; }
        wg_scratch[16 + 4 * e] = unit;
        wg_scratch[17 + 4 * e] = off;
        wg_scratch[18 + 4 * e] = kvh * total1 + (unit == kvh * n_units + u ? first + off : x[k]);
        // for the merge: unit, begin of the share in it
        if (e == 0) p.plan_rec[i] = make_int2(unit, off);
        else if (i == n_wgs - 1) p.plan_rec[n_wgs] = make_int2(-1, 0);
      }
    }
  }
  __syncthreads();
  sh.unit = __builtin_amdgcn_readfirstlane(wg_scratch[16]);
  sh.begin = __builtin_amdgcn_readfirstlane(wg_scratch[17]);
  sh.length = __builtin_amdgcn_readfirstlane(wg_scratch[22] - wg_scratch[18]);
  return sh;
}

// How a launch deals out its work.
enum Mode {
  WHOLE,  // a workgroup per row block (and shard, where shards are kept apart)
  SPLIT,  // grid.z parts of the KV axis per row block, fp32 partials in the workspace
  PLAN,   // equal shares of everything (above)
  ACC,    // WHOLE, merged into a running (O, LSE) in the epilogue (Equation 4 step by step)
  RING    // WHOLE, the shards walked one by one in ring order, each behind its arrival flag
          // (bounded wait), with one running (O, l, m) in registers: the merge of Equation 4
          // happens inside the online softmax
};

// A workgroup's walk: 256 consecutive (token, head-in-group) rows of one KV head, over the
// queries of all ranks of the table back to back, against the visible blocks of the KV shards.
// BAND: packed batch. Positions are shifted per sequence and a query also has a lower bound
// q_lo (the shift of its sequence): visible iff q_lo <= kv_pos <= q_pos.
template <int D, typename TO, bool BAND, Mode MODE>
__device__ __forceinline__ void prefill_body(const Params& p) {
  using G = Geo<D>;
  constexpr int ROW = G::ROW;
  extern __shared__ __align__(16) char smem[];
  char* const kbuf0 = smem;
  char* const vbuf0 = smem + G::OFF_V;
  int32_t* const posbuf0 = (int32_t*)(smem + G::OFF_POS);
  int* const wg_scratch = (int*)(smem + G::OFF_SCRATCH);
  int4* const live = (int4*)(smem + G::OFF_LIVE);            // addresses of K and V (below)
  int2* const live_pos = (int2*)(smem + G::OFF_LIVE_POS);    // address of kv_pos, keys above it
  int2* const live_range = (int2*)(smem + G::OFF_LIVE_RANGE);  // (min, max) of kv_pos
  int2* const lds_bounds = (int2*)(smem + G::OFF_BOUNDS);
  uint16_t* const weight = (uint16_t*)(smem + G::OFF_WEIGHT);
  const PlanLds L = {(LdsShard*)(smem + G::OFF_SHARDS), (LdsRank*)(smem + G::OFF_RANKS),
                     (int32_t*)(smem + G::OFF_RANK_TOK), (uint8_t*)(smem + G::OFF_BLOCK_SHARD)};
  int* const share_index = (int*)(smem + G::OFF_INDEX);
  const uint32_t smem_lds = (uint32_t)(size_t)(CP_LDS_AS char*)smem;

  const int touched = touch_arguments<Params>();
  // ---- what this workgroup does first ----
  int row_block = 0, kvh = 0, z_shard = 0, z_sub = 0, rank = 0;
  Share share = {0, 0, 0};
  if constexpr (MODE == PLAN) {
    share = plan_share<D, BAND>(p, lds_bounds, weight, L, share_index, wg_scratch, threadIdx.x);
    if (p.cut_units && share.length == 0) return;
    const int units = p.n_row_blocks * p.n_z;
    kvh = share.unit / units;
    const int u = share.unit - kvh * units;
    z_shard = p.n_z > 1 ? u / p.n_row_blocks : 0;
    row_block = u - z_shard * p.n_row_blocks;
    asm volatile("" ::"v"(touched));
    lds_barrier();   // the plan's scratch is read
  } else {
    // The KV heads of a row block are neighbours in dispatch order: the rows of one head are
    // n_kv_heads * 2 D bytes apart, so workgroups that all read the same head use only some of
    // the memory channels.
    // grid.z: the n_sub parts of the KV axis, of every shard in turn when shards are kept apart
    int x = blockIdx.x, z = blockIdx.z;
    if constexpr (MODE == WHOLE || MODE == SPLIT) {
      if (p.xcd_slice) {
        const GridPos at = xcd_slice(x, z, gridDim.x, gridDim.z);
        x = at.x;
        z = at.z;
      }
    }
    const int i = x / p.n_kv_heads;
    kvh = x - i * p.n_kv_heads;
    row_block = ordered_row_block(i, p.n_row_blocks, p.n_ranks, threadIdx.x & 63, p.chunks,
                                  MODE == RING ? 1 : BM);
    z_shard = p.per_shard ? z / p.n_sub : 0;
    z_sub = z - z_shard * p.n_sub;
    if constexpr (MODE == RING) {   // row blocks do not straddle ranks here
      while (p.rb_begin[rank + 1] <= row_block) ++rank;
      row_block -= p.rb_begin[rank];
    }
  }

  // Rank of the query `token` of a lane's row, in a row block whose first query is t0 (PLAN, several
  // ranks): most row blocks lie within one.
  auto planned_rank = [&](int t0, int token, int lane) __attribute__((always_inline)) -> int {
    const int begin = L.tok_begin[min(lane, p.n_ranks)];
    int a = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < p.n_ranks && t0 >= begin)) - 1;
    if (__builtin_amdgcn_ballot_w64(token >= __builtin_amdgcn_readlane(begin, a + 1)) != 0)
      while (token >= L.tok_begin[a + 1]) ++a;
    return a;
  };
  // Asks for what this lane needs of its query row in row block `rb`: position, lower bound, Q
  // fragments. A row past the end takes the last one's (it is known by its index), so that nothing is
  // waited for here: loads under a condition were, 1.2 us of every epilogue that makes them.
  auto request_rows = [&](int rb, int head, int n_rows, int tid, int32_t& qp, int32_t& ql,
                          u32x4_t (&qf)[G::NKS]) __attribute__((always_inline)) {
    const int lane = tid & 63, g = lane >> 5;
    const int r = min(rb * BM + (__builtin_amdgcn_readfirstlane(tid >> 6)) * 32 + (lane & 31), n_rows - 1);
    int token = (int)((uint32_t)r / (uint32_t)p.group);
    const int hg = r - token * p.group;
    auto q = (Glb<const bf16_t>)argument(MODE == RING ? p.t.q[rank] : p.q);
    auto q_pos = argument(MODE == RING ? p.t.q_pos[rank] : p.q_pos);
    const int packed_token = token;
    if (MODE != RING && p.n_ranks > 1) {
      const int t0 = (int)((uint32_t)(rb * BM) / (uint32_t)p.group);
      if constexpr (MODE == PLAN) {
        const int a = planned_rank(t0, token, lane);
        q = (Glb<const bf16_t>)L.ranks[a].q;
        q_pos = (Glb<const int32_t>)L.ranks[a].q_pos;
        token -= L.tok_begin[a];
      } else {
        // (scalar loads where the row block lies within one rank, which it mostly does)
        const int a0 = rank_of_token(p.t, t0);
        q = (Glb<const bf16_t>)p.t.q[a0];
        q_pos = (Glb<const int32_t>)p.t.q_pos[a0];
        int first = p.t.tok_begin[a0];
        if ((int64_t)rb * BM + BM > (int64_t)p.t.tok_begin[a0 + 1] * p.group) {
          const int a = rank_of_token(p.t, token);
          q = (Glb<const bf16_t>)p.t.q[a];
          q_pos = (Glb<const int32_t>)p.t.q_pos[a];
          first = p.t.tok_begin[a];
        }
        token -= first;
      }
    }
    q += (((int64_t)token * p.n_kv_heads + head) * p.group + hg) * D + g * 8;
    qp = q_pos[token];
    ql = BAND ? p.q_lo[packed_token] : INT32_MIN;
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks) qf[ks] = *(Glb<const u32x4_t>)(q + ks * 16);
  };
  int32_t next_qp = 0, next_ql = 0;   // of the next unit's rows (PLAN: behind the epilogue of this one)
  u32x4_t next_qf[G::NKS];
  bool rows_requested = false;

  for (;;) {  // (PLAN: the units of the share, else once)
    // (The thread index is made opaque here: what is computed from it would otherwise be kept in
    // registers across the units, of which there are none to spare.)
    int tid = threadIdx.x;
    if constexpr (MODE == PLAN) asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n = lane & 31, g = lane >> 5;
    // ---- blocks of this workgroup (the ring walk moves on from shard to shard) ----
    int cur_shard = MODE == RING ? rank : z_shard;
    const bool one_shard = MODE == RING || p.per_shard;
    int b_begin = one_shard && p.n_shards > 1 ? p.t.blk_begin[cur_shard] : 0;
    int b_end = one_shard && p.n_shards > 1 ? p.t.blk_begin[cur_shard + 1] : p.n_blocks;
    if (MODE == SPLIT && p.sub_blocks > 0) {
      b_begin = z_sub * p.sub_blocks;
      b_end = min(b_end, b_begin + p.sub_blocks);
    }
    auto block_bounds = [&](int b) -> int2 {
      return MODE == PLAN ? lds_bounds[b] : p.bounds[b >> p.bounds_shift];
    };

    // ---- this lane's query row ----
    // (rows and row blocks of 256 fit 31 bits: checked by the launcher)
    const int n_rows = MODE == RING ? (p.t.tok_begin[rank + 1] - p.t.tok_begin[rank]) * p.group
                                    : p.rows;
    const int r0 = row_block * BM + wave * 32;   // of the wavefront
    const bool row_ok = (uint32_t)(r0 + n) < (uint32_t)n_rows;
    // The start-up chain is q_pos -> visible blocks -> first tile; the bounds of the first 512
    // blocks are requested now so that they arrive together with q_pos, and the Q fragments
    // (needed last) are requested after both and waited for only before the first product.
    int2 first_bounds = make_int2(0, 0);
    if (b_begin + tid < b_end) first_bounds = block_bounds(b_begin + tid);
    if (MODE != PLAN || !rows_requested)
      request_rows(row_block, kvh, n_rows, tid, next_qp, next_ql, next_qf);
    const int32_t qp = row_ok ? next_qp : CP_POS_PAD_Q, ql = row_ok ? next_ql : INT32_MIN;
    bf16x8_t qf[G::NKS];
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8_t, next_qf[ks]);
    const float scale_log2 = p.scale_log2;

    if constexpr (MODE != PLAN) asm volatile("" ::"v"(touched));
    // ---- query position range of the wavefront and of the workgroup ----
    // rows that can see anything: a padded query (CP_POS_PAD_Q) and the rows past the end of
    // the shard cannot, and stay out of the ranges below
    // (head_dim 64: any position but the padding's, as on the vector kernel)
    const bool sees = row_ok && (D == 64 ? qp != CP_POS_PAD_Q : qp >= 0);
    const int w_qmin = wave_min(sees ? qp : INT32_MAX), w_qmax = wave_max(qp);
    const int w_lomin = BAND ? wave_min(sees ? ql : INT32_MAX) : 0;
    const int w_lomax = BAND ? wave_max(sees ? ql : INT32_MIN) : 0;
    if (lane == 0) {
      wg_scratch[wave] = w_qmax;
      if (BAND) wg_scratch[NWAVE + 1 + wave] = w_lomin;
    }
    lds_barrier();
    int wg_qmax = INT32_MIN, wg_lomin = INT32_MAX;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) {
      wg_qmax = max(wg_qmax, wg_scratch[w]);
      if (BAND) wg_lomin = min(wg_lomin, wg_scratch[NWAVE + 1 + w]);
    }
    // wave-uniform by construction; say so, so that control flow stays on the scalar unit
    wg_qmax = __builtin_amdgcn_readfirstlane(wg_qmax);
    if (BAND) wg_lomin = __builtin_amdgcn_readfirstlane(wg_lomin);

    bool have_ref = false;  // every row of the wavefront has a finite reference maximum
    PipeRegs<D> R;
    // Reference max of scaled scores (log2 domain). A row that can see nothing gets a reference
    // no score reaches: its exponentials are all zero whichever softmax form its
    // wavefront takes (so one padded row does not keep the other 31 on the masked form), or NaN if
    // its query is not finite, which nothing says of a padded one. The epilogue writes O = 0,
    // LSE = -inf for it.
    R.m_run = sees ? -INFINITY : kDeadRowRef;
    R.l_run = 0.f;        // running denominator over this lane's half of the keys
#pragma unroll
    for (int db = 0; db < G::NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) R.o[db][i] = 0.f;

    // ---- tile loader: this wavefront brings rows (wave & 1) * 16 .. + 15 of the tile's block
    // wave / 2, of K and of V, 1 KiB (LOAD_ROWS rows) per instruction; lane l covers row
    // l / CHUNKS of them, chunk position l % CHUNKS. Part I of a tile is one such instruction
    // for K and one for V. Rows past the end of the shard are clamped to its last row (they are
    // masked by their position).
    const uint32_t stride_b = (uint32_t)p.n_kv_heads * ROW;  // bytes between tokens
    const int l_row = lane / G::CHUNKS, l_pos = lane % G::CHUNKS;
    struct Tile {          // (wave-uniform)
      const char* k;       // this wavefront's block
      const char* v;
      int last;            // its last valid row
      int mask;            // bit b: block b has a key that is hidden from one of this
                           // wavefront's rows; bit 4 + b: from all of them
    };
    auto issue_part = [&](auto ic, const Tile& t, int b) __attribute__((always_inline)) {
      constexpr int I = decltype(ic)::value;
      if constexpr (I < G::PARTS) {
        const int pr = I * G::LOAD_ROWS + l_row;  // row % 16 selects the permutation
        const int row = (wave & 1) * 16 + pr;
        const uint32_t roff = __umul24((uint32_t)min(row, t.last), stride_b);
        load_lds16(t.k + (roff + ((l_pos ^ G::k_perm(pr)) * 16)),
                   kbuf0 + b * G::KD + (wave * 16 + I * G::LOAD_ROWS) * ROW);
        load_lds16(t.v + (roff + ((l_pos ^ G::v_perm(pr)) * 16)),
                   vbuf0 + b * G::KD + (wave * 16 + I * G::LOAD_ROWS) * ROW);
      }
    };

    // ---- fragment addressing (LDS byte addresses, buffer 0) ----
    // K: lane (n, g) reads chunk 2*ks + g of key row n of a block
    uint32_t kaddr[G::NKS];
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks)
      kaddr[ks] = smem_lds + n * ROW + ((2 * ks + g) ^ G::k_perm(n)) * 16;
    // V: in its 16-lane group this lane addresses key vj of four and 8 bytes (4 channels) vq
    const int grp = lane >> 4, vj = (lane & 15) >> 2, vq = lane & 3;
    uint32_t vaddr[G::NDB];
#pragma unroll
    for (int db = 0; db < G::NDB; ++db)
      vaddr[db] = smem_lds + G::OFF_V + ((grp >> 1) * 4 + vj) * ROW +
                  (((db * 4 + (grp & 1) * 2 + (vq >> 1)) ^ G::v_perm(vj)) * 16) + (vq & 1) * 8;
    uint32_t paddr = smem_lds + G::OFF_POS + g * 16;

    auto visible = [&](const int2& b) -> bool {
      return b.x <= wg_qmax && (!BAND || b.y >= wg_lomin);
    };
    // The part of the list of visible blocks that is walked here: [part_lo, part_hi). Parts are
    // whole steps of the list.
    int part_lo = 0, part_hi = INT32_MAX;
    bool whole = true, first_piece = true;  // PLAN: the unit is not cut; its first piece
    // (the visible ones of the first chunk, counted here, are listed from the same count below)
    uint64_t first_mask = 0;
    int first_base = 0, first_total = 0;
    if constexpr (MODE == SPLIT || MODE == PLAN) {
      int total = 0;
      const bool more = (MODE == SPLIT ? p.sub_blocks == 0 : p.cut_units != 0) &&
                        b_end - b_begin > NTHREADS;   // chunks to count
      int cnt = 0;
      if (more) {
        for (int b = b_begin + NTHREADS + tid; b < b_end; b += NTHREADS)
          cnt += visible(block_bounds(b)) ? 1 : 0;
        cnt = wave_sum(cnt);
      }
      first_mask = __builtin_amdgcn_ballot_w64(b_begin + tid < b_end && visible(first_bounds));
      int* const counts = wg_scratch + 24;
      if (lane == 0) {
        counts[wave] = __builtin_popcountll(first_mask);
        counts[NWAVE + wave] = cnt;
      }
      lds_barrier();
#pragma unroll
      for (int w = 0; w < NWAVE; ++w) {
        const int c = counts[w];
        if (w < wave) first_base += c;
        first_total += c;
        total += counts[NWAVE + w];
      }
      first_total = __builtin_amdgcn_readfirstlane(first_total);
      total = __builtin_amdgcn_readfirstlane(total) + first_total;
      if constexpr (MODE == SPLIT) {
        if (p.sub_blocks == 0) {
          // (in 32 bits: a memory full of keys has some 2^24 steps, and CP_MAX_PARTS is 64; a 64-bit
          // division is 500 cycles of every start)
          constexpr int kStep = G::STEP_BLOCKS;
          const uint32_t steps = (uint32_t)(total + kStep - 1) / kStep;
          part_lo = kStep * (int)(steps * (uint32_t)z_sub / (uint32_t)p.n_sub);
          part_hi = kStep * (int)(steps * (uint32_t)(z_sub + 1) / (uint32_t)p.n_sub);
        }
      } else if (p.cut_units) {
        const int planned =
            __builtin_amdgcn_readfirstlane((int)weight[z_shard * p.n_row_blocks + row_block]);
        const int end = min(kUnitCost + planned, share.begin + share.length);
        const int lo = max(0, share.begin - kUnitCost), hi = end - kUnitCost;
        share.length -= end - share.begin;
        if (hi <= lo) return;  // the share ends within the unit's start-up
        whole = lo == 0 && hi == planned;
        first_piece = lo == 0;
        constexpr int kStep = G::STEP_BLOCKS;
        const int steps = (total + kStep - 1) / kStep;   // (pieces can come out empty: they are written as such)
        part_lo = kStep * (int)((uint32_t)(steps * lo) / (uint32_t)planned);
        part_hi = kStep * (int)((uint32_t)(steps * hi) / (uint32_t)planned);
      }
    }

    int flag_peek = 0;
    const int n_steps = MODE == RING ? p.n_shards : 1;
    for (int step = 0; step < n_steps; ++step) {
      if constexpr (MODE == RING) {
        if (step > 0) {
          cur_shard = cur_shard > 0 ? cur_shard - 1 : p.n_shards - 1;
          b_begin = p.t.blk_begin[cur_shard];
          b_end = p.t.blk_begin[cur_shard + 1];
        }
        if (!ring_enter(p, rank, step, tid, wg_scratch, flag_peek))
          continue;  // the shard never arrived: reported through ring_error, walk goes on
      }
      int seen = 0;  // visible blocks before this chunk of the range
      for (int c0 = b_begin; c0 < b_end; c0 += MAX_LIVE) {
        // Compact the blocks some query of the workgroup can see (smallest key position not
        // beyond the largest query position) into an ascending list in LDS.
        int n_live;       // tiles
        bool half_tail;   // the last one has two blocks at most
        {
          const int b = c0 + tid;
          int2 bb = first_bounds;
          bool lv;
          uint64_t mask;
          int base = 0, total = 0;
          if ((MODE == SPLIT || MODE == PLAN) && c0 == b_begin) {
            lv = (first_mask >> lane & 1) != 0;
            mask = first_mask;
            base = first_base;
            total = first_total;
          } else {
            lds_barrier();  // previous chunk (list, tile buffers) fully consumed
            lv = false;
            if (b < b_end) {
              if (c0 != b_begin || step != 0) bb = block_bounds(b);
              lv = visible(bb);
            }
            mask = __builtin_amdgcn_ballot_w64(lv);
            if (lane == 0) wg_scratch[wave] = __builtin_popcountll(mask);
            lds_barrier();
#pragma unroll
            for (int w = 0; w < NWAVE; ++w) {
              const int c = wg_scratch[w];
              if (w < wave) base += c;
              total += c;
            }
            total = __builtin_amdgcn_readfirstlane(total);
          }
          const int lo = max(part_lo, seen), hi = min(part_hi, seen + total);
          const int idx = seen + base + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
          if (lv && idx >= lo && idx < hi) {
            // (the shard through scalar loads where there is one; a lookup per lane is a memory
            // latency more)
            LdsShard e;
            if (p.n_shards == 1) {
              e = {(const void*)argument(p.k), (const void*)argument(p.v),
                   (const int32_t*)argument(p.kv_pos), p.n_kv, 0};
            } else if (MODE != PLAN && one_shard) {
              e = {p.t.k[cur_shard], p.t.v[cur_shard], p.t.kv_pos[cur_shard],
                   p.t.n_kv[cur_shard], p.t.blk_begin[cur_shard]};
            } else {
              int sh = cur_shard;
              if constexpr (MODE == PLAN) {
                if (!one_shard) sh = L.block_shard[b];
                e = L.shards[sh];
              } else {
#pragma unroll 8
                for (int i = 1; i < p.n_shards; ++i) sh += b >= p.t.blk_begin[i];
                e = {p.t.k[sh], p.t.v[sh], p.t.kv_pos[sh], p.t.n_kv[sh], p.t.blk_begin[sh]};
              }
            }
            const int key0 = (b - e.blk_begin) * BLOCK;
            const int valid = min(BLOCK, e.n_kv - key0);
            const uint64_t off = (uint64_t)key0 * stride_b + (uint32_t)kvh * ROW;
            const uint64_t ka = (uint64_t)e.k + off, va = (uint64_t)e.v + off;
            const uint64_t pa = (uint64_t)(e.kv_pos + key0);
            // (the last valid row travels in the upper 16 bits of V's address, which are zero, and the
            // count of keys in those of their positions')
            const int4 kv = make_int4((int)ka, (int)(ka >> 32), (int)va,
                                      (int)(va >> 32) | (valid - 1) << 16);
            live[idx - lo] = kv;
            live_pos[idx - lo] = make_int2((int)pa, (int)(pa >> 32) | valid << 16);
            // (a ragged block always pays for the mask: its largest position is the pad's)
            live_range[idx - lo] = make_int2(bb.x, valid < BLOCK ? INT32_MAX : bb.y);
            if (idx == hi - 1) {  // fill the last tile with blocks of no keys
              for (int i = idx - lo + 1; (i & 3) != 0; ++i) {
                live[i] = kv;
                live_pos[i] = make_int2((int)pa, (int)(pa >> 32));
                live_range[i] = make_int2(INT32_MAX, INT32_MAX);
              }
            }
          }
          seen += total;
          n_live = (max(0, hi - lo) + 3) >> 2;
          half_tail = (uint32_t)(hi - lo - 1) % 4 < 2;
        }
        lds_barrier();
        if (n_live == 0) continue;

        // ---- prologue: tile 0 into buffer 0, Q stage of block 0 ----
        // (kv_pos of a tile goes through a register: the tail needs the pad value)
        int32_t next_pos = 0;
        auto read_entry = [&](int idx, Tile& t) {
          const int i = (idx < n_live ? idx : n_live - 1) * 4;
          const int4 kv = live[i + (wave >> 1)];
          const int2 range = live_range[i + (lane & 3)];
          auto uni = [](int x) { return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(x); };
          t.k = (const char*)(uni(kv.x) | uni(kv.y) << 32);
          const int v_hi = __builtin_amdgcn_readfirstlane(kv.w);
          t.v = (const char*)(uni(kv.z) | (uint64_t)(uint32_t)(v_hi & 0xffff) << 32);
          t.last = (int)((uint32_t)v_hi >> 16);
          bool m = range.y > w_qmin, none = range.x > w_qmax;
          if (BAND) {
            m |= range.x < w_lomax;
            none |= range.y < w_lomin;
          }
          const int mm = (int)(__builtin_amdgcn_ballot_w64(m) & 15);
          t.mask = mm | ((int)__builtin_amdgcn_ballot_w64(none) & mm) << 4;
          if (wave < TILE / 64) {   // kv_pos of the key tid
            const int2 own = live_pos[i + (tid >> 5)];
            next_pos = CP_POS_PAD_KV;
            if ((tid & 31) < (int)((uint32_t)own.y >> 16)) {
              const auto pos = (Glb<const int32_t>)((uint64_t)(uint32_t)own.x |
                                                    (uint64_t)(uint32_t)(own.y & 0xffff) << 32);
              next_pos = pos[tid & 31];
            }
          }
        };
        Tile next;
        int mask;
        {
          Tile t0;
          read_entry(0, t0);
          mask = t0.mask;
          issue_part(IntC<0>{}, t0, 0);
          issue_part(IntC<1>{}, t0, 0);
          issue_part(IntC<2>{}, t0, 0);
          issue_part(IntC<3>{}, t0, 0);
          if (tid < TILE) posbuf0[tid] = next_pos;
          __syncthreads();  // waits for the tile (vmcnt) and publishes it
          read_entry(1, next);
#pragma unroll
          for (int ks = 0; ks < G::NKS; ++ks) R.kf[ks] = lds_read_b128<0>(kaddr[ks]);
#pragma unroll
          for (int ks = 0; ks < G::NKS; ks += 4)
            lgkm_wait<0>(R.kf[ks], R.kf[ks + 1], R.kf[ks + 2], R.kf[ks + 3]);
#pragma unroll
          for (int i = 0; i < 16; ++i) R.s[0][i] = 0.f;
#pragma unroll
          for (int ks = 0; ks < G::NKS; ++ks)
            R.s[0] = mfma32(__builtin_bit_cast(bf16x8_t, R.kf[ks]), qf[ks], R.s[0]);
          __builtin_amdgcn_sched_barrier(0);
          // the empty P stage of the first step: V and P are zero
#pragma unroll
          for (int m = 0; m < G::NVF; ++m) R.vf[m] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
          for (int t = 0; t < G::TERMS; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) R.pb[1][t][0][i] = R.pb[1][t][1][i] = 0u;
          __builtin_amdgcn_sched_barrier(0);
        }

        // The next tile is requested during the first two steps, one part (a K and a V
        // instruction per wavefront) at a time: a burst fills the memory pipeline's queue and
        // stalls every wavefront behind it.
        auto no_hook = [](auto) {};
        constexpr int PPS = G::PARTS / 2;  // parts per step
        // (Where the loop begins in a line of 64 bytes tells, with one and the same code: 131072 tokens
        // over 16 ranks behind flags take 57.87 ms from 28 or 60 on and 58.24 from 16 on, rings at
        // head_dim 64 up to .7 %. The other kernels do not tell.)
        if constexpr (MODE == RING || D == 64) asm volatile(".p2align 6");
        for (int it = 0; it < n_live; ++it) {
          const bool has_next = it + 1 < n_live;
          const int nb = (it + 1) & 1;
          pipe_body<D, 0, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, mask & 1,
                                mask & 16, have_ref,
                                [&](auto mc) __attribute__((always_inline)) {
                                  constexpr int M = decltype(mc)::value;
                                  if (M == 1 && __builtin_expect(has_next, 1)) issue_part(IntC<0>{}, next, nb);
                                  if (M == 9 && __builtin_expect(has_next, 1)) issue_part(IntC<1>{}, next, nb);
                                });
          pipe_body<D, 1, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, mask & 2,
                                mask & 32, have_ref,
                                [&](auto mc) __attribute__((always_inline)) {
                                  constexpr int M = decltype(mc)::value;
                                  if (M == 1 && __builtin_expect(has_next, 1)) issue_part(IntC<PPS>{}, next, nb);
                                  if (M == 9 && __builtin_expect(has_next, 1)) issue_part(IntC<3>{}, next, nb);
                                });
          // (the pipeline is at the same parity after two blocks as after four. Nothing of this tile is
          // in flight then but the V fragments, which the drain waits for. us, without and with: 320
          // tokens of 8 heads on 2 over 2 ranks at head_dim 64 19.5 and 17.9, 900 of 16 on 2 33.9 and
          // 31.3, 700 of 16 at head_dim 128 26.6 and 25.2, six packed prompts of 200 to 3000 98.1 and 95.8.)
          if (__builtin_expect(half_tail && !has_next, 0)) break;
          pipe_body<D, 2, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, mask & 4,
                                mask & 64, have_ref, no_hook);
          // barrier Y: the next tile has landed in every wavefront
          __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
          if (has_next && tid < TILE) posbuf0[nb * TILE + tid] = next_pos;
          const int cur_mask = mask;
          mask = next.mask;
          read_entry(it + 2, next);  // no direct-to-LDS load is in flight here
          __syncthreads();
#pragma unroll
          for (int ks = 0; ks < G::NKS; ++ks) kaddr[ks] ^= G::KD;  // K of the next tile from here on
          pipe_body<D, 3, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, cur_mask & 8,
                                cur_mask & 128, have_ref, no_hook);
          // barrier X: every LDS read of this tile has completed; its buffers may be refilled
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
          __syncthreads();
#pragma unroll
          for (int db = 0; db < G::NDB; ++db) vaddr[db] ^= G::KD;
          paddr ^= POS_BYTES;
        }

        // ---- drain: P stage of the last block ----
        {
          auto last = [&](auto mc) __attribute__((always_inline)) {
            constexpr int M = decltype(mc)::value;
            if constexpr (M < G::NVF) {
              lgkm_wait<2 * (G::NVF - 1 - M)>(R.vf[M]);
#pragma unroll
              for (int t = 0; t < G::TERMS; ++t)
                R.o[M % G::NDB] = mfma32(__builtin_bit_cast(bf16x8_t, R.vf[M]),
                                         __builtin_bit_cast(bf16x8_t, R.pb[1][t][M / G::NDB]),
                                         R.o[M % G::NDB]);
            }
          };
          last(IntC<0>{}); last(IntC<1>{}); last(IntC<2>{}); last(IntC<3>{});
          last(IntC<4>{}); last(IntC<5>{}); last(IntC<6>{}); last(IntC<7>{});
          __builtin_amdgcn_sched_barrier(0);
        }
        // back to buffer-0 addressing for the next chunk
        if ((n_live - (half_tail ? 1 : 0)) & 1) {
#pragma unroll
          for (int ks = 0; ks < G::NKS; ++ks) kaddr[ks] ^= G::KD;
#pragma unroll
          for (int db = 0; db < G::NDB; ++db) vaddr[db] ^= G::KD;
          paddr ^= POS_BYTES;
        }
      }
    }

    // ---- epilogue ----
    // (The lane's row again: kept over the walk, it and what is made of it took more registers than
    // there are, and a kernel with two spilled registers started 2 us later.)
    int tid_e = threadIdx.x;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63, n_e = lane_e & 31, g_e = lane_e >> 5;
    const int r = r0 + n_e;
    // PLAN: what the next unit needs of its rows travels behind this epilogue (its registers are the
    // walk's: it costs none), and its address arithmetic is out of the next start.
    int next_rb = row_block + 1, next_z = z_shard, next_kvh = kvh;
    // (defined on every path: else the old ones are kept for the others)
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks) next_qf[ks] = u32x4_t{0u, 0u, 0u, 0u};
    if constexpr (MODE == PLAN) {
      rows_requested = p.cut_units && share.length > 0;
      if (next_rb == p.n_row_blocks) {
        next_rb = 0;
        if (++next_z == p.n_z) {
          next_z = 0;
          ++next_kvh;
        }
      }
      // (No tile is on its way, but where the compiler cannot see it, behind a walk that ends early, it
      // waits for them, and for the rows, at the barrier below.)
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      if (rows_requested)
        request_rows(next_rb, next_kvh, p.rows, tid_e, next_qp, next_ql, next_qf);
    }
    const float l_sum = R.l_run + xor32(R.l_run);
    const float l_tot = sees ? l_sum : 0.f;
    const bool no_key = l_tot == 0.f;
    float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    const float lse_val =
        l_tot > 0.f ? (R.m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
    // Where this lane's row goes: its O (as an address) and its LSE. `partial`: to the
    // workspace, in fp32.
    const bool partial = MODE == SPLIT || (MODE == PLAN && !whole);
    int64_t row_lin;        // row of [tokens, N_H] in the buffer written to
    Glb<char> o_row;
    Glb<float> lse_row = nullptr;
    if (MODE == PLAN && partial) {
      const int slot =
          2 * __builtin_amdgcn_readfirstlane(*share_index) + (first_piece ? 1 : 0);
      row_lin = (int64_t)slot * BM + wave * 32 + n_e;
      o_row = (Glb<char>)(p.part_out + row_lin * D);
      lse_row = (Glb<float>)(p.part_lse + row_lin);
    } else {
      int token = row_ok ? (int)((uint32_t)r / (uint32_t)p.group) : 0;
      const int hg = row_ok ? r - token * p.group : 0;
      auto o = (Glb<char>)argument(MODE == RING ? p.t.out[rank] : p.out);
      auto l = argument(MODE == RING ? p.t.lse[rank] : p.lse);
      if (MODE == PLAN && p.n_ranks > 1) {
        const int t0 = (int)((uint32_t)(row_block * BM) / (uint32_t)p.group);
        const int a = planned_rank(t0, token, lane_e);
        token -= row_ok ? L.tok_begin[a] : token;
        o = (Glb<char>)L.ranks[a].out;
        l = (Glb<float>)L.ranks[a].lse;
      } else if (MODE != SPLIT && MODE != RING && p.n_ranks > 1) {
        const int a = rank_of_token(p.t, token);
        token -= p.t.tok_begin[a];
        o = (Glb<char>)p.t.out[a];
        l = (Glb<float>)p.t.lse[a];
      }
      row_lin = ((int64_t)token * p.n_kv_heads + kvh) * p.group + hg;
      if (MODE == SPLIT) {
        row_lin += (int64_t)(z_shard * p.n_sub + z_sub) * p.rows_all_heads;
        o = (Glb<char>)p.part_out;
        l = (Glb<float>)p.part_lse;
      } else {
        o += (int64_t)z_shard * p.out_shard_stride;
        if (l != nullptr) l += (int64_t)z_shard * p.lse_shard_stride;
      }
      o_row = o + row_lin * (D * (int64_t)(MODE == SPLIT ? 4 : sizeof(TO)));
      if (l != nullptr) lse_row = l + row_lin;
    }
    // Rows that a V they do not see has spoiled (see VectorRow). Not in the ring walk, whose main
    // loop would pay for it with 200 spilled registers.
    uint32_t spoiled = 0;
    if constexpr (MODE != RING) {
      float most = 0.f;   // finite if O is (the maximum of a NaN is NaN)
#pragma unroll
      for (int db = 0; db < G::NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; i += 2)
          most = __builtin_elementwise_maximum(
              __builtin_elementwise_maximum(__builtin_fabsf(R.o[db][i]),
                                            __builtin_fabsf(R.o[db][i + 1])), most);
      most = __builtin_elementwise_maximum(most, xor32(most));
      spoiled = (uint32_t)__builtin_amdgcn_ballot_w64(
          row_ok && l_tot > 0.f && l_tot < INFINITY && !(most < INFINITY));
    }
    float share_of_row = 1.f;   // ACC: weight of this step
    // ACC: weights of Equation 4 for the pair (running result, this step). a_old scales the
    // stored row, the step's row is scaled on its way into the staging buffer. A row the step
    // saw nothing of keeps its stored value (a_old = 1, nothing staged): it is not touched at
    // all unless this is the step that writes the final output.
    float a_old = 0.f;
    if constexpr (MODE == ACC) {
      const float lse_old = row_ok ? *lse_row : -INFINITY;
      const float m = fmaxf(lse_old, lse_val);
      const float w_old = m == -INFINITY ? 0.f : __expf(lse_old - m);
      const float w_cur = m == -INFINITY ? 0.f : __expf(lse_val - m);
      const float den = w_old + w_cur;
      const float rden = den > 0.f ? 1.f / den : 0.f;
      a_old = l_tot > 0.f ? w_old * rden : 1.f;
      share_of_row = w_cur * rden;
      inv *= share_of_row;
      const float lse_new = den > 0.f ? m + __logf(den) : -INFINITY;
      if (row_ok && g_e == 0) {
        if (l_tot > 0.f) *lse_row = lse_new;
        if (p.final_lse != nullptr) p.final_lse[row_lin] = lse_new;
      }
    } else {
      if (row_ok && g_e == 0 && lse_row != nullptr) *lse_row = lse_val;
    }

    // Transpose through LDS (the tile buffers are dead once every wavefront has left the walk;
    // each wavefront then uses a private region). Accumulator (db, i) of lane (n, g) is channel
    // db*32 + (i/4)*8 + g*4 + i%4 of query n.
    __syncthreads();
    char* const stage = smem + wave * 32 * G::OUT_STRIDE;
#pragma unroll
    for (int db = 0; db < G::NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const int d0 = db * 32 + i4 * 8 + g_e * 4;
        floatx4_t w = {R.o[db][i4 * 4 + 0] * inv, R.o[db][i4 * 4 + 1] * inv,
                       R.o[db][i4 * 4 + 2] * inv, R.o[db][i4 * 4 + 3] * inv};
        *(floatx4_t*)(stage + n_e * G::OUT_STRIDE + d0 * 4) = w;
      }
    if (no_key) {   // (O may be NaN there)
#pragma unroll
      for (int i = 0; i < D / 8; ++i)
        *(floatx4_t*)(stage + n_e * G::OUT_STRIDE + (i * 8 + g_e * 4) * 4) =
            floatx4_t{0.f, 0.f, 0.f, 0.f};
    }
    wave_lds_fence();
    if constexpr (MODE != RING) {
      while (__builtin_expect(spoiled != 0, 0)) {
        const int rr = __builtin_ctz(spoiled);
        spoiled &= spoiled - 1;
        const int row = row_block * BM + wave * 32 + rr;
        int token = (int)((uint32_t)row / (uint32_t)p.group);
        const int hg = row - token * p.group;
        const int a = p.n_ranks > 1 ? rank_of_token(p.t, token) : 0;
        token -= p.t.tok_begin[a];
        VectorRow<bf16_t, D> vr;
        vr.q = (const bf16_t*)p.t.q[a] + (((int64_t)token * p.n_kv_heads + kvh) * p.group + hg) * D;
        vr.scale_log2 = scale_log2;
        vr.qp = __builtin_amdgcn_readlane(qp, rr);
        vr.ql = BAND ? __builtin_amdgcn_readlane(ql, rr) : INT32_MIN;
        int sh = z_shard, idx = 0;
        for (int c = b_begin; c < b_end; c += 64) {   // the blocks walked above
          uint64_t mask = __builtin_amdgcn_ballot_w64(
              c + lane_e < b_end && visible(block_bounds(min(c + lane_e, b_end - 1))));
          for (; mask != 0; mask &= mask - 1, ++idx) {
            if (idx < part_lo || idx >= part_hi) continue;
            const int b = c + __builtin_ctzll(mask);
            while (!one_shard && b >= p.t.blk_begin[sh + 1]) ++sh;
            const int key0 = (b - p.t.blk_begin[sh]) * BLOCK;
            const int64_t off = ((int64_t)key0 * p.n_kv_heads + kvh) * D;
            vr.keys((const bf16_t*)p.t.k[sh] + off, (const bf16_t*)p.t.v[sh] + off,
                    p.t.kv_pos[sh] + key0, min(BLOCK, p.t.n_kv[sh] - key0),
                    (uint32_t)p.n_kv_heads * D, lane_e);
          }
        }
        const float f = __shfl(share_of_row, rr, 64) / vr.l;
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
          ((float*)(stage + rr * G::OUT_STRIDE))[lane_e * (D / 64) + c] = vr.acc[c] * f;
        wave_lds_fence();
      }
    }
    // (rows in order: row rr of the wavefront exists iff its lane's does)
    const uint64_t rows_ok = __builtin_amdgcn_ballot_w64(row_ok);
    auto row_address = [&](int rr) -> Glb<char> {
      const uint64_t x = (uint64_t)o_row;
      const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, rr, 64);
      const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), rr, 64);
      return (Glb<char>)((uint64_t)hi << 32 | lo);
    };
    if constexpr (MODE == ACC) {
      // The stored row (fp32) times its weight is added to the step's row, 4 channels per
      // lane; the sum goes back to its place, or to the final output on the last step.
      const bool to_final = p.final_out != nullptr;  // uniform
      const bool seen_row = l_tot > 0.f;
      constexpr int LPR = D / 4, RPP = 64 / LPR;     // lanes per row, rows per pass
#pragma unroll
      for (int pass = 0; pass < 32 / RPP; ++pass) {
        const int rr = pass * RPP + lane_e / LPR, c = (lane_e % LPR) * 4;
        const int64_t rl = __shfl(row_lin, rr, 64);
        float* const old_row = p.acc + rl * D + c;
        const float ao = __shfl(a_old, rr, 64);
        const bool touch = (to_final || __shfl((int)seen_row, rr, 64) != 0) && (rows_ok >> rr & 1);
        floatx4_t a = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4);
        if (touch) {
          if (ao != 0.f) {
            const floatx4_t old = *(const floatx4_t*)old_row;
#pragma unroll
            for (int x = 0; x < 4; ++x) a[x] = fmaf(ao, old[x], a[x]);
          }
          if (!to_final) {
            *(floatx4_t*)old_row = a;
          } else {
            TO* const o = (TO*)p.final_out + rl * D + c;
            if constexpr (sizeof(TO) == 4) {
              *(floatx4_t*)o = a;
            } else {
              bf16x4_t w;
#pragma unroll
              for (int x = 0; x < 4; ++x) w[x] = static_cast<bf16_t>(a[x]);
              *(bf16x4_t*)o = w;
            }
          }
        }
      }
    } else if (MODE != SPLIT && sizeof(TO) == 2 && !partial) {
      constexpr int LPR = D / 8, RPP = 64 / LPR;
#pragma unroll
      for (int pass = 0; pass < 32 / RPP; ++pass) {
        const int rr = pass * RPP + lane_e / LPR, c = (lane_e % LPR) * 8;
        const Glb<char> o = row_address(rr);
        const floatx4_t a = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4);
        const floatx4_t b = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4 + 16);
        bf16x8_t w;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          w[x] = static_cast<bf16_t>(a[x]);
          w[4 + x] = static_cast<bf16_t>(b[x]);
        }
        if (rows_ok >> rr & 1) *(Glb<bf16x8_t>)(o + c * 2) = w;
      }
    } else {
      constexpr int LPR = D / 4, RPP = 64 / LPR;
#pragma unroll
      for (int pass = 0; pass < 32 / RPP; ++pass) {
        const int rr = pass * RPP + lane_e / LPR, c = (lane_e % LPR) * 4;
        const Glb<char> o = row_address(rr);
        const floatx4_t a = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4);
        if (rows_ok >> rr & 1) *(Glb<floatx4_t>)(o + c * 4) = a;
      }
    }
    if constexpr (MODE != PLAN) return;
    if (!rows_requested) return;
    row_block = next_rb;
    z_shard = next_z;
    kvh = next_kvh;
    share.begin = 0;
    lds_barrier();   // the staging buffer is read before the next unit's tiles arrive (the
                     // stores need not have left)
  }
}

template <int D, typename TO, bool BAND, Mode MODE>
__global__ __launch_bounds__(NTHREADS) void prefill_mfma_kernel(const Params p) {
  prefill_body<D, TO, BAND, MODE>(p);
}

// All ring steps of every rank, each behind its arrival flag (the RING variant).
template <typename TO>
__global__ __launch_bounds__(NTHREADS) void prefill_ring_walk_kernel(const Params p) {
  prefill_body<128, TO, false, RING>(p);
}

// Equation 4 over the pieces of the units that PLAN cut: grid.x is the share boundary, grid.y a
// part of the unit's rows. The first boundary inside a unit merges it (most boundaries cut one,
// into two pieces). Bound by the partials, up to 67 MB each way, and by latency where there are
// few: a thread has all its rows' loads of two pieces in flight at once.
constexpr int kMergeParts = 8;
template <int D, typename TO>
__global__ __launch_bounds__(256) void plan_merge_kernel(const Params p) {
  const int touched = touch_arguments<Params>();
  const int i = blockIdx.x + 1;
  // (a share that begins behind the start-up of a unit cuts it; the records end with unit -1)
  const int2 prev = p.plan_rec[i - 1], rec = p.plan_rec[i], next = p.plan_rec[i + 1];
  if (rec.x < 0 || rec.y == 0) return;
  if (prev.x == rec.x && prev.y != 0) return;
  int last = i;                       // the last workgroup with a piece of the unit
  if (next.x == rec.x)
    while (p.plan_rec[last + 1].x == rec.x) ++last;
  constexpr int TPR = D / 4, RPP = 256 / TPR;   // threads per row, rows per pass
  constexpr int U = BM / kMergeParts / RPP;     // rows per thread
  const int col = (threadIdx.x % TPR) * 4;
  const int row0 = blockIdx.y * (BM / kMergeParts) + threadIdx.x / TPR;
  // Where this thread's rows go, looked up before the pieces are waited for (and the lines of the
  // arguments asked for together: packed prompts 15.8 -> 14.0 us, 4096 tokens at head_dim 64 8.2 -> 7.5).
  const int units = p.n_row_blocks * p.n_z;
  const int kvh = rec.x / units, u = rec.x - kvh * units;
  const int z = u / p.n_row_blocks, rb = u - z * p.n_row_blocks;
  TO* o[U];
  float* o_lse[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const int64_t r = min<int64_t>((int64_t)rb * BM + row0 + k * RPP, (int64_t)p.rows - 1);
    const int token = (int)((uint32_t)r / (uint32_t)p.group);
    const int hg = (int)(r - (int64_t)token * p.group);
    const int a = p.n_ranks > 1 ? rank_of_token(p.t, token) : 0;
    const int64_t lin = ((int64_t)(token - p.t.tok_begin[a]) * p.n_kv_heads + kvh) * p.group + hg;
    o[k] = (TO*)((char*)p.t.out[a] + z * p.out_shard_stride) + lin * D + col;
    o_lse[k] = p.t.lse[a] != nullptr ? p.t.lse[a] + z * p.lse_shard_stride + lin : nullptr;
  }
  asm volatile("" ::"v"(touched));
  float lmax[U], den[U];
  floatx4_t acc[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    lmax[k] = -INFINITY;
    den[k] = 0.f;
    acc[k] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  for (int j0 = i - 1; j0 <= last; j0 += 2) {
    floatx4_t x[U][2];
    float l[U][2];
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int j = min(j0 + b, last);   // (slots hold whole row blocks)
        const int64_t s = (int64_t)(j == i - 1 ? 2 * j + 1 : 2 * j) * BM + row0 + k * RPP;
        l[k][b] = p.part_lse[s];
        x[k][b] = __builtin_nontemporal_load((const floatx4_t*)(p.part_out + s * D + col));
      }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const float l1 = j0 + 1 <= last ? l[k][1] : -INFINITY;
      const float m = fmaxf(lmax[k], fmaxf(l[k][0], l1));
      if (m != -INFINITY) {
        const float old = __expf(lmax[k] - m), w0 = __expf(l[k][0] - m), w1 = __expf(l1 - m);
        den[k] = fmaf(den[k], old, w0 + w1);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          acc[k][c] = fmaf(acc[k][c], old, fmaf(w0, x[k][0][c], w1 * x[k][1][c]));
        lmax[k] = m;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    if ((int64_t)rb * BM + row0 + k * RPP >= p.rows) continue;
    const float inv = den[k] > 0.f ? 1.f / den[k] : 0.f;
    if constexpr (sizeof(TO) == 4) {
      *(floatx4_t*)o[k] = acc[k] * inv;
    } else {
      bf16x4_t w;
#pragma unroll
      for (int c = 0; c < 4; ++c) w[c] = static_cast<bf16_t>(acc[k][c] * inv);
      *(bf16x4_t*)o[k] = w;
    }
    if (col == 0 && o_lse[k] != nullptr)
      *o_lse[k] = den[k] > 0.f ? lmax[k] + __logf(den[k]) : -INFINITY;
  }
}
