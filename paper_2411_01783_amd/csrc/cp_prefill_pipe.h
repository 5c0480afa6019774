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
//     P(i-1):  O^T += V^T P^T of the previous block        (D / 16 MFMA, matrix pipe)
//     SM(i):   mask, row maximum, exponentials of block i   (vector pipe)
//     Q(i+1):  S^T = K Q^T of the next block                (D / 16 MFMA, matrix pipe)
// The three are independent, so the vector work is issued between the MFMAs of its
// neighbours, one slice per MFMA (two at D = 64), in source order (scheduling fences keep
// that order). LDS fragment reads are inline assembly with hand-counted lgkmcnt waits, issued
// D / 16 MFMAs before their use: the compiler would otherwise wait for the tile prefetch
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

// Sizes and LDS layout for head_dim D. The list of visible tiles holds, per tile, the
// addresses of its K and V rows (this KV head) and of its positions, so that a workgroup walks
// tiles of any number of KV shards with one loop.
template <int D>
struct Geo {
  static constexpr int ROW = D * 2;              // one K or V row in bytes
  static constexpr int KD = TILE * ROW;          // one tile buffer of K or of V
  static constexpr int BLK = 32 * ROW;           // one 32-key block of a tile
  static constexpr int NKS = D / 16;             // MFMAs of S^T per block, K fragments
  static constexpr int NDB = D / 32;             // 32-channel blocks of O^T
  static constexpr int NVF = 2 * NDB;            // MFMAs of O^T per block, V^T fragments
  static constexpr int CHUNKS = ROW / 16;        // 16-byte chunks of a row
  static constexpr int LOAD_ROWS = 64 / CHUNKS;  // rows one 1 KiB load instruction brings
  static constexpr int PARTS = 16 / LOAD_ROWS;   // load instructions per wavefront for K (or V)
  static constexpr int OFF_V = 2 * KD;
  static constexpr int OFF_POS = OFF_V + 2 * KD;
  static constexpr int OFF_SCRATCH = OFF_POS + 2 * POS_BYTES;
  static constexpr int OFF_LIVE = OFF_SCRATCH + 128;
  static constexpr int OFF_LIVE_LO = OFF_LIVE + MAX_LIVE * 32;
  static constexpr int SMEM = OFF_LIVE_LO + MAX_LIVE * 4;
  static constexpr int OUT_STRIDE = D * 4 + 16;  // epilogue staging: one fp32 output row + pad
  static_assert(NWAVE * 32 * OUT_STRIDE <= SMEM, "epilogue staging fits in the allocation");
  static_assert(SMEM <= 160 * 1024, "LDS budget of one CU");
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

// Workgroup barrier that orders LDS traffic only: global loads issued before it (the Q
// fragments, the tile-bound prefetch) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Everything a wavefront carries from block to block. All indices are compile-time.
template <int D>
struct PipeRegs {
  floatx16_t o[D / 32];    // O^T accumulators, blocks of 32 channels
  floatx16_t s[2];         // scores of block i (index: parity of i) and of block i+1
  u32x4_t pb[2][2];        // probabilities (bf16 pairs) of block i (parity of i) / i-1, two 16-key slices
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
                                          float scale_log2, bool need_mask, bool& have_ref,
                                          Hook hook) {
  using G = Geo<D>;
  constexpr int CUR = BLK & 1, NXT = CUR ^ 1;
  constexpr int KOFF = ((BLK + 1) & 3) * G::BLK;
  constexpr int VOFF = BLK * G::BLK;
  constexpr int H = G::NKS;          // MFMAs per half step
  constexpr int SL = 8 / H;          // vector slices per MFMA
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
  // Full form (masked tiles, and until every row of the wavefront has a reference): block
  // maximum, and the reference is raised when the maximum exceeds it by more than
  // kRescaleSlack. Fast form (everything else): no maximum at all. The exponentials are taken
  // against the standing reference, whatever the block holds; the reference is never above a
  // score the row has seen, so nothing underflows that should not, and a block whose
  // exponentials sum to more than kOverflowSum (a score 40 log2 units above the reference) is
  // detected from its sum and redone in the full form. O and l are rescaled at the end of
  // the step, after the MFMAs that still belong to the old reference. The denominator sums
  // the unrounded exponentials: LSE must be good to 1e-3 even on rows with a handful of
  // keys, which bf16 rounding of P would not give.
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
      unsigned pk = pack_bf16(e[v - 1], e[v]);
      pin(pk);
      pin(lsum1);
      R.pb[CUR][v >> 3][(v & 7) >> 1] = pk;
    } else {
      lsum0 += e[v];
      pin(lsum0);
    }
  };

  auto valu = [&](auto jc) __attribute__((always_inline)) {
    constexpr int J = decltype(jc)::value;
    if constexpr (J == 0) {
      const bool full = need_mask | !have_ref;  // scalar flags: one branch on the hot path
      if (__builtin_expect(full, 0)) {  // wave-uniform, rare: laid out off the hot path
        if (need_mask) {
          // Masked tiles are the few on the diagonal: their kv_pos reads are simply waited
          // for (which also completes every older LDS read, so the counted waits hold).
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
        const float m_step = block_max() * scale_log2;
        raise = m_step > R.m_run + kRescaleSlack;  // true on the first visible block
        const float m_new = raise ? m_step : R.m_run;
        alpha = __builtin_amdgcn_exp2f(R.m_run - (m_new == -INFINITY ? 0.f : m_new));
        R.l_run *= alpha;
        R.m_run = m_new;
        m_use = m_new == -INFINITY ? 0.f : m_new;
        have_ref = __builtin_amdgcn_ballot_w64(m_new == -INFINITY) == 0;
      } else {
        m_use = R.m_run;
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

  auto slices = [&](auto mc) __attribute__((always_inline)) {
    constexpr int M = decltype(mc)::value;
    valu(IntC<M * SL>{});
    if constexpr (SL == 2) valu(IntC<M * SL + 1>{});
  };

  // ---- first half: P(i-1) on the matrix pipe, K fragments of block i+1 requested ----
  auto first = [&](auto mc) __attribute__((always_inline)) {
    constexpr int M = decltype(mc)::value;
    if constexpr (M < H) {
      // LDS operations issued after V fragment M: H - 1 - M later V fragments (two reads each)
      // and M K fragments
      lgkm_wait<2 * (H - 1 - M) + M>(R.vf[M]);
      R.o[M % G::NDB] = mfma32(__builtin_bit_cast(bf16x8_t, R.vf[M]),
                               __builtin_bit_cast(bf16x8_t, R.pb[NXT][M / G::NDB]),
                               R.o[M % G::NDB]);
      R.kf[M] = lds_read_b128<KOFF>(kaddr[M]);
      hook(IntC<M>{});
      slices(IntC<M>{});
      __builtin_amdgcn_sched_barrier(0);
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
      slices(IntC<H + M>{});
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  second(IntC<0>{}); second(IntC<1>{}); second(IntC<2>{}); second(IntC<3>{});
  second(IntC<4>{}); second(IntC<5>{}); second(IntC<6>{}); second(IntC<7>{});

  // A block of the fast form whose exponentials ran away from the reference (rare): redo
  // its softmax in the full form. No row's sum can pass the test with an infinity or a NaN.
  float blk = lsum0 + lsum1;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(blk <= kOverflowSum)) != 0, 0)) {
    const float m_step = block_max() * scale_log2;
    const float m_new = fmaxf(R.m_run, m_step);
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
__device__ __forceinline__ int ring_flag(const Params& p, int step) {
  return __hip_atomic_load(p.arrived + step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Makes sure that the shard of ring step `step` may be read. With arrival flags, thread 0 looks
// at the step's flag first: `peek` is what it read of that flag while the previous shard
// was being walked (so a shard that arrived in time costs no round trip here); if that was
// zero it polls (uncached loads, a short sleep between them, at most p.spin_limit of them).
// The whole workgroup learns the outcome through LDS; false = the flag never came up:
// bit `step` of *p.ring_error is set and the caller leaves the shard out. Every wait ends.
__device__ __forceinline__ bool ring_enter(const Params& p, int step, int tid, int* wg_scratch,
                                           int& peek) {
  if (p.arrived == nullptr) return true;
  int* const slot = wg_scratch + 20 + (step & 1);  // two slots: a wavefront may lag one step
  if (tid == 0) {
    int ok = 1;
    if (peek == 0) {
      int budget = p.spin_limit;
      while (ring_flag(p, step) == 0) {
        if (--budget <= 0) {
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(32);
      }
    }
    if (!ok) atomicOr(p.ring_error, 1 << step);  // which step gave up (n_shards <= 32)
    *slot = ok;
    // a look at the next step's flag, used when the walk gets there
    peek = step + 1 < p.t.n_shards ? ring_flag(p, step + 1) : 0;
  }
  lds_barrier();
  const int ok = __builtin_amdgcn_readfirstlane(*slot);
  // The shard's data is read after its flag: every load of it is issued after this barrier,
  // which thread 0 reaches only with the flag's value in hand. No cache invalidation: the
  // caller gives every step a buffer of its own that is complete before its flag is set and
  // is not written again while the kernel runs, so no line of it can be in a cache before the
  // flag is seen. (An agent-scope acquire here invalidates the XCD's L2 once per workgroup and
  // shard and costs 3.5 % of the walk.)
  return ok != 0;
}

// The walk of one workgroup: 256 consecutive (token, head-in-group) rows of one KV head, over
// the queries of all ranks of the table back to back, against the visible tiles of the KV
// shards.
// BAND: packed batch. Positions are shifted per sequence and a query also has a lower bound
// q_lo (the shift of its sequence): visible iff q_lo <= kv_pos <= q_pos.
// SPLIT: the launch splits the KV axis over grid.z and writes fp32 partials to the workspace.
// ACC: the result is merged into a running (O, LSE) in the epilogue instead of being written
// as a partial (Equation 4 applied step by step); see the epilogue.
// RING: the shards are walked one by one in ring order (from p.ring_start downwards), each
// behind its arrival flag (bounded wait), with one running (O, l, m) in registers: the merge of
// Equation 4 happens inside the online softmax.
template <int D, typename TO, bool BAND, bool SPLIT, bool ACC, bool RING>
__device__ __forceinline__ void prefill_body(const Params& p) {
  static_assert(!RING || (!BAND && !SPLIT && !ACC), "the ring walk is its own variant");
  using G = Geo<D>;
  constexpr int ROW = G::ROW;
  extern __shared__ __align__(16) char smem[];
  char* const kbuf0 = smem;
  char* const vbuf0 = smem + G::OFF_V;
  int32_t* const posbuf0 = (int32_t*)(smem + G::OFF_POS);
  int* const wg_scratch = (int*)(smem + G::OFF_SCRATCH);
  int4* const live = (int4*)(smem + G::OFF_LIVE);
  int32_t* const live_lo_pos = (int32_t*)(smem + G::OFF_LIVE_LO);
  const uint32_t smem_lds = (uint32_t)(size_t)(CP_LDS_AS char*)smem;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 31, g = lane >> 5;
  const int row_block = ordered_row_block(blockIdx.x, gridDim.x, p.t.n_ranks, lane);
  const int kvh = blockIdx.y;
  // grid.z: the n_sub parts of the KV axis, of every shard in turn when shards are kept apart
  const int z_shard = p.per_shard ? blockIdx.z / p.n_sub : 0;
  const int z_sub = blockIdx.z - z_shard * p.n_sub;

  // ---- tiles of this workgroup (the ring walk moves on from shard to shard) ----
  int cur_shard = RING ? p.ring_start : z_shard;
  int t_begin = RING || p.per_shard ? p.t.tile_begin[cur_shard] : 0;
  int t_end = RING || p.per_shard ? p.t.tile_begin[cur_shard + 1] : p.n_tiles;

  // ---- this lane's query row ----
  // (rows fit 31 bits: checked by the launcher)
  const int64_t r = (int64_t)row_block * BM + wave * 32 + n;
  const bool row_ok = r < p.rows;
  // The start-up chain is q_pos -> visible tiles -> first tile; the bounds of the first 512
  // tiles are requested now so that they arrive together with q_pos, and the Q fragments
  // (needed last) are requested after both and waited for only before the first product.
  int2 first_bounds = make_int2(0, 0);
  if (t_begin + wave * 64 + lane < t_end) first_bounds = p.bounds[t_begin + wave * 64 + lane];
  int32_t qp = CP_POS_PAD_Q, ql = INT32_MIN;
  bf16x8_t qf[G::NKS];
  {
    const int token = row_ok ? (int)((uint32_t)r / (uint32_t)p.group) : 0;
    const int hg = row_ok ? (int)(r - (int64_t)token * p.group) : 0;
    const bf16_t* q = (const bf16_t*)p.t.q[0];
    const int32_t* q_pos = p.t.q_pos[0];
    int first = 0;
    if (p.t.n_ranks > 1) {
      const int a = rank_of_token(p.t, token);
      q = (const bf16_t*)p.t.q[a];
      q_pos = p.t.q_pos[a];
      first = p.t.tok_begin[a];
    }
    if (row_ok) qp = q_pos[token - first];
    if (BAND && row_ok) ql = p.q_lo[token];
    const int64_t row = ((int64_t)(token - first) * p.n_kv_heads + kvh) * p.group + hg;
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks) {
      uint4 x = make_uint4(0, 0, 0, 0);
      if (row_ok) x = *(const uint4*)(q + row * D + ks * 16 + g * 8);
      qf[ks] = __builtin_bit_cast(bf16x8_t, x);
    }
  }
  const float scale_log2 = p.scale_log2;

  // ---- query position range of the wavefront and of the workgroup ----
  // rows that can see anything: a padded query (CP_POS_PAD_Q) and the rows past the end of
  // the shard cannot, and stay out of the ranges below
  const bool sees = row_ok && qp >= 0;
  int w_qmin = sees ? qp : INT32_MAX, w_qmax = qp;
  int w_lomin = BAND && sees ? ql : INT32_MAX, w_lomax = BAND && sees ? ql : INT32_MIN;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    w_qmin = min(w_qmin, __shfl_xor(w_qmin, o, 64));
    w_qmax = max(w_qmax, __shfl_xor(w_qmax, o, 64));
    if (BAND) {
      w_lomin = min(w_lomin, __shfl_xor(w_lomin, o, 64));
      w_lomax = max(w_lomax, __shfl_xor(w_lomax, o, 64));
    }
  }
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
  w_qmin = __builtin_amdgcn_readfirstlane(w_qmin);
  if (BAND) {
    wg_lomin = __builtin_amdgcn_readfirstlane(wg_lomin);
    w_lomax = __builtin_amdgcn_readfirstlane(w_lomax);
  }

  bool have_ref = false;  // every row of the wavefront has a finite reference maximum
  PipeRegs<D> R;
  // Reference max of scaled scores (log2 domain). A row that can see nothing gets a finite
  // reference no score reaches: its exponentials are all zero whichever softmax form its
  // wavefront takes (so one padded row does not keep the other 31 on the masked form), its
  // denominator stays zero, and the epilogue writes O = 0, LSE = -inf for it.
  R.m_run = sees ? -INFINITY : kDeadRowRef;
  R.l_run = 0.f;        // running denominator over this lane's half of the keys
#pragma unroll
  for (int db = 0; db < G::NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) R.o[db][i] = 0.f;

  // ---- tile loader: this wavefront brings rows wave*16 .. wave*16+15 of K and of V, 1 KiB
  // (LOAD_ROWS rows) per instruction; lane l covers row l / CHUNKS of them, chunk position
  // l % CHUNKS. Part I of a tile is one such instruction for K and one for V. Rows past the end
  // of the shard are clamped to its last row (they are masked by their position).
  const uint32_t stride_b = (uint32_t)p.n_kv_heads * ROW;  // bytes between tokens
  const int l_row = lane / G::CHUNKS, l_pos = lane % G::CHUNKS;
  struct Tile {          // (wave-uniform)
    const char* k;
    const char* v;
    const int32_t* pos;
    int n_valid;
    bool mask;  // one of its keys can be hidden from one of this wavefront's rows (this
                // includes the tiles that only other wavefronts of the workgroup can see)
  };
  auto issue_part = [&](auto ic, const Tile& t, int b) __attribute__((always_inline)) {
    constexpr int I = decltype(ic)::value;
    if constexpr (I < G::PARTS) {
      const int row = wave * 16 + I * G::LOAD_ROWS + l_row;
      const uint32_t roff = __umul24((uint32_t)min(row, t.n_valid - 1), stride_b);
      const int pr = I * G::LOAD_ROWS + l_row;  // row % 16 selects the permutation
      load_lds16(t.k + (roff + ((l_pos ^ G::k_perm(pr)) * 16)),
                 kbuf0 + b * G::KD + (wave * 16 + I * G::LOAD_ROWS) * ROW);
      load_lds16(t.v + (roff + ((l_pos ^ G::v_perm(pr)) * 16)),
                 vbuf0 + b * G::KD + (wave * 16 + I * G::LOAD_ROWS) * ROW);
    }
  };
  // kv_pos of the tile goes through a register (the tail needs the pad value)
  auto load_pos = [&](const Tile& t) -> int32_t {
    return tid < t.n_valid ? t.pos[tid] : CP_POS_PAD_KV;   // (used by tid < TILE)
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
  // Where the KV axis is split, every part takes an equal share of the tiles that this
  // workgroup can see: entries [part_lo, part_hi) of the list of visible tiles. A range of more
  // than one list has to be counted first.
  int part_lo = 0, part_hi = INT32_MAX;
  if (!RING && p.n_sub > 1 && t_end - t_begin > MAX_LIVE) {
    int cnt = 0;
    for (int t = t_begin + tid; t < t_end; t += NTHREADS) cnt += visible(p.bounds[t]) ? 1 : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    lds_barrier();
    if (lane == 0) wg_scratch[wave] = cnt;
    lds_barrier();
    int total = 0;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) total += wg_scratch[w];
    total = __builtin_amdgcn_readfirstlane(total);
    part_lo = (int)((int64_t)total * z_sub / p.n_sub);
    part_hi = (int)((int64_t)total * (z_sub + 1) / p.n_sub);
  }

  int flag_peek = 0;
  const int n_steps = RING ? p.t.n_shards : 1;
  for (int step = 0; step < n_steps; ++step) {
    if constexpr (RING) {
      if (step > 0) {
        cur_shard = cur_shard > 0 ? cur_shard - 1 : p.t.n_shards - 1;
        t_begin = p.t.tile_begin[cur_shard];
        t_end = p.t.tile_begin[cur_shard + 1];
      }
      if (!ring_enter(p, step, tid, wg_scratch, flag_peek))
        continue;  // the shard never arrived: reported through ring_error, walk goes on
    }
    int seen = 0;  // visible tiles before this chunk of the range
    for (int c0 = t_begin; c0 < t_end; c0 += MAX_LIVE) {
      // Compact the tiles some query of the workgroup can see (smallest key position not
      // beyond the largest query position) into an ascending list in LDS.
      lds_barrier();  // previous chunk (list, tile buffers) fully consumed
      int n_live;
      {
        const int t = c0 + wave * 64 + lane;
        int2 b = make_int2(0, 0);
        bool lv = false;
        if (t < t_end) {
          b = (c0 == t_begin && step == 0) ? first_bounds : p.bounds[t];
          lv = visible(b);
        }
        const uint64_t mask = __builtin_amdgcn_ballot_w64(lv);
        if (lane == 0) wg_scratch[wave] = __builtin_popcountll(mask);
        lds_barrier();
        int base = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) {
          const int c = wg_scratch[w];
          if (w < wave) base += c;
          total += c;
        }
        total = __builtin_amdgcn_readfirstlane(total);
        if (!RING && p.n_sub > 1 && t_end - t_begin <= MAX_LIVE) {
          part_lo = (int)((uint32_t)(total * z_sub) / (uint32_t)p.n_sub);
          part_hi = (int)((uint32_t)(total * (z_sub + 1)) / (uint32_t)p.n_sub);
        }
        const int lo = max(part_lo, seen), hi = min(part_hi, seen + total);
        const int idx = seen + base + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
        if (lv && idx >= lo && idx < hi) {
          int sh = cur_shard;
          if (!RING && !p.per_shard) {
#pragma unroll 8
            for (int i = 1; i < p.t.n_shards; ++i) sh += t >= p.t.tile_begin[i];
          }
          const int key0 = (t - p.t.tile_begin[sh]) * TILE;
          const int valid = min(TILE, p.t.n_kv[sh] - key0);
          const uint64_t off = (uint64_t)key0 * stride_b + (uint32_t)kvh * ROW;
          const uint64_t ka = (uint64_t)p.t.k[sh] + off, va = (uint64_t)p.t.v[sh] + off;
          const uint64_t pa = (uint64_t)(p.t.kv_pos[sh] + key0);
          // (a ragged tile always pays for the mask: its largest position is the pad's)
          live[2 * (idx - lo)] = make_int4((int)ka, (int)(ka >> 32), (int)va, (int)(va >> 32));
          live[2 * (idx - lo) + 1] =
              make_int4((int)pa, (int)(pa >> 32), valid, valid < TILE ? INT32_MAX : b.y);
          if (BAND) live_lo_pos[idx - lo] = b.x;
        }
        seen += total;
        n_live = max(0, hi - lo);
      }
      lds_barrier();
      if (n_live == 0) continue;

      // ---- prologue: tile 0 into buffer 0, Q stage of block 0 ----
      int32_t next_pos = 0;
      auto read_entry = [&](int idx, Tile& t) {
        const int i = idx < n_live ? idx : n_live - 1;
        const int4 a = live[2 * i], b = live[2 * i + 1];
        auto uni = [](int x) { return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(x); };
        t.k = (const char*)(uni(a.x) | uni(a.y) << 32);
        t.v = (const char*)(uni(a.z) | uni(a.w) << 32);
        t.pos = (const int32_t*)(uni(b.x) | uni(b.y) << 32);
        t.n_valid = __builtin_amdgcn_readfirstlane(b.z);
        t.mask = __builtin_amdgcn_readfirstlane(b.w) > w_qmin;
        if (BAND) t.mask |= __builtin_amdgcn_readfirstlane(live_lo_pos[i]) < w_lomax;
      };
      Tile next;
      bool need_mask;
      {
        Tile t0;
        read_entry(0, t0);
        read_entry(1, next);
        need_mask = t0.mask;
        issue_part(IntC<0>{}, t0, 0);
        issue_part(IntC<1>{}, t0, 0);
        issue_part(IntC<2>{}, t0, 0);
        issue_part(IntC<3>{}, t0, 0);
        const int32_t pos = load_pos(t0);
        if (tid < TILE) posbuf0[tid] = pos;
        __syncthreads();  // waits for the tile (vmcnt) and publishes it
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
        // stand-in V fragments for the empty P stage of the first step (finite data, P = 0)
#pragma unroll
        for (int m = 0; m < G::NVF; ++m) R.vf[m] = lds_read_vt_frag<0, ROW>(vaddr[m % G::NDB]);
#pragma unroll
        for (int i = 0; i < 4; ++i) R.pb[1][0][i] = R.pb[1][1][i] = 0u;
        __builtin_amdgcn_sched_barrier(0);
      }

      // The next tile is requested during the first two steps, one part (a K and a V
      // instruction per wavefront) at a time: a burst fills the memory pipeline's queue and
      // stalls every wavefront behind it.
      auto no_hook = [](auto) {};
      constexpr int PPS = G::PARTS / 2;  // parts per step
      for (int it = 0; it < n_live; ++it) {
        const bool has_next = it + 1 < n_live;
        const int nb = (it + 1) & 1;
        pipe_body<D, 0, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, need_mask, have_ref,
                              [&](auto mc) __attribute__((always_inline)) {
                                constexpr int M = decltype(mc)::value;
                                if (M == 1 && __builtin_expect(has_next, 1)) issue_part(IntC<0>{}, next, nb);
                                if (M == 9 && __builtin_expect(has_next, 1)) issue_part(IntC<1>{}, next, nb);
                              });
        pipe_body<D, 1, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, need_mask, have_ref,
                              [&](auto mc) __attribute__((always_inline)) {
                                constexpr int M = decltype(mc)::value;
                                if (M == 1 && __builtin_expect(has_next, 1)) issue_part(IntC<PPS>{}, next, nb);
                                if (M == 2 * G::NKS - 7 && __builtin_expect(has_next, 1)) {
                                  if constexpr (PPS > 1) issue_part(IntC<3>{}, next, nb);
                                  next_pos = load_pos(next);
                                }
                              });
        pipe_body<D, 2, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, need_mask, have_ref, no_hook);
        // barrier Y: the next tile has landed in every wavefront
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        if (has_next && tid < TILE) posbuf0[nb * TILE + tid] = next_pos;
        const bool cur_mask = need_mask;
        need_mask = next.mask;
        read_entry(it + 2, next);  // no direct-to-LDS load is in flight here
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < G::NKS; ++ks) kaddr[ks] ^= G::KD;  // K of the next tile from here on
        pipe_body<D, 3, BAND>(R, qf, kaddr, vaddr, paddr, qp, ql, scale_log2, cur_mask, have_ref, no_hook);
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
            R.o[M % G::NDB] = mfma32(__builtin_bit_cast(bf16x8_t, R.vf[M]),
                                     __builtin_bit_cast(bf16x8_t, R.pb[1][M / G::NDB]),
                                     R.o[M % G::NDB]);
          }
        };
        last(IntC<0>{}); last(IntC<1>{}); last(IntC<2>{}); last(IntC<3>{});
        last(IntC<4>{}); last(IntC<5>{}); last(IntC<6>{}); last(IntC<7>{});
        __builtin_amdgcn_sched_barrier(0);
      }
      // back to buffer-0 addressing for the next chunk
      if (n_live & 1) {
#pragma unroll
        for (int ks = 0; ks < G::NKS; ++ks) kaddr[ks] ^= G::KD;
#pragma unroll
        for (int db = 0; db < G::NDB; ++db) vaddr[db] ^= G::KD;
        paddr ^= POS_BYTES;
      }
    }
  }

  // ---- epilogue ----
  static_assert(!(ACC && SPLIT), "the running result is merged by unsplit launches only");
  const float l_tot = R.l_run + xor32(R.l_run);
  float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_val =
      l_tot > 0.f ? (R.m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
  // Where this lane's row goes: its O (as an address) and its LSE.
  int64_t row_lin;        // row of [tokens, N_H] in the buffer written to
  char* o_row;
  float* lse_row = nullptr;
  {
    const int token = row_ok ? (int)((uint32_t)r / (uint32_t)p.group) : 0;
    const int hg = row_ok ? (int)(r - (int64_t)token * p.group) : 0;
    int first = 0;
    char* o = (char*)p.t.out[0];
    float* l = p.t.lse[0];
    if (!SPLIT && p.t.n_ranks > 1) {
      const int a = rank_of_token(p.t, token);
      first = p.t.tok_begin[a];
      o = (char*)p.t.out[a];
      l = p.t.lse[a];
    }
    row_lin = ((int64_t)(token - first) * p.n_kv_heads + kvh) * p.group + hg;
    if (SPLIT) {
      row_lin += (int64_t)blockIdx.z * p.rows_all_heads;
      o = (char*)p.part_out;
      l = p.part_lse;
    } else {
      o += (int64_t)z_shard * p.out_shard_stride;
      if (l != nullptr) l += (int64_t)z_shard * p.lse_shard_stride;
    }
    o_row = o + row_lin * (D * (int64_t)(SPLIT ? 4 : sizeof(TO)));
    if (l != nullptr) lse_row = l + row_lin;
  }
  // ACC: weights of Equation 4 for the pair (running result, this step). a_old scales the
  // stored row, the step's row is scaled on its way into the staging buffer. A row the step
  // saw nothing of keeps its stored value (a_old = 1, nothing staged): it is not touched at
  // all unless this is the step that writes the final output.
  float a_old = 0.f;
  if (ACC) {
    const float lse_old = row_ok ? *lse_row : -INFINITY;
    const float m = fmaxf(lse_old, lse_val);
    const float w_old = m == -INFINITY ? 0.f : __expf(lse_old - m);
    const float w_cur = m == -INFINITY ? 0.f : __expf(lse_val - m);
    const float den = w_old + w_cur;
    const float rden = den > 0.f ? 1.f / den : 0.f;
    a_old = l_tot > 0.f ? w_old * rden : 1.f;
    inv *= w_cur * rden;
    const float lse_new = den > 0.f ? m + __logf(den) : -INFINITY;
    if (row_ok && g == 0) {
      if (l_tot > 0.f) *lse_row = lse_new;
      if (p.final_lse != nullptr) p.final_lse[row_lin] = lse_new;
    }
  } else {
    if (row_ok && g == 0 && lse_row != nullptr) *lse_row = lse_val;
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
      const int d0 = db * 32 + i4 * 8 + g * 4;
      floatx4_t w = {R.o[db][i4 * 4 + 0] * inv, R.o[db][i4 * 4 + 1] * inv,
                     R.o[db][i4 * 4 + 2] * inv, R.o[db][i4 * 4 + 3] * inv};
      *(floatx4_t*)(stage + n * G::OUT_STRIDE + d0 * 4) = w;
    }
  wave_lds_fence();
  const int64_t r0 = (int64_t)row_block * BM + wave * 32;
  auto row_address = [&](int rr) -> char* {
    const uint64_t x = (uint64_t)o_row;
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, rr, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), rr, 64);
    return (char*)((uint64_t)hi << 32 | lo);
  };
  if constexpr (ACC) {
    // The stored row (fp32, o_row) times its weight is added to the step's row, 4 channels per
    // lane; the sum goes back to its place, or to the final output on the last step.
    const bool to_final = p.final_out != nullptr;  // uniform
    const bool seen_row = l_tot > 0.f;
    constexpr int LPR = D / 4, RPP = 64 / LPR;     // lanes per row, rows per pass
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int rr = pass * RPP + lane / LPR, c = (lane % LPR) * 4;
      float* const old_row = p.acc + (int64_t)__shfl(row_lin, rr, 64) * D + c;
      const float ao = __shfl(a_old, rr, 64);
      const bool touch = (to_final || __shfl((int)seen_row, rr, 64) != 0) && r0 + rr < p.rows;
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
          TO* const o = (TO*)p.final_out + (int64_t)__shfl(row_lin, rr, 64) * D + c;
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
  } else if constexpr (!SPLIT && sizeof(TO) == 2) {
    constexpr int LPR = D / 8, RPP = 64 / LPR;
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int rr = pass * RPP + lane / LPR, c = (lane % LPR) * 8;
      char* const o = row_address(rr);
      const floatx4_t a = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4);
      const floatx4_t b = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4 + 16);
      bf16x8_t w;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        w[x] = static_cast<bf16_t>(a[x]);
        w[4 + x] = static_cast<bf16_t>(b[x]);
      }
      if (r0 + rr < p.rows) *(bf16x8_t*)(o + c * 2) = w;
    }
  } else {
    constexpr int LPR = D / 4, RPP = 64 / LPR;
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int rr = pass * RPP + lane / LPR, c = (lane % LPR) * 4;
      char* const o = row_address(rr);
      const floatx4_t a = *(const floatx4_t*)(stage + rr * G::OUT_STRIDE + c * 4);
      if (r0 + rr < p.rows) *(floatx4_t*)(o + c * 4) = a;
    }
  }
}

template <int D, typename TO, bool BAND, bool SPLIT, bool ACC = false>
__global__ __launch_bounds__(NTHREADS) void prefill_mfma_kernel(const Params p) {
  prefill_body<D, TO, BAND, SPLIT, ACC, false>(p);
}

// All ring steps of a rank in one launch, each behind its arrival flag (the RING variant).
template <typename TO>
__global__ __launch_bounds__(NTHREADS) void prefill_ring_walk_kernel(const Params p) {
  prefill_body<128, TO, false, false, false, true>(p);
}
