// Merge attention (Appendix B, Equation 4): bandwidth-bound streaming kernel.
//
// Every thread owns one 16-byte slice of one output row and reads the matching
// slice of each of the n_parts partial outputs exactly once, so the HBM traffic
// is the algorithmic minimum: n_parts * (row bytes + 4) in, row bytes (+4) out.
// The n_parts loads of a thread are independent and issued back to back; the
// LSE values of a row are read by all threads of the row (one cache line).
#include "cp_common.h"

namespace cp {
namespace {

struct MergePtrs {
  const void* out[CP_MAX_PARTS];
  const float* lse[CP_MAX_PARTS];
};

template <typename TP, int VEC>
__device__ __forceinline__ void load_vec(const TP* p, float (&x)[VEC]);

template <>
__device__ __forceinline__ void load_vec<float, 4>(const float* p, float (&x)[4]) {
  const floatx4_t t = __builtin_nontemporal_load((const floatx4_t*)p);
  x[0] = t[0]; x[1] = t[1]; x[2] = t[2]; x[3] = t[3];
}
template <>
__device__ __forceinline__ void load_vec<bf16_t, 8>(const bf16_t* p, float (&x)[8]) {
  const bf16x8_t t = __builtin_nontemporal_load((const bf16x8_t*)p);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = static_cast<float>(t[i]);
}

template <typename TO, int VEC>
__device__ __forceinline__ void store_vec(TO* p, const float (&x)[VEC]);
template <>
__device__ __forceinline__ void store_vec<float, 4>(float* p, const float (&x)[4]) {
  floatx4_t t = {x[0], x[1], x[2], x[3]};
  *(floatx4_t*)p = t;
}
template <>
__device__ __forceinline__ void store_vec<float, 8>(float* p, const float (&x)[8]) {
  floatx4_t a = {x[0], x[1], x[2], x[3]}, b = {x[4], x[5], x[6], x[7]};
  ((floatx4_t*)p)[0] = a;
  ((floatx4_t*)p)[1] = b;
}
template <>
__device__ __forceinline__ void store_vec<bf16_t, 4>(bf16_t* p, const float (&x)[4]) {
  bf16x4_t t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = static_cast<bf16_t>(x[i]);
  *(bf16x4_t*)p = t;
}
template <>
__device__ __forceinline__ void store_vec<bf16_t, 8>(bf16_t* p, const float (&x)[8]) {
  bf16x8_t t;
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = static_cast<bf16_t>(x[i]);
  *(bf16x8_t*)p = t;
}

// NP > 0: compile-time part count (fully unrolled); NP == 0: run-time count.
template <typename TP, typename TO, int VEC, int NP>
__global__ __launch_bounds__(256) void merge_kernel(MergePtrs ptrs, int n_parts_rt, int64_t rows,
                                                     int head_dim, TO* __restrict__ out,
                                                     float* __restrict__ lse_out) {
  const int n_parts = NP > 0 ? NP : n_parts_rt;
  const int vec_per_row = head_dim / VEC;
  const int64_t n_vec = rows * vec_per_row;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n_vec;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = idx / vec_per_row;
    const int col = (int)(idx - row * vec_per_row) * VEC;

    // With a compile-time part count the LSE values stay in registers; with a run-time
    // count they are read twice (a per-thread array indexed at run time would live in scratch).
    float lmax = -INFINITY;
    float lv[NP > 0 ? NP : 1];
#pragma unroll
    for (int s = 0; s < n_parts; ++s) {
      const float x = ptrs.lse[s][row];
      if (NP > 0) lv[NP > 0 ? s : 0] = x;
      lmax = fmaxf(lmax, x);
    }
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    float den = 0.f;
    if (lmax != -INFINITY) {
#pragma unroll
      for (int s = 0; s < n_parts; ++s) {
        const float x = NP > 0 ? lv[NP > 0 ? s : 0] : ptrs.lse[s][row];
        const float w = __expf(x - lmax);  // exp(-inf) = 0 for empty partials
        den += w;
        // a partial with zero weight is not read (its O may hold anything)
        if (w != 0.f) {
          const TP* p = (const TP*)ptrs.out[s] + row * head_dim;
          float x4[VEC];
          load_vec<TP, VEC>(p + col, x4);
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[i] = fmaf(w, x4[i], acc[i]);
        }
      }
      const float inv = 1.f / den;
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] *= inv;
    }
    store_vec<TO, VEC>(out + row * head_dim + col, acc);
    if (lse_out != nullptr && col == 0)
      lse_out[row] = lmax == -INFINITY ? -INFINITY : lmax + __logf(den);
  }
}

// Partials at a constant stride (split-KV scratch, ring slots), every row written: finite
// values and LSE = -inf where a part saw nothing. Bound by latency on few rows and by bandwidth
// on many; in both a thread wants all its requests out at once: it asks for the LSE values of
// all parts and for up to 16 data vectors back to back, and the arithmetic is branch-free (a
// branch on the weights would pull the loads behind the wait for the LSE values). NP is the
// part count rounded up; parts past the end repeat the last one with weight zero. The addresses
// step from part to part: as products of the part's index they do not fit the scalar registers at
// 64 parts (one sequence of 131072 keys: 7.6 -> 5.4 us). A single rank's pointers are scalar
// loads with the other arguments; looked up by rank they are a vector load that everything else
// waits for.
template <typename TP, typename TO, int VEC, int NP>
__global__ __launch_bounds__(256) void merge_table_kernel(const MergeTable m, int row_shift) {
  constexpr int BATCH = NP < 16 ? NP : 16;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = idx >> row_shift;                          // head_dim / VEC threads per row
  const int col = ((int)idx & ((1 << row_shift) - 1)) * VEC;
  const int head_dim = VEC << row_shift;
  if (row >= m.rows) return;
  const void* part = m.part[0];
  const float* part_lse = m.part_lse[0];
  void* out = m.out[0];
  float* lse_out = m.lse[0];
  int64_t r = row;
  if (m.n_ranks > 1) {
    int a = 0;
#pragma unroll 8
    for (int i = 1; i < m.n_ranks; ++i) a += row >= m.row_begin[i];
    part = m.part[a];
    part_lse = m.part_lse[a];
    out = m.out[a];
    lse_out = m.lse[a];
    r -= m.row_begin[a];
  }
  const int n_parts = m.n_parts;
  const int64_t first = (int64_t)blockIdx.y * n_parts;
  const float* lse = part_lse + first * m.part_lse_elems + r;
  const char* src = (const char*)part + first * m.part_bytes +
                    (r * head_dim + col) * (int64_t)sizeof(TP);
  // (the part count anew for every use: the comparisons with it, kept, would fill the scalar
  // registers)
  auto count = [n_parts] {
    int n = n_parts;
    asm volatile("" : "+s"(n));
    return n;
  };
  float lv[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) {
    lv[s] = *lse;
    lse += s + 1 < count() ? m.part_lse_elems : 0;
  }
  float acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  float den = 0.f, lmax = -INFINITY;
#pragma unroll
  for (int b = 0; b < NP / BATCH; ++b) {
    float xs[BATCH][VEC];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      load_vec<TP, VEC>((const TP*)src, xs[i]);
      src += b * BATCH + i + 1 < count() ? m.part_bytes : 0;
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the requests together, ahead of the arithmetic
    if (b == 0) {
#pragma unroll
      for (int s = 0; s < NP; ++s) {
        if (s >= count()) lv[s] = -INFINITY;
        lmax = fmaxf(lmax, lv[s]);
      }
    }
    const bool any = lmax != -INFINITY;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float w = any ? __expf(lv[b * BATCH + i] - lmax) : 0.f;  // exp(-inf) = 0
      den += w;
#pragma unroll
      for (int c = 0; c < VEC; ++c) acc[c] = fmaf(w, xs[i][c], acc[c]);
    }
  }
  const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
  for (int c = 0; c < VEC; ++c) acc[c] *= inv;
  char* const o = (char*)out + (int64_t)blockIdx.y * m.group_out_bytes;
  store_vec<TO, VEC>((TO*)o + r * head_dim + col, acc);
  if (lse_out != nullptr && col == 0)
    lse_out[(int64_t)blockIdx.y * m.group_lse_elems + r] =
        den > 0.f ? lmax + __logf(den) : -INFINITY;
}

// fp32 partials of several groups (KV shards whose results are kept apart): the parts of every group
// merged into the group's result, as merge_table_kernel does it, and Equation 4 over the groups along
// the way, over what is stored: a bf16 slot's values are rounded first, and every bit is that of two
// launches. In those the groups' results are read again, and the second one starts behind the first.
// Bound by its chain of arguments, LSE and vectors. A thread has the 16 vectors of 16 / NP groups in
// flight at once. The LSE of all parts of a row are asked for ahead of them, by all threads of the row
// together, which keep them in LDS; then they work out a group's weight or two each. us (traced), two
// launches and one: 2048 rows of 16 groups of 2 parts 11.0 + 6.0 and 12.2, 1024 rows of 16 of 4 9.3 +
// 4.8 and 11.6, of 8 of 8 8.3 + 4.3 and 9.2, of 4 of 16 7.9 + 4.7 and 8.6.
// Up to 64 parts, for which the row's LSE have room (whole calls, us: 1008 rows of 7 groups of 9 46.7
// and 42.5, of 9 of 7 45.7 and 41.4). A thread walks the groups: with more of them it loses to the
// second launch sooner or later (512 rows of 16 of 8 13.4 and 14.8, in a form without LDS).
constexpr int kMaxGroupParts = 64;
struct GroupsOut {
  void* out[kMaxTable];
  float* lse[kMaxTable];
};
template <typename TS, typename TO, int NP>
__global__ __launch_bounds__(256) void merge_over_groups_kernel(const MergeTable m, const GroupsOut f,
                                                                int row_shift) {
  constexpr int VEC = 4, GB = 16 / NP;
  constexpr int MIN_ROW = 16;                         // threads per row at least (64 channels)
  constexpr int OWN = kMaxTable / MIN_ROW;            // groups a thread looks up at most
  constexpr int OWN_PARTS = kMaxGroupParts / MIN_ROW; // and parts
  __shared__ float lse_of[256 / MIN_ROW][kMaxGroupParts];
  const int touched = touch_arguments<MergeTable>();
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = idx >> row_shift;                          // head_dim / VEC threads per row
  const int per_row = 1 << row_shift, own = (int)threadIdx.x & (per_row - 1);
  const int col = own * VEC, head_dim = VEC << row_shift;
  asm volatile("" ::"v"(touched));
  if (row >= m.rows) return;   // (all threads of a row: blocks hold whole rows)
  int a = 0;
#pragma unroll 8
  for (int i = 1; i < m.n_ranks; ++i) a += row >= m.row_begin[i];
  const int64_t r = row - m.row_begin[a];
  const float* const lse0 = m.part_lse[a] + r;
  const char* const src0 = (const char*)m.part[a] + (r * head_dim + col) * (int64_t)sizeof(float);
  char* const slot0 = (char*)m.out[a];
  float* const slot_lse = m.lse[a];
  const int n_all = m.n_groups * m.n_parts;
  float* const lse_row = lse_of[threadIdx.x >> row_shift];   // (this wavefront's own)
  float own_lse[OWN_PARTS];
#pragma unroll
  for (int k = 0; k < OWN_PARTS; ++k)
    own_lse[k] = lse0[min(own + k * per_row, n_all - 1) * m.part_lse_elems];
  // Weights of a group's parts from their LSE, and the sum of the weights; returns the group's LSE.
  auto weights = [&](int g, float (&w)[NP], float& den) {
    float lmax = -INFINITY;
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const float x = lse_row[g * m.n_parts + min(s, m.n_parts - 1)];
      w[s] = s < m.n_parts ? x : -INFINITY;
      lmax = fmaxf(lmax, w[s]);
    }
    const bool any = lmax != -INFINITY;
    den = 0.f;
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      w[s] = any ? __expf(w[s] - lmax) : 0.f;  // exp(-inf) = 0
      den += w[s];
    }
    return den > 0.f ? lmax + __logf(den) : -INFINITY;
  };
  float group_w[OWN] = {};   // of the groups `own` and `own` + per_row
  float total[VEC] = {0.f, 0.f, 0.f, 0.f}, total_den = 0.f, total_max = -INFINITY;
  for (int g0 = 0; g0 < m.n_groups; g0 += GB) {
    float x[GB][NP][VEC];
#pragma unroll
    for (int g = 0; g < GB; ++g)
#pragma unroll
      for (int s = 0; s < NP; ++s) {   // (clamped: past the end the last one, dropped below)
        const int64_t k = (int64_t)min(g0 + g, m.n_groups - 1) * m.n_parts + min(s, m.n_parts - 1);
        load_vec<float, VEC>((const float*)(src0 + k * m.part_bytes), x[g][s]);
      }
    __builtin_amdgcn_sched_barrier(0);  // keep the requests together, ahead of the arithmetic
    if (g0 == 0) {
#pragma unroll
      for (int k = 0; k < OWN_PARTS; ++k)
        if (own + k * per_row < n_all) lse_row[own + k * per_row] = own_lse[k];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
      for (int k = 0; k < OWN; ++k) {
        const int g = own + k * per_row;
        group_w[k] = -INFINITY;
        if (g >= m.n_groups) continue;
        float w[NP], den;
        group_w[k] = weights(g, w, den);
        if (slot_lse != nullptr) slot_lse[(int64_t)g * m.group_lse_elems + r] = group_w[k];
        total_max = fmaxf(total_max, group_w[k]);
      }
      for (int o = per_row >> 1; o > 0; o >>= 1) total_max = fmaxf(total_max, __shfl_xor(total_max, o, 64));
#pragma unroll
      for (int k = 0; k < OWN; ++k)
        group_w[k] = total_max != -INFINITY ? __expf(group_w[k] - total_max) : 0.f;
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const int at = g0 + g;
      if (at >= m.n_groups) break;   // uniform
      float part_w[NP], den;
      weights(at, part_w, den);
      float acc[VEC] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NP; ++s)
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[c] = fmaf(part_w[s], x[g][s][c], acc[c]);
      const float inv = den > 0.f ? 1.f / den : 0.f;
      const float w = __shfl(at < per_row ? group_w[0] : group_w[1], at & (per_row - 1), per_row);
      total_den += w;
#pragma unroll
      for (int c = 0; c < VEC; ++c) {
        acc[c] = to_float(from_float<TS>(acc[c] * inv));   // (what the slot holds)
        total[c] = fmaf(w, acc[c], total[c]);
      }
      store_vec<TS, VEC>((TS*)(slot0 + (int64_t)at * m.group_out_bytes) + r * head_dim + col, acc);
    }
  }
  const float inv = total_den > 0.f ? 1.f / total_den : 0.f;
#pragma unroll
  for (int c = 0; c < VEC; ++c) total[c] *= inv;
  store_vec<TO, VEC>((TO*)f.out[a] + r * head_dim + col, total);
  if (f.lse[a] != nullptr && col == 0)
    f.lse[a][r] = total_den > 0.f ? total_max + __logf(total_den) : -INFINITY;
}

template <typename TP, typename TO, int VEC>
int launch_np(const MergePtrs& ptrs, int n_parts, int64_t rows, int head_dim, void* out,
              float* lse_out, hipStream_t stream) {
  const int64_t n_vec = rows * (head_dim / VEC);
  if (n_vec == 0) return CP_OK;
  int64_t blocks = (n_vec + 255) / 256;
  const int64_t cap = 256 * 32;  // grid-stride beyond 32 workgroups per CU
  if (blocks > cap) blocks = cap;
#define CP_MERGE_LAUNCH(NP)                                                                  \
  hipLaunchKernelGGL((merge_kernel<TP, TO, VEC, NP>), dim3((unsigned)blocks), dim3(256), 0,  \
                     stream, ptrs, n_parts, rows, head_dim, (TO*)out, lse_out)
  switch (n_parts) {
    case 2: CP_MERGE_LAUNCH(2); break;
    case 4: CP_MERGE_LAUNCH(4); break;
    case 8: CP_MERGE_LAUNCH(8); break;
    case 16: CP_MERGE_LAUNCH(16); break;
    default: CP_MERGE_LAUNCH(0); break;
  }
#undef CP_MERGE_LAUNCH
  return check_launch();
}

}  // namespace

int launch_merge(int64_t rows, int32_t head_dim, int32_t n_parts, const void* const* outs,
                 const float* const* lses, int32_t part_dtype, void* out, int32_t out_dtype,
                 float* lse_out, hipStream_t stream) {
  MergePtrs ptrs;
  for (int s = 0; s < CP_MAX_PARTS; ++s) {
    ptrs.out[s] = s < n_parts ? outs[s] : nullptr;
    ptrs.lse[s] = s < n_parts ? lses[s] : nullptr;
  }
  if (part_dtype == CP_FP32) {
    if (out_dtype == CP_FP32)
      return launch_np<float, float, 4>(ptrs, n_parts, rows, head_dim, out, lse_out, stream);
    return launch_np<float, bf16_t, 4>(ptrs, n_parts, rows, head_dim, out, lse_out, stream);
  }
  if (out_dtype == CP_FP32)
    return launch_np<bf16_t, float, 8>(ptrs, n_parts, rows, head_dim, out, lse_out, stream);
  return launch_np<bf16_t, bf16_t, 8>(ptrs, n_parts, rows, head_dim, out, lse_out, stream);
}

namespace {

template <typename TP, typename TO, int VEC>
int launch_table_t(const MergeTable& m, int32_t head_dim, hipStream_t stream) {
  const int per_row = head_dim / VEC;   // 64 or 128 channels: a power of two
  if (per_row < 1 || (per_row & (per_row - 1)) != 0 || head_dim % VEC != 0)
    return CP_ERR_UNSUPPORTED;
  const int64_t n_vec = m.rows * per_row;
  if (n_vec == 0) return CP_OK;
  // one wavefront per workgroup while that is what spreads the rows over the 256 CUs
  const int threads = n_vec * m.n_groups < 256 * 4 * 256 ? 64 : 256;
  const int64_t blocks = (n_vec + threads - 1) / threads;
  if (blocks > 0x7fffffffLL) return CP_ERR_SHAPE;
  const dim3 grid((unsigned)blocks, m.n_groups);
#define CP_MERGE_TABLE(NP)                                                                     \
  hipLaunchKernelGGL((merge_table_kernel<TP, TO, VEC, NP>), grid, dim3(threads), 0, stream, m, \
                     __builtin_ctz((unsigned)per_row))
  if (m.n_parts <= 2) CP_MERGE_TABLE(2);
  else if (m.n_parts <= 4) CP_MERGE_TABLE(4);
  else if (m.n_parts <= 8) CP_MERGE_TABLE(8);
  else if (m.n_parts <= 16) CP_MERGE_TABLE(16);
  else if (m.n_parts <= 32) CP_MERGE_TABLE(32);
  else CP_MERGE_TABLE(64);
#undef CP_MERGE_TABLE
  return check_launch();
}

}  // namespace

constexpr int64_t kStreamRows = 4096;

int launch_merge_table(const MergeTable& m, int32_t head_dim, int32_t part_dtype,
                       int32_t out_dtype, hipStream_t stream) {
  if (m.n_parts < 1 || m.n_parts > CP_MAX_PARTS || m.n_groups < 1 || m.n_groups > 65535)
    return CP_ERR_SHAPE;
  // Many rows of one rank: bound by bandwidth and not by latency, and the streaming kernel with its
  // compile-time part counts moves them faster (a call of 1000 queries of 16 heads, 4 parts of 16000
  // rows: 30.3 us with the kernel above, 28.4).
  const int n = m.n_parts;
  if (m.n_ranks == 1 && m.n_groups == 1 && m.rows >= kStreamRows &&
      (n == 2 || n == 4 || n == 8 || n == 16)) {
    const void* outs[CP_MAX_PARTS];
    const float* lses[CP_MAX_PARTS];
    for (int i = 0; i < n; ++i) {
      outs[i] = (const char*)m.part[0] + i * m.part_bytes;
      lses[i] = m.part_lse[0] + i * m.part_lse_elems;
    }
    return launch_merge(m.rows, head_dim, n, outs, lses, part_dtype, m.out[0], out_dtype, m.lse[0],
                        stream);
  }
  if (part_dtype == CP_FP32)
    return out_dtype == CP_FP32 ? launch_table_t<float, float, 4>(m, head_dim, stream)
                                : launch_table_t<float, bf16_t, 4>(m, head_dim, stream);
  return out_dtype == CP_FP32 ? launch_table_t<bf16_t, float, 8>(m, head_dim, stream)
                              : launch_table_t<bf16_t, bf16_t, 8>(m, head_dim, stream);
}

bool merge_over_groups_applies(const MergeTable& m) {
  return m.n_groups > 1 && m.n_parts > 1 && m.n_parts <= 16 && m.n_groups * m.n_parts <= kMaxGroupParts;
}

namespace {

template <typename TS, typename TO>
int launch_over_groups_t(const MergeTable& m, int32_t head_dim, const GroupsOut& f,
                         hipStream_t stream) {
  if (head_dim != 64 && head_dim != 128) return CP_ERR_UNSUPPORTED;
  const int per_row = head_dim / 4;
  const int64_t n_vec = m.rows * per_row;
  if (n_vec == 0) return CP_OK;
  // one wavefront per workgroup while that is what spreads the rows over the 256 CUs
  const int threads = n_vec < 256 * 4 * 256 ? 64 : 256;
  const int64_t blocks = (n_vec + threads - 1) / threads;
  if (blocks > 0x7fffffffLL) return CP_ERR_SHAPE;
#define CP_MERGE_GROUPS(NP)                                                                    \
  hipLaunchKernelGGL((merge_over_groups_kernel<TS, TO, NP>), dim3((unsigned)blocks),            \
                     dim3(threads), 0, stream, m, f, __builtin_ctz((unsigned)per_row))
  if (m.n_parts <= 2) CP_MERGE_GROUPS(2);
  else if (m.n_parts <= 4) CP_MERGE_GROUPS(4);
  else if (m.n_parts <= 8) CP_MERGE_GROUPS(8);
  else CP_MERGE_GROUPS(16);
#undef CP_MERGE_GROUPS
  return check_launch();
}

}  // namespace

int launch_merge_over_groups(const MergeTable& m, int32_t head_dim, int32_t out_dtype,
                             const OverShards& over, hipStream_t stream) {
  GroupsOut f = {};
  for (int a = 0; a < m.n_ranks; ++a) {
    f.out[a] = over.out[a];
    f.lse[a] = over.lse[a];
  }
  if (out_dtype == CP_FP32)
    return over.dtype == CP_FP32 ? launch_over_groups_t<float, float>(m, head_dim, f, stream)
                                 : launch_over_groups_t<float, bf16_t>(m, head_dim, f, stream);
  return over.dtype == CP_FP32 ? launch_over_groups_t<bf16_t, float>(m, head_dim, f, stream)
                               : launch_over_groups_t<bf16_t, bf16_t>(m, head_dim, f, stream);
}

}  // namespace cp
