// Packed (variable-length) batches for the MFMA prefill kernel (Algorithm 2's fused
// variable-length inputs, Section 3.4).
//
// The prefill kernel masks with one position per token. Several sequences packed into one
// call are told apart by moving every sequence into its own position range: sequence b is
// shifted by base_b = sum over b' < b of span_b', where span_b' = 1 + the largest position
// any query or key of sequence b' carries. A key is then visible to a query iff
//   q_lo <= kv_enc <= q_hi,   q_lo = base_b,   q_hi = base_b + q_pos,   kv_enc = base_b + kv_pos,
// which is the causal mask inside the sequence and nothing across sequences. Padding keeps
// its meaning: a padded key stays at INT32_MAX, a padded query gets the empty range [0, -1].
// The shifted positions must stay below 2^31 - 1 (sum of the spans); beyond that the scan
// saturates and the later sequences see nothing.
//
// The ranks of a ring are shifted together: sequence b's span is taken over all ranks' shares of
// it, so that one launch attends from any rank's queries to any shard's keys. Three small
// launches (a launch costs more than the work), two for batches of up to kScanHere sequences.
#include "cp_common.h"

namespace cp {
namespace {

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int kScanHere = 1024;  // batches up to this size: the encode kernel scans the spans

struct SeqTable {
  const int32_t* q_pos[kMaxTable];
  const int32_t* kv_pos[kMaxTable];
  const int32_t* cu_q[kMaxTable];
  const int32_t* cu_kv[kMaxTable];
  int32_t tok_begin[kMaxTable + 1];  // queries: ranks back to back
  int32_t key_begin[kMaxTable + 1];  // keys: shards back to back
  int32_t n_ranks, n_shards, batch;
};

// span[b] = 1 + the largest position of sequence b; one workgroup per sequence
__global__ __launch_bounds__(256) void seq_span_kernel(const SeqTable t,
                                                        int32_t* __restrict__ span) {
  __shared__ int32_t red[4];
  const int b = blockIdx.x;
  int32_t m = -1;
  for (int s = 0; s < t.n_shards; ++s) {
    const int32_t* const pos = t.kv_pos[s];
    const int hi = t.cu_kv[s][b + 1];
    for (int i = t.cu_kv[s][b] + threadIdx.x; i < hi; i += 256) {
      const int32_t x = pos[i];
      if (x != CP_POS_PAD_KV) m = max(m, x);
    }
  }
  for (int a = 0; a < t.n_ranks; ++a) {
    const int32_t* const pos = t.q_pos[a];
    const int hi = t.cu_q[a][b + 1];
    for (int i = t.cu_q[a][b] + threadIdx.x; i < hi; i += 256) m = max(m, pos[i]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) span[b] = max(max(red[0], red[1]), max(red[2], red[3])) + 1;
}

// base[b] = exclusive prefix of span, saturating; one thread (batches are short lists)
__global__ void seq_base_kernel(const int32_t* __restrict__ span, int32_t batch,
                                int32_t* __restrict__ base) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int64_t acc = 0;
  for (int b = 0; b < batch; ++b) {
    base[b] = (int32_t)min<int64_t>(acc, INT32_MAX - 1);
    acc += span[b];
  }
}

// sequence of packed token i: last b with cu[b] <= i
__device__ __forceinline__ int seq_of(const int32_t* __restrict__ cu, int batch, int i) {
  int lo = 0, hi = batch;  // invariant: cu[lo] <= i < cu[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// SCAN: `base` is span, and every workgroup forms the prefix sums in LDS.
template <bool SCAN>
__global__ __launch_bounds__(256) void seq_encode_kernel(const SeqTable t,
                                                          const int32_t* __restrict__ base,
                                                          int32_t* __restrict__ q_hi,
                                                          int32_t* __restrict__ q_lo,
                                                          int32_t* __restrict__ kv_enc) {
  __shared__ int64_t pre[SCAN ? kScanHere : 1];
  if constexpr (SCAN) {
    // four sequences per thread, the threads' sums scanned by doubling steps
    __shared__ int64_t sums[256];
    const int b0 = threadIdx.x * 4;
    int64_t x[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = sum;
      sum += b0 + i < t.batch ? base[b0 + i] : 0;
    }
    sums[threadIdx.x] = sum;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
      const int64_t y = (int)threadIdx.x >= o ? sums[threadIdx.x - o] : 0;
      __syncthreads();
      sums[threadIdx.x] += y;
      __syncthreads();
    }
    const int64_t before = sums[threadIdx.x] - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[b0 + i] = min<int64_t>(before + x[i], INT32_MAX - 1);
    __syncthreads();
  }
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < t.tok_begin[t.n_ranks]) {
    int a = 0;
    for (int r = 1; r < t.n_ranks; ++r) a += i >= t.tok_begin[r];
    const int li = i - t.tok_begin[a];
    const int32_t x = t.q_pos[a][li];
    const int b = seq_of(t.cu_q[a], t.batch, li);
    const int64_t s = SCAN ? pre[b] : base[b];
    const bool ok = x >= 0 && s + x < INT32_MAX;
    q_hi[i] = ok ? (int32_t)(s + x) : CP_POS_PAD_Q;
    q_lo[i] = ok ? (int32_t)s : 0;
  }
  if (i < t.key_begin[t.n_shards]) {
    int a = 0;
    for (int r = 1; r < t.n_shards; ++r) a += i >= t.key_begin[r];
    const int li = i - t.key_begin[a];
    const int32_t x = t.kv_pos[a][li];
    const int b = seq_of(t.cu_kv[a], t.batch, li);
    const int64_t s = SCAN ? pre[b] : base[b];
    kv_enc[i] = (x == CP_POS_PAD_KV || s + x >= INT32_MAX) ? CP_POS_PAD_KV : (int32_t)(s + x);
  }
}

struct Layout {
  size_t span_off, base_off, q_hi_off, q_lo_off, kv_off, total;
};
Layout layout(int32_t batch, int64_t total_q, int64_t total_kv) {
  Layout w;
  w.span_off = 0;
  w.base_off = round256((size_t)batch * 4);
  w.q_hi_off = w.base_off + round256((size_t)batch * 4);
  w.q_lo_off = w.q_hi_off + round256((size_t)total_q * 4);
  w.kv_off = w.q_lo_off + round256((size_t)total_q * 4);
  w.total = w.kv_off + round256((size_t)total_kv * 4);
  return w;
}

}  // namespace

size_t varseq_workspace_bytes(int32_t batch, int64_t total_q, int64_t total_kv) {
  return layout(batch, total_q, total_kv).total;
}

int launch_varseq_encode(int32_t batch, int64_t total_kv, AttnTable& t, const int32_t* const* cu_q,
                         const int32_t* const* cu_kv, void* workspace, const int32_t** q_lo,
                         hipStream_t stream) {
  const int64_t total_q = t.tok_begin[t.n_ranks];
  if (total_kv > 0x7fffffffLL - 256 || total_q > 0x7fffffffLL - 256) return CP_ERR_SHAPE;
  const Layout w = layout(batch, total_q, total_kv);
  char* ws = (char*)workspace;
  int32_t* span = (int32_t*)(ws + w.span_off);
  int32_t* base = (int32_t*)(ws + w.base_off);
  int32_t* q_hi = (int32_t*)(ws + w.q_hi_off);
  int32_t* kv_enc = (int32_t*)(ws + w.kv_off);
  *q_lo = (const int32_t*)(ws + w.q_lo_off);
  SeqTable s = {};
  s.n_ranks = t.n_ranks; s.n_shards = t.n_shards; s.batch = batch;
  int32_t keys = 0;
  for (int a = 0; a < t.n_ranks; ++a) {
    s.q_pos[a] = t.q_pos[a]; s.cu_q[a] = cu_q[a]; s.tok_begin[a] = t.tok_begin[a];
    t.q_pos[a] = q_hi + t.tok_begin[a];
  }
  s.tok_begin[t.n_ranks] = t.tok_begin[t.n_ranks];
  for (int b = 0; b < t.n_shards; ++b) {
    s.kv_pos[b] = t.kv_pos[b]; s.cu_kv[b] = cu_kv[b]; s.key_begin[b] = keys;
    t.kv_pos[b] = kv_enc + keys;
    keys += t.n_kv[b];
  }
  s.key_begin[t.n_shards] = keys;
  hipLaunchKernelGGL(seq_span_kernel, dim3(batch), dim3(256), 0, stream, s, span);
  const int64_t n = std::max<int64_t>(total_q, keys);
  const dim3 grid((unsigned)((n + 255) / 256));
  if (batch <= kScanHere) {
    if (n > 0)
      hipLaunchKernelGGL(seq_encode_kernel<true>, grid, dim3(256), 0, stream, s, span, q_hi,
                         (int32_t*)*q_lo, kv_enc);
  } else {
    hipLaunchKernelGGL(seq_base_kernel, dim3(1), dim3(64), 0, stream, span, batch, base);
    if (n > 0)
      hipLaunchKernelGGL(seq_encode_kernel<false>, grid, dim3(256), 0, stream, s, base, q_hi,
                         (int32_t*)*q_lo, kv_enc);
  }
  return check_launch();
}

}  // namespace cp
