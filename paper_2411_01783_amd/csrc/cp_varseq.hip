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
// it, so that one launch attends from any rank's queries to any shard's keys. One small launch (a
// launch costs more than the work) for few sequences (encode_in_one_launch), two for batches of up to
// kScanHere sequences, else three.
#include "cp_common.h"
#include "cp_launch_rules.h"

namespace cp {
namespace {

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int kScanHere = 1024;  // batches up to this size: the encode kernel scans the spans
constexpr int kBatchHere = 64;   // a lane each scans the spans (encode_in_one_launch takes fewer)

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

__device__ __forceinline__ void encode_q(int32_t x, int64_t base, int32_t* hi, int32_t* lo) {
  const bool ok = x >= 0 && base + x < INT32_MAX;
  *hi = ok ? (int32_t)(base + x) : CP_POS_PAD_Q;
  *lo = ok ? (int32_t)base : 0;
}
__device__ __forceinline__ int32_t encode_kv(int32_t x, int64_t base) {
  return (x == CP_POS_PAD_KV || base + x >= INT32_MAX) ? CP_POS_PAD_KV : (int32_t)(base + x);
}

// Spans and encoded positions in one launch: every workgroup takes the spans of all sequences
// itself, from positions that lie in L2 after the first workgroup, and encodes its 1024 tokens. A
// wavefront takes every 16th piece (a sequence's share on one rank), one after the other; the
// boundaries of its pieces are fetched by its lanes together (the rule leaves it 23 at most), so that a
// piece costs one round trip per 512 positions. Bound by those round trips. Two prompts of 32 to 64 tokens 21.2 -> 18.4 us a call, six of 200 to 3000
// over 4 ranks 113.7 -> 109.2, twelve of 200 to 600 over 2 ranks 69.0 -> 66.6 (two launches before).
__global__ __launch_bounds__(1024) void seq_encode_all_kernel(const SeqTable t,
                                                               int32_t* __restrict__ q_hi,
                                                               int32_t* __restrict__ q_lo,
                                                               int32_t* __restrict__ kv_enc) {
  __shared__ int32_t top[kBatchHere];   // largest position, then base
  const int touched = touch_arguments<SeqTable>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < kBatchHere) top[tid] = -1;
  const int n_lists = t.n_shards + t.n_ranks, n_pieces = n_lists * t.batch;
  const int i = blockIdx.x * 1024 + tid;
  // this thread's own tokens, asked for before anything is waited for
  int ql = 0, kl = 0;
  int32_t qx = 0, kx = 0;
  const bool has_q = i < t.tok_begin[t.n_ranks], has_k = i < t.key_begin[t.n_shards];
  // (scalar loads and selects: looked up by lane, the list's arguments are another latency. Five prompts
  // of 100 to 900 tokens over 2 ranks 6.2 -> 5.3 us.)
  const int32_t *q_cu = t.cu_q[0], *k_cu = t.cu_kv[0];
  if (has_q) {
    const int32_t* pos = t.q_pos[0];
    int begin = 0;
#pragma unroll 4
    for (int r = 1; r < t.n_ranks; ++r) {
      const int x = t.tok_begin[r];
      const int32_t *const y = t.q_pos[r], *const c = t.cu_q[r];
      const bool in = i >= x;
      begin = in ? x : begin;
      pos = in ? y : pos;
      q_cu = in ? c : q_cu;
    }
    ql = i - begin;
    qx = pos[ql];
  }
  if (has_k) {
    const int32_t* pos = t.kv_pos[0];
    int begin = 0;
#pragma unroll 4
    for (int r = 1; r < t.n_shards; ++r) {
      const int x = t.key_begin[r];
      const int32_t *const y = t.kv_pos[r], *const c = t.cu_kv[r];
      const bool in = i >= x;
      begin = in ? x : begin;
      pos = in ? y : pos;
      k_cu = in ? c : k_cu;
    }
    kl = i - begin;
    kx = pos[kl];
  }
  asm volatile("" ::"v"(touched));
  __syncthreads();
  const int mine = wave + lane * 16;
  int lo = 0, hi = 0, list = 0, seq = 0;
  if (mine < n_pieces) {
    list = mine / t.batch;
    seq = mine - list * t.batch;
    const int32_t* const cu = list < t.n_shards ? t.cu_kv[list] : t.cu_q[list - t.n_shards];
    lo = cu[seq];
    hi = cu[seq + 1];
  }
  const int n = (n_pieces - wave + 15) / 16;
  for (int j = 0; j < n; ++j) {
    const int l = __builtin_amdgcn_readlane(list, j), b = __builtin_amdgcn_readlane(seq, j);
    const int first = __builtin_amdgcn_readlane(lo, j), end = __builtin_amdgcn_readlane(hi, j);
    const bool keys = l < t.n_shards;
    const int32_t* const pos = keys ? t.kv_pos[l] : t.q_pos[l - t.n_shards];
    int m = -1;
    for (int k = first; k < end; k += 8 * 64) {
      int32_t x[8];   // (clamped, not skipped: all eight are on their way at once)
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = pos[min(k + u * 64 + lane, end - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (!keys || x[u] != CP_POS_PAD_KV) m = max(m, x[u]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (lane == 0) atomicMax(&top[b], m);   // (LDS)
  }
  __syncthreads();
  // exclusive prefix of the spans, saturating: a sequence per lane of the first wavefront
  if (wave == 0) {
    const int64_t span = lane < t.batch ? (int64_t)top[lane] + 1 : 0;
    int64_t sum = span;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up(sum, o, 64);
      if (lane >= o) sum += y;
    }
    top[lane] = (int32_t)min<int64_t>(sum - span, INT32_MAX - 1);
  }
  __syncthreads();
  if (has_q) encode_q(qx, top[seq_of(q_cu, t.batch, ql)], q_hi + i, q_lo + i);
  if (has_k) kv_enc[i] = encode_kv(kx, top[seq_of(k_cu, t.batch, kl)]);
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
    encode_q(x, SCAN ? pre[b] : base[b], q_hi + i, q_lo + i);
  }
  if (i < t.key_begin[t.n_shards]) {
    int a = 0;
    for (int r = 1; r < t.n_shards; ++r) a += i >= t.key_begin[r];
    const int li = i - t.key_begin[a];
    const int32_t x = t.kv_pos[a][li];
    const int b = seq_of(t.cu_kv[a], t.batch, li);
    kv_enc[i] = encode_kv(x, SCAN ? pre[b] : base[b]);
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
  const int64_t n = std::max<int64_t>(total_q, keys);
  if (encode_in_one_launch(batch, t.n_ranks + t.n_shards, total_q + keys)) {
    if (n > 0)
      hipLaunchKernelGGL(seq_encode_all_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(1024), 0,
                         stream, s, q_hi, (int32_t*)*q_lo, kv_enc);
    return check_launch();
  }
  hipLaunchKernelGGL(seq_span_kernel, dim3(batch), dim3(256), 0, stream, s, span);
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
