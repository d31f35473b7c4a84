// Construction of the draft token tree from the draft model's outputs (the step before the
// verification; the paper drafts in the EAGLE-3 manner, Section 3.1, and leaves the arrangement of
// the drafted tokens open: this is the dynamic tree of that line of work).
//
//   topk_logprob   per row of draft logits: the k best tokens (ties: lower id) and their
//                  log-probabilities.  Pass 1, one workgroup per (row, chunk of the vocabulary):
//                  the chunk is read from memory once, reduced to its maximum and its sum of
//                  exponentials, and its k best entries are picked as order-preserving integer
//                  keys.  Pass 2, one workgroup per row: the k best of the chunks' winners and
//                  the row's logsumexp from the chunks' partials.
//   tree_grow      one level: scores of the new candidates (ONE float32 addition each,
//                  parent's score + log-probability), the K best of them become the frontier.
//   tree_finalize  re-ranking of all candidates, the N - 1 best are kept and numbered in
//                  candidate order (parents first); parent, token, depth, ancestor mask per node.
// Ranking is by counting: rank(c) = number of candidates that beat c, where a beats c iff its
// score is higher, or equal with a lower candidate index: a strict total order, so the ranks are
// a permutation and every output slot is written exactly once.
#include "hb_internal.h"

namespace hb {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxTopK = 32;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned long long wg_max_key(unsigned long long x, unsigned long long *red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long y = __shfl_xor(x, off, 64);
    x = y > x ? y : x;
  }
  __syncthreads();  // red may still be read from the previous call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  unsigned long long r = red[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r = red[w] > r ? red[w] : r;
  return r;
}

__device__ __forceinline__ float wg_max_f(float x, float *red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__device__ __forceinline__ float wg_sum_f(float x, float *red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// key of (value, index): larger value first, then lower index; -0 counts as +0
__device__ __forceinline__ unsigned long long sel_key(float v, uint32_t idx) { return argmax_key(v + 0.f, idx); }

// The k largest of the distinct keys[0 .. cnt) into win[0 .. k), largest first, by counting: the
// rank of a key is the number of keys above it.  Slots without a key (cnt < k) are 0.  The caller
// has made keys[] visible; win[] is visible to every thread on return.
__device__ __forceinline__ void rank_select(const unsigned long long *keys, int cnt, int k, unsigned long long *win) {
  if (threadIdx.x < k) win[threadIdx.x] = 0ull;
  __syncthreads();
  for (int i = threadIdx.x; i < cnt; i += kThreads) {
    const unsigned long long mine = keys[i];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < cnt; ++j) rank += keys[j] > mine ? 1 : 0;
    if (rank < k) win[rank] = mine;
  }
  __syncthreads();
}

struct Partial {  // one per (row, chunk), followed in memory by k keys
  float max, sum;
};

// Logits per chunk: 64 per thread, held in registers.  Always the most a workgroup holds: it takes 5
// to 10 us whatever its chunk, and every chunk adds k winners to the merge, whose ranking is quadratic
// (16 rows x 152064 in chunks of 3072: 33 us, of 16384: 13 us).
constexpr int kChunk = 16384;
constexpr int kPerThread = kChunk / kThreads;
constexpr int kListCap = 2048;              // candidates that pass the threshold

// Pass 1 of the top-k: one workgroup per (chunk, row).  The chunk goes from memory straight into
// registers (every load is in flight before the first value is used).  The k best entries are
// found without sorting: a threshold T that at least k values of the chunk reach (from the
// per-thread maxima, see below) is a lower bound of the chunk's k-th largest value, so only values
// >= T can be among the k best; those few are collected in LDS (as order-preserving keys) and
// the k best picked there by counting ranks.
// Many equal values can let more pass than the list holds; then k rounds of a workgroup-wide
// maximum run over the chunk instead (same result, slower).
//
// What bounds it is vector instruction issue, and code that has to stay in the instruction cache.
// The path from registers works by 16-byte pieces, without NaN tests and without a branch per value: a
// NaN or an infinity shows in the sum of exponentials, or nothing is above -inf, and such a chunk is done
// again with a test per value; so is one of too few values for a threshold.  160 rows x 152064 float32 with the merge 33.7 -> 28.8 us (24 us = 4 TB/s in this pass), 16 rows 33 -> 13 us,
// one row 42 -> 11 us (those two mostly by larger chunks).
struct ChunkShared {
  unsigned long long red[kThreads / 64];
  float fred[kThreads / 64];
  unsigned long long win[kMaxTopK];
  unsigned long long list[kListCap];
  int list_n;
  float thr_w[kThreads / 64];
};

// Threshold T with at least k values >= T in the chunk: every wavefront takes the k-th largest
// of its 64 lane maxima (a lane counts the maxima strictly above its own, lane by lane through
// readlane; the smallest maximum with fewer than k above it is the k-th largest), which k of its
// own values reach; T is the largest of the wavefronts' thresholds.  A wavefront with fewer
// than k lanes holding values (`has`) sets no threshold; if none does, everything passes.
__device__ __forceinline__ float chunk_threshold(float mt, bool has, int k, float *thr_w) {
  int above = 0;
#pragma unroll
  for (int l = 0; l < 64; ++l) {
    const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mt), l));
    above += other > mt ? 1 : 0;
  }
  const int holders = __popcll(__ballot(has));
  float tw = (has && above < k) ? mt : __builtin_huge_valf();
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) tw = fminf(tw, __shfl_xor(tw, off, 64));
  if (holders < k) tw = -__builtin_huge_valf();
  if ((threadIdx.x & 63) == 0) thr_w[threadIdx.x >> 6] = tw;
  __syncthreads();
  return fmaxf(fmaxf(thr_w[0], thr_w[1]), fmaxf(thr_w[2], thr_w[3]));
}

// A chunk from registers.  False: not done (a NaN, an infinity, too many candidates); every thread of
// the workgroup returns the same.  The 16-byte pieces of memory are the unit: a piece's maximum is
// kept, and the few pieces that reach the threshold are read again.  The values before the first and
// behind the last whole piece go to one thread each.
template <typename T>
__device__ __forceinline__ bool fast_chunk(const T *row, int v0, int n, int k, ChunkShared &sh, float &mx, float &sum) {
  constexpr int PER = 16 / (int)sizeof(T), kPieces = kPerThread / PER;
  const int tid = threadIdx.x;
  const int head = min(n, (int)((0u - (uint32_t)(uintptr_t)row) & 15u) / (int)sizeof(T));
  const int n_full = (n - head) / PER, rest = n - n_full * PER;  // rest: head and tail together
  const u32x4 *src = (const u32x4 *)(row + head);
  const float ninf = -__builtin_huge_valf();
  const int single = tid < head ? tid : tid + n_full * PER;      // this thread's value outside the pieces
  const float tail = tid < rest ? load_f32<T>(row + single) : ninf;
  u32x4 w[kPieces];
  if (n_full > 0) {
#pragma unroll
    for (int q = 0; q < kPieces; ++q) w[q] = src[min(q * kThreads + tid, n_full - 1)];
  }
  if (tid == 0) sh.list_n = 0;
  auto value = [](const u32x4 &v, int e) {
    if (sizeof(T) == 4) return __uint_as_float(v[e]);
    return __uint_as_float((e & 1) ? (v[e >> 1] & 0xffff0000u) : (v[e >> 1] << 16));
  };
  auto max3 = [](float x, float y, float z) {  // fmaxf would quieten every operand first
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
  };
  float pm[kPieces], mt = tail;
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    pm[q] = ninf;
    if (q * kThreads < n_full) {
      float m = max3(value(w[q], 0), value(w[q], 1), value(w[q], 2));
      m = PER == 4 ? max3(m, m, value(w[q], 3)) : max3(m, value(w[q], 3), value(w[q], 4));
      if (PER == 8) m = max3(max3(m, value(w[q], 5 % PER), value(w[q], 6 % PER)), m, value(w[q], 7 % PER));
      pm[q] = q * kThreads + tid < n_full ? m : ninf;
      mt = max3(mt, mt, pm[q]);
    }
  }
  mx = wg_max_f(mt, sh.fred);
  // Nothing above -inf, or a signalling NaN: v_max3 makes it a quiet one, and the next maximum then
  // forgets the values beside it.
  if (!(mx > ninf)) return false;
  const float thr = chunk_threshold(mt, tid < n_full || tid < rest, k, sh.thr_w);
  const float c1 = 1.4426950408889634f, c0 = -mx * 1.4426950408889634f;
  float s = __builtin_amdgcn_exp2f(fmaf(tail, c1, c0));
  uint32_t reach = 0;  // pieces with a value that reaches the threshold
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    if (q * kThreads < n_full) {
      float p0 = 0.f, p1 = 0.f;
#pragma unroll
      for (int e = 0; e < PER; ++e) ((e & 1) ? p1 : p0) += __builtin_amdgcn_exp2f(fmaf(value(w[q], e), c1, c0));
      s += q * kThreads + tid < n_full ? p0 + p1 : 0.f;
      reach |= q * kThreads + tid < n_full && pm[q] >= thr ? 1u << q : 0u;
    }
  }
  auto offer = [&](float x, int pos) {
    if (x >= thr) {
      const int at = atomicAdd(&sh.list_n, 1);
      if (at < kListCap) sh.list[at] = sel_key(x, (uint32_t)(v0 + pos));
    }
  };
  if (tid < rest) offer(tail, single);
  while (reach) {
    const int at = __builtin_ctz(reach) * kThreads + tid;
    reach &= reach - 1;
    const u32x4 v = src[at];
#pragma unroll 1
    for (int e = 0; e < PER; ++e) {
      const uint32_t u = sizeof(T) == 4 ? (e < 2 ? (e ? v[1] : v[0]) : (e == 2 ? v[2] : v[3]))
                                        : ((e < 4 ? (e < 2 ? v[0] : v[1]) : (e < 6 ? v[2] : v[3])) << (e & 1 ? 0 : 16)) & 0xffff0000u;
      offer(__uint_as_float(u), head + at * PER + e);
    }
  }
  sum = wg_sum_f(s, sh.fred);  // its barriers also publish list and list_n
  const int cnt = sh.list_n;
  // The maximum's own exponential is 1.  A maximum near the type's limits (a mask of the lowest value)
  // leaves the range when scaled, in c0, and too few values for a threshold may share an offset that c0
  // rounds off: any_chunk takes the differences first.  Tested here, where registers are free again.
  if (!(sum >= 0.5f && sum < __builtin_huge_valf()) || cnt > kListCap || !(thr > ninf)) return false;
  rank_select(sh.list, cnt, k, sh.win);
  return true;
}

// The same for any values, read from memory in every pass; NaN counts as -inf.
template <typename T>
__device__ __forceinline__ void any_chunk(const T *row, int v0, int n, int k, ChunkShared &sh, float &mx, float &sum) {
  const int tid = threadIdx.x;
  const float ninf = -__builtin_huge_valf();
  auto value = [&](int i) {
    const float f = load_f32<T>(row + i);
    return f == f ? f : ninf;
  };
  if (tid == 0) sh.list_n = 0;
  float mt = ninf;
#pragma unroll 4
  for (int i = tid; i < n; i += kThreads) mt = fmaxf(mt, value(i));
  mx = wg_max_f(mt, sh.fred);
  if (!(mx > ninf)) {  // the lowest ids win
    if (tid < k) sh.win[tid] = tid < n ? sel_key(ninf, (uint32_t)(v0 + tid)) : 0ull;
    sum = 0.f;
    return;
  }
  const float thr = chunk_threshold(mt, tid < n, k, sh.thr_w);
  float s = 0.f;
#pragma unroll 4
  for (int i = tid; i < n; i += kThreads) {
    const float x = value(i);
    s += __expf(x - mx);
    if (x >= thr) {
      const int at = atomicAdd(&sh.list_n, 1);
      if (at < kListCap) sh.list[at] = sel_key(x, (uint32_t)(v0 + i));
    }
  }
  sum = wg_sum_f(s, sh.fred);  // its barriers also publish list and list_n
  const int cnt = sh.list_n;
  if (cnt <= kListCap) {
    rank_select(sh.list, cnt, k, sh.win);
    return;
  }
  unsigned long long last = ~0ull;
  for (int r = 0; r < k; ++r) {
    unsigned long long best = 0ull;
#pragma unroll 4
    for (int i = tid; i < n; i += kThreads) {
      const unsigned long long key = sel_key(value(i), (uint32_t)(v0 + i));
      best = (key < last && key > best) ? key : best;
    }
    best = wg_max_key(best, sh.red);
    if (tid == 0) sh.win[r] = best;
    last = best;
  }
}

template <typename T>
__global__ __launch_bounds__(kThreads, 4) void topk_chunk_kernel(int V, int k, int chunk, int n_chunks,
                                                                 const T *__restrict__ logits,
                                                                 unsigned char *__restrict__ work) {
  __shared__ ChunkShared sh;
  const int c = blockIdx.x, m = blockIdx.y;
  const int tid = threadIdx.x;
  const int v0 = c * chunk;
  const int n = min(chunk, V - v0);
  const T *row = logits + (size_t)m * V + v0;
  float mx, sum;
  if (!fast_chunk(row, v0, n, k, sh, mx, sum)) {
    __syncthreads();  // given up: its list is done with
    any_chunk(row, v0, n, k, sh, mx, sum);
  }
  __syncthreads();
  unsigned char *slot = work + ((size_t)m * n_chunks + c) * (sizeof(Partial) + (size_t)k * 8);
  if (tid == 0) {
    Partial p;
    p.max = mx;
    p.sum = sum;
    *(Partial *)slot = p;
  }
  if (tid < k) ((unsigned long long *)(slot + sizeof(Partial)))[tid] = sh.win[tid];
}

__global__ __launch_bounds__(kThreads) void topk_merge_kernel(int V, int k, int n_chunks,
                                                              const unsigned char *__restrict__ work,
                                                              int32_t *__restrict__ out_ids,
                                                              float *__restrict__ out_logp) {
  __shared__ unsigned long long red[kThreads / 64];
  __shared__ float fred[kThreads / 64];
  __shared__ unsigned long long win[kMaxTopK];
  __shared__ unsigned long long list[kListCap];
  const int m = blockIdx.x;
  const size_t stride = sizeof(Partial) + (size_t)k * 8;
  const unsigned char *base = work + (size_t)m * n_chunks * stride;
  float mx = -__builtin_huge_valf();
  for (int c = threadIdx.x; c < n_chunks; c += kThreads) mx = fmaxf(mx, ((const Partial *)(base + c * stride))->max);
  mx = wg_max_f(mx, fred);
  float sum = 0.f;
  for (int c = threadIdx.x; c < n_chunks; c += kThreads) {
    const Partial p = *(const Partial *)(base + c * stride);
    if (p.max > -__builtin_huge_valf()) sum += p.sum * __expf(p.max - mx);
  }
  sum = wg_sum_f(sum, fred);
  const float lse = mx + __logf(sum);
  // the chunks' winners are keys already
  const int n = n_chunks * k;
  if (n <= kListCap) {
    for (int i = threadIdx.x; i < n; i += kThreads)
      list[i] = ((const unsigned long long *)(base + (i / k) * stride + sizeof(Partial)))[i % k];
    __syncthreads();
    rank_select(list, n, k, win);
  } else {  // k rounds of the maximum below the last one
    unsigned long long last = ~0ull;
    for (int r = 0; r < k; ++r) {
      unsigned long long best = 0ull;
      for (int i = threadIdx.x; i < n; i += kThreads) {
        const unsigned long long key = ((const unsigned long long *)(base + (i / k) * stride + sizeof(Partial)))[i % k];
        best = (key < last && key > best) ? key : best;
      }
      best = wg_max_key(best, red);
      if (threadIdx.x == 0) win[r] = best;
      last = best;
    }
    __syncthreads();
  }
  if (threadIdx.x < k) {
    const unsigned long long key = win[threadIdx.x];
    const bool ok = key != 0ull;
    out_ids[(size_t)m * k + threadIdx.x] = ok ? (int32_t)argmax_key_index(key) : -1;
    out_logp[(size_t)m * k + threadIdx.x] = ok ? fminf(argmax_key_value(key) - lse, 0.f) : -__builtin_huge_valf();
  }
}

// score order: a beats b iff higher score, or equal score and lower index (no NaN in s[])
__device__ __forceinline__ bool beats(float sa, int a, float sb, int b) { return sa > sb || (sa == sb && a < b); }

__global__ __launch_bounds__(kThreads) void tree_grow_kernel(int K, int level, int C,
                                                             const int32_t *__restrict__ child_ids,
                                                             const float *__restrict__ child_logp,
                                                             float *__restrict__ cand_score,
                                                             int32_t *__restrict__ cand_token,
                                                             int32_t *__restrict__ cand_parent,
                                                             int32_t *__restrict__ frontier,
                                                             int32_t *__restrict__ frontier_slot) {
  __shared__ float s_new[kMaxTopK * kMaxTopK];
  const int b = blockIdx.x;
  const int F = level == 0 ? 1 : K;
  const int n_new = F * K;
  const int first = level == 0 ? 0 : K + (level - 1) * K * K;
  for (int t = threadIdx.x; t < n_new; t += kThreads) {
    const int f = t / K;
    int par = level == 0 ? -1 : frontier[(size_t)b * K + f];
    par = par < -1 ? -1 : (par >= first ? first - 1 : par);  // stay inside the pool whatever the caller left there
    const float base = par < 0 ? 0.f : cand_score[(size_t)b * C + par];
    float s = base + child_logp[((size_t)b * F) * K + t];
    if (!(s == s)) s = -__builtin_huge_valf();
    s_new[t] = s;
    cand_score[(size_t)b * C + first + t] = s;
    cand_token[(size_t)b * C + first + t] = child_ids[((size_t)b * F) * K + t];
    cand_parent[(size_t)b * C + first + t] = par;
  }
  __syncthreads();  // all reads of the old frontier are done
  for (int t = threadIdx.x; t < n_new; t += kThreads) {
    int rank = t;
    if (level > 0) {
      const float s = s_new[t];
      rank = 0;
#pragma unroll 8
      for (int u = 0; u < n_new; ++u) rank += beats(s_new[u], u, s, t) ? 1 : 0;
    }
    if (rank < K) {
      frontier[(size_t)b * K + rank] = first + t;
      frontier_slot[(size_t)b * K + rank] = t / K;
    }
  }
}

constexpr int kFinalThreads = 1024;  // one workgroup per sequence: sixteen wavefronts share the C^2 / 2 comparisons

__global__ __launch_bounds__(kFinalThreads) void tree_finalize_kernel(
    int B, int C, int n, const float *__restrict__ cand_score, const int32_t *__restrict__ cand_token,
    const int32_t *__restrict__ cand_parent, const int32_t *__restrict__ root_token, int32_t *__restrict__ node_offset,
    int32_t *__restrict__ parent, int32_t *__restrict__ draft_ids, int32_t *__restrict__ depth,
    unsigned long long *__restrict__ anc, int32_t *__restrict__ node_cand, float *__restrict__ node_score) {
  extern __shared__ unsigned char dyn[];
  float *s = (float *)dyn;                 // C scores
  int16_t *node_of = (int16_t *)(s + C);   // C: node index of a kept candidate, 0 otherwise
  unsigned char *kept = (unsigned char *)(node_of + C);  // C: the candidate is among the n - 1 best
  __shared__ int wave_kept[kFinalThreads / 64];
  __shared__ int spar[64];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int keep = n - 1;
  for (int c = tid; c < C; c += kFinalThreads) {
    float x = cand_score[(size_t)b * C + c];
    s[c] = (x == x) ? x : -__builtin_huge_valf();
  }
  __syncthreads();
  // ranks: four neighbouring lanes share a candidate, each counts a quarter of the others
  const int sub = tid & 3;
  constexpr int kPerPass = kFinalThreads / 4;
  const int c_end = (C + kPerPass - 1) / kPerPass * kPerPass;  // the same trip count for every lane
  for (int c = tid >> 2; c < c_end; c += kPerPass) {
    const bool live = c < C;
    const float sc = live ? s[c] : 0.f;
    int rank = 0;
    if (live) {
#pragma unroll 8
      for (int u = sub; u < C; u += 4) rank += beats(s[u], u, sc, c) ? 1 : 0;
    }
    rank += __shfl_xor(rank, 1, 64);
    rank += __shfl_xor(rank, 2, 64);
    if (live && sub == 0) kept[c] = rank < keep ? 1 : 0;
  }
  __syncthreads();
  // each thread owns a contiguous run of candidates, so that kept candidates are counted in order
  const int per = (C + kFinalThreads - 1) / kFinalThreads;
  const int c0 = min(C, tid * per), c1 = min(C, c0 + per);
  int cnt = 0;
  for (int c = c0; c < c1; ++c) cnt += kept[c];
  // exclusive prefix count over the threads: inside the wavefront by shifts, then the wavefronts before
  int incl = cnt;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(incl, off, 64);
    if ((tid & 63) >= off) incl += y;
  }
  if ((tid & 63) == 63) wave_kept[tid >> 6] = incl;
  __syncthreads();
  int before = incl - cnt;
  for (int w = 0; w < (tid >> 6); ++w) before += wave_kept[w];
  for (int c = c0; c < c1; ++c) {
    const bool k = kept[c] != 0;
    node_of[c] = k ? (int16_t)(1 + before) : (int16_t)0;
    before += k ? 1 : 0;
  }
  __syncthreads();
  const size_t o = (size_t)b * n;
  for (int c = c0; c < c1; ++c) {
    const int i = node_of[c];
    if (i == 0) continue;
    int pc = cand_parent[(size_t)b * C + c];
    pc = pc < 0 ? -1 : (pc >= c ? -1 : pc);  // a parent comes before its children, else: the root
    const int p = pc < 0 ? 0 : node_of[pc];  // a dropped parent (malformed scores) also maps to the root
    spar[i] = p;
    parent[o + i] = p;
    draft_ids[o + i] = cand_token[(size_t)b * C + c];
    node_cand[o + i] = c;
    node_score[o + i] = s[c];
  }
  if (tid == 0) {
    spar[0] = -1;
    parent[o] = -1;
    draft_ids[o] = root_token[b];
    node_cand[o] = -1;
    node_score[o] = 0.f;
    node_offset[b] = b * n;
    if (b == B - 1) node_offset[B] = B * n;
  }
  __syncthreads();
  if (tid < n) {
    unsigned long long a = 1ull << tid;
    int d = 0, x = tid;
    for (int guard = 0; guard < 64; ++guard) {
      const int p = spar[x];
      if (p < 0 || p >= x) break;
      a |= 1ull << p;
      ++d;
      x = p;
    }
    depth[o + tid] = d;
    anc[o + tid] = a;
  }
}

}  // namespace

size_t topk_workspace_bytes(int32_t M, int32_t V, int32_t k) {
  const int chunk = kChunk;
  const size_t n_chunks = ((size_t)V + chunk - 1) / chunk;
  return (size_t)M * n_chunks * (sizeof(Partial) + (size_t)k * 8);
}

hipError_t launch_topk_logprob(int32_t dtype, int32_t M, int32_t V, int32_t k, const void *logits, int32_t *out_ids,
                               float *out_logp, void *work, hipStream_t s) {
  const int chunk = kChunk;
  const int n_chunks = (V + chunk - 1) / chunk;
  dim3 grid((unsigned)n_chunks, (unsigned)M);
  if (dtype == HB_BF16)
    topk_chunk_kernel<bf16_t><<<grid, kThreads, 0, s>>>(V, k, chunk, n_chunks, (const bf16_t *)logits,
                                                        (unsigned char *)work);
  else
    topk_chunk_kernel<float><<<grid, kThreads, 0, s>>>(V, k, chunk, n_chunks, (const float *)logits,
                                                       (unsigned char *)work);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  topk_merge_kernel<<<M, kThreads, 0, s>>>(V, k, n_chunks, (const unsigned char *)work, out_ids, out_logp);
  return hipGetLastError();
}

hipError_t launch_tree_grow(int32_t B, int32_t K, int32_t level, int32_t C, const int32_t *child_ids,
                            const float *child_logp, float *cand_score, int32_t *cand_token, int32_t *cand_parent,
                            int32_t *frontier, int32_t *frontier_slot, hipStream_t s) {
  tree_grow_kernel<<<B, kThreads, 0, s>>>(K, level, C, child_ids, child_logp, cand_score, cand_token, cand_parent,
                                          frontier, frontier_slot);
  return hipGetLastError();
}

hipError_t launch_tree_finalize(int32_t B, int32_t C, int32_t n, const float *cand_score, const int32_t *cand_token,
                                const int32_t *cand_parent, const int32_t *root_token, int32_t *node_offset,
                                int32_t *parent, int32_t *draft_ids, int32_t *depth, unsigned long long *anc,
                                int32_t *node_cand, float *node_score, hipStream_t s) {
  const size_t lds = (size_t)C * (sizeof(float) + sizeof(int16_t) + 1) + 16;
  tree_finalize_kernel<<<B, kFinalThreads, lds, s>>>(B, C, n, cand_score, cand_token, cand_parent, root_token, node_offset,
                                                parent, draft_ids, depth, anc, node_cand, node_score);
  return hipGetLastError();
}

}  // namespace hb
