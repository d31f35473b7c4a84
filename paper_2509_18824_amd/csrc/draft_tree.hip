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
// Candidate a beats c iff its score is higher, or equal with a lower candidate index: a strict total
// order, held in one 64-bit key.  A level's ranking is by counting (the number of keys above), so the ranks
// are a permutation and every output slot is written exactly once; the re-ranking needs no order, only who
// is among the best.
#include "hb_internal.h"

#include <type_traits>

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

// Logits per chunk: 64 per thread.  Always the most a workgroup holds: it takes 5
// to 10 us whatever its chunk, and every chunk adds k winners to the merge, whose ranking is quadratic
// (16 rows x 152064 in chunks of 3072: 33 us, of 16384: 13 us).
constexpr int kChunk = 16384;
constexpr int kPerThread = kChunk / kThreads;
constexpr int kListCap = 2048;              // candidates that pass the threshold
constexpr int kThresholdSlack = 4;          // lanes of a wavefront that may pass beside the k it is made from

// Pass 1 of the top-k: one workgroup per (chunk, row).  A thread's 16-byte pieces stream through registers,
// eight in flight; each gives its maximum and its share of the sum of exponentials as it arrives, and only the
// maxima are kept, so that eight wavefronts fit a SIMD and every chunk of a level is resident at once.  The k
// best entries are found without sorting: a threshold T that at least k values of the chunk reach (from the
// per-thread maxima, see below) is a lower bound of the chunk's k-th largest value, so only values
// >= T can be among the k best; the few pieces that reach it are read again, those values collected in
// LDS (as order-preserving keys) and the k best picked there by counting ranks.
// Many values equal to the threshold can let more pass than the list holds; then k rounds of a workgroup-wide
// maximum run over the chunk instead (same result, slower).
//
// What bounds it: memory (from 1 to 160 rows 96 MB take 17 us more), and the chain behind the last load, with
// the merge's launch 10 us.  No NaN tests and no branch per value: a NaN or an infinity shows in the sum of
// exponentials, or nothing is above -inf, and such a chunk is done again with a test per value; so is one of
// too few values for a threshold.  With the merge, against whole chunks held in registers (five
// workgroups per CU, the exponentials behind a pass for the maximum): 160 rows x 152064 float32 28.7 -> 27.3 us,
// bfloat16 23.8 -> 21.8, 160 x 50257 16.8 -> 15.2, 16 x 152064 13.7 -> 12.1.
struct ChunkShared {
  unsigned long long red[kThreads / 64];
  float fred[kThreads / 64];
  unsigned long long win[kMaxTopK];
  unsigned long long list[kListCap];
  int list_n;
  float thr_w[kThreads / 64];
};

// Threshold T with at least k values >= T in the chunk: every wavefront takes the k-th largest
// of its 64 lane maxima (found bit by bit, a ballot each: a quarter of the vector instructions of
// counting every lane against every other), which k of its own values reach; T is the largest of
// the wavefronts' thresholds.  A wavefront with fewer than k lanes holding values (`has`) sets no
// threshold; if none does, everything passes.
// The upper 16 bits of the k-th maximum do as long as hardly more lanes reach them than k: for values whose
// spread is small against their size (a common offset) they would let everything pass, and the lower bits are
// found as well (160 rows x 152064 float32 less 10000: 202 us with the upper bits alone, 25.4 so, like without the
// offset; all 32 bits always cost 0.4 us of those 25 and of the 10.5 of one row).
__device__ __forceinline__ float chunk_threshold(float mt, bool has, int k, float *thr_w) {
  const uint32_t u = __float_as_uint(mt);
  const uint32_t key = has ? ((u & 0x80000000u) ? ~u : (u | 0x80000000u)) : 0u;
  uint32_t t = 0;
  auto next_bit = [&](int bit) {
    const uint32_t up = t | (1u << bit);
    t = __popcll(__ballot(key >= up)) >= k ? up : t;
  };
#pragma unroll
  for (int bit = 31; bit >= 16; --bit) next_bit(bit);
  if (__popcll(__ballot(key >= t)) > k + kThresholdSlack) {
#pragma unroll 1
    for (int bit = 15; bit >= 0; --bit) next_bit(bit);
  }
  float tw = __uint_as_float((t & 0x80000000u) ? (t & 0x7fffffffu) : ~t);
  if (t <= 0x007fffffu) tw = -__builtin_huge_valf();  // at or below the key of -inf, or too few lanes
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
  constexpr int kAhead = kPieces < 8 ? kPieces : 8;  // pieces in flight
  const int tid = threadIdx.x;
  const int head = min(n, (int)((0u - (uint32_t)(uintptr_t)row) & 15u) / (int)sizeof(T));
  const int n_full = (n - head) / PER, rest = n - n_full * PER;  // rest: head and tail together
  const u32x4 *src = (const u32x4 *)(row + head);
  const float ninf = -__builtin_huge_valf();
  const int single = tid < head ? tid : tid + n_full * PER;      // this thread's value outside the pieces
  const float tail = tid < rest ? load_f32<T>(row + single) : ninf;
  auto load = [&](int q) { return src[min(q * kThreads + tid, n_full - 1)]; };
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
  // s: this thread's sum of 2^(x log2 e - ref), with no pass for the maximum before it.  ref is the running
  // maximum as a whole number: a change of it scales s by a power of two, and what counts in the sum has a
  // small exponent that rounds once.  It never falls below kLeastRef: there x log2 e is off a whole number by
  // half of its last bit, and by 2^439 at a mask of -1e10 that stands in a thread's first piece, an infinity that
  // sent the chunk the slow way (160 rows x 152064 float32, nine tenths masked so: 58.9 us, 24.9 so).
  constexpr float kLeastRef = -0x1p30f;
  const float c1 = 1.4426950408889634f;
  float pm[kPieces], mt = ninf, s = 0.f, ref = kLeastRef;
  auto scaled = [](float x, float by) { return ldexpf(x, (int)__builtin_amdgcn_fmed3f(by, -400.f, 0.f)); };
  auto follow = [&](float m) {
    const float r = fmaxf(ref, rintf(m * c1));
    s = scaled(s, ref - r);
    ref = r;
  };
  // whole: every piece is there in part at least, and no branch stands between a load and the wait for it
  auto pass = [&](auto whole) {
    u32x4 w[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) w[q] = load(q);
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      pm[q] = ninf;
      if (whole || q * kThreads < n_full) {
        const u32x4 v = w[q % kAhead];
        const bool mine = (whole && q < kPieces - 1) || q * kThreads + tid < n_full;
        float m = max3(value(v, 0), value(v, 1), value(v, 2));
        m = PER == 4 ? max3(m, m, value(v, 3)) : max3(m, value(v, 3), value(v, 4));
        if (PER == 8) m = max3(max3(m, value(v, 5 % PER), value(v, 6 % PER)), m, value(v, 7 % PER));
        pm[q] = mine ? m : ninf;
        mt = max3(mt, mt, pm[q]);
        follow(pm[q]);
        float p0 = 0.f, p1 = 0.f;
#pragma unroll
        for (int e = 0; e < PER; ++e) ((e & 1) ? p1 : p0) += __builtin_amdgcn_exp2f(fmaf(value(v, e), c1, -ref));
        s += mine ? p0 + p1 : 0.f;
        if (q + kAhead < kPieces) w[q % kAhead] = load(q + kAhead);
      }
    }
  };
  if (n_full > (kPieces - 1) * kThreads) {
    pass(std::true_type{});
  } else if (n_full > 0) {
    pass(std::false_type{});
  } else {
#pragma unroll
    for (int q = 0; q < kPieces; ++q) pm[q] = ninf;
  }
  mt = max3(mt, mt, tail);
  follow(tail);
  s += __builtin_amdgcn_exp2f(fmaf(tail, c1, -ref));
  float mw = mt;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mw = fmaxf(mw, __shfl_xor(mw, off, 64));
  if ((tid & 63) == 0) sh.fred[tid >> 6] = mw;  // published by the threshold's barrier
  const float thr = chunk_threshold(mt, tid < n_full || tid < rest, k, sh.thr_w);
  mx = fmaxf(fmaxf(sh.fred[0], sh.fred[1]), fmaxf(sh.fred[2], sh.fred[3]));
  // Nothing above -inf, or a signalling NaN: v_max3 makes it a quiet one, and the next maximum then
  // forgets the values beside it.
  if (!(mx > ninf)) return false;
  const float top = fmaxf(kLeastRef, rintf(mx * c1));  // the largest ref
  s = scaled(s, ref - top);
  uint32_t reach = 0;  // pieces with a value that reaches the threshold
#pragma unroll
  for (int q = 0; q < kPieces; ++q) reach |= q * kThreads + tid < n_full && pm[q] >= thr ? 1u << q : 0u;
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
  sum = wg_sum_f(s, sh.fred) * __builtin_amdgcn_exp2f(-fmaf(mx, c1, -top));  // the barriers also publish list and list_n
  const int cnt = sh.list_n;
  // The maximum's own exponential is 1.  A maximum near the type's limits (a mask of the lowest value)
  // leaves the range when scaled: any_chunk takes the differences first.  Tested here, where registers are free again.
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
  const int n = n_chunks * k;
  // Up to 64 chunks and 256 winners: everything is requested at once, every wavefront sums the row up by itself, and a
  // winner writes itself out, so that one barrier is all (in a graph, 160 rows x 152064 27.6 -> 27.1 us for both passes, 16 rows 11.4 -> 10.8).
  if (n_chunks <= 64 && n <= kThreads) {
    const int i = threadIdx.x, lane = i & 63;
    const unsigned long long mine = i < n ? ((const unsigned long long *)(base + (i / k) * stride + sizeof(Partial)))[i % k] : 0ull;
    Partial p = {-__builtin_huge_valf(), 0.f};
    if (lane < n_chunks) p = *(const Partial *)(base + lane * stride);
    list[i] = mine;
    float mx = p.max;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float sum = p.max > -__builtin_huge_valf() ? p.sum * __expf(p.max - mx) : 0.f;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    const float lse = mx + __logf(sum);
    __syncthreads();
    int rank = 0, some = 0;
#pragma unroll 16
    for (int j = 0; j < n; ++j) {
      rank += list[j] > mine ? 1 : 0;
      some += list[j] ? 1 : 0;
    }
    if (mine && rank < k) {
      out_ids[(size_t)m * k + rank] = (int32_t)argmax_key_index(mine);
      out_logp[(size_t)m * k + rank] = fminf(argmax_key_value(mine) - lse, 0.f);
    }
    if (i >= some && i < k) {  // fewer winners than places
      out_ids[(size_t)m * k + i] = -1;
      out_logp[(size_t)m * k + i] = -__builtin_huge_valf();
    }
    return;
  }
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

__global__ __launch_bounds__(kThreads) void tree_grow_kernel(int K, int level, int C,
                                                             const int32_t *__restrict__ child_ids,
                                                             const float *__restrict__ child_logp,
                                                             float *__restrict__ cand_score,
                                                             int32_t *__restrict__ cand_token,
                                                             int32_t *__restrict__ cand_parent,
                                                             int32_t *__restrict__ frontier,
                                                             int32_t *__restrict__ frontier_slot) {
  __shared__ unsigned long long keys[kMaxTopK * kMaxTopK];
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
    keys[t] = sel_key(s, (uint32_t)t);
    cand_score[(size_t)b * C + first + t] = s;
    cand_token[(size_t)b * C + first + t] = child_ids[((size_t)b * F) * K + t];
    cand_parent[(size_t)b * C + first + t] = par;
  }
  __syncthreads();  // all reads of the old frontier are done
  for (int t = threadIdx.x; t < n_new; t += kThreads) {
    int rank = t;
    if (level > 0) {
      const unsigned long long mine = keys[t];
      rank = 0;
#pragma unroll 8
      for (int u = 0; u < n_new; ++u) rank += keys[u] > mine ? 1 : 0;
    }
    if (rank < K) {
      frontier[(size_t)b * K + rank] = first + t;
      frontier_slot[(size_t)b * K + rank] = t / K;
    }
  }
}

// One workgroup of NW wavefronts per sequence; a thread keeps a run of up to P candidates in registers, in
// order.  The keep best are those above the keep-th largest score, found bit by bit (a ballot per bit and
// register), and the first of those equal to it: C comparisons per bit instead of C^2 by counting.  One
// wavefront, and so no barrier, as long as the candidates fit it: what bounds it is the chain of 32 counts
// behind the loads, each of P ballots, so P is no larger than the candidates ask for.  In a graph, against ranks by
// counting: 6 candidates 3.7 -> 3.5 us (6.6 with P = 8), 55 4.2 -> 3.6 (6.7), 200 6.2 -> 5.0 (6.9), 410 12.2 -> 7.1,
// 784 32.6 -> 13.0, 3875 685 -> 17.1.
template <int NW, int P>
__global__ __launch_bounds__(64 * NW) void tree_finalize_kernel(
    int B, int C, int n, const float *__restrict__ cand_score, const int32_t *__restrict__ cand_token,
    const int32_t *__restrict__ cand_parent, const int32_t *__restrict__ root_token, int32_t *__restrict__ node_offset,
    int32_t *__restrict__ parent, int32_t *__restrict__ draft_ids, int32_t *__restrict__ depth,
    unsigned long long *__restrict__ anc, int32_t *__restrict__ node_cand, float *__restrict__ node_score) {
  __shared__ int16_t node_of[64 * NW * P];  // node index of a kept candidate, 0 otherwise
  __shared__ int counts[2][NW];
  __shared__ int spar[64];
  const int b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6;
  const int keep = n - 1;
  const int per = (C + 64 * NW - 1) / (64 * NW), c0 = tid * per;
  float score[P];
  int32_t tok[P], par[P];
  uint32_t key[P];  // ordered like the scores, -0 as +0, NaN as -inf; 0: none
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int c = min(c0 + i, C - 1);
    score[i] = cand_score[(size_t)b * C + c];
    tok[i] = cand_token[(size_t)b * C + c];
    par[i] = cand_parent[(size_t)b * C + c];
  }
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if (!(score[i] == score[i])) score[i] = -__builtin_huge_valf();
    key[i] = i < per && c0 + i < C ? (uint32_t)(sel_key(score[i], 0u) >> 32) : 0u;
  }
  // the sum over the workgroup of a wavefront's count; slots alternate, so one barrier each is enough
  auto total = [&](int mine, int slot) {
    if (NW == 1) return mine;
    if ((tid & 63) == 0) counts[slot][wave] = mine;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += counts[slot][w];
    return sum;
  };
  auto at_least = [&](uint32_t t) {
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) cnt += __popcll(__ballot(key[i] >= t));
    return cnt;
  };
  uint32_t last = 0;  // the keep-th largest key
#pragma unroll 1
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t up = last | (1u << bit);
    if (total(at_least(up), bit & 1) >= keep) last = up;
  }
  // before this thread, candidates above the last one kept and (upper half) equal to it: C <= 4096
  int mine = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) mine += (key[i] > last ? 1 : 0) + (key[i] == last ? 1 << 16 : 0);
  int before = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(before, off, 64);
    if ((tid & 63) >= off) before += y;
  }
  int all = __shfl(before, 63, 64);
  before -= mine;
  if (NW > 1) {
    __syncthreads();
    if ((tid & 63) == 0) counts[0][wave] = all;
    __syncthreads();
    all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) before += counts[0][w];
      all += counts[0][w];
    }
  }
  const int ties = keep - (all & 0xffff);
  int node[P];
  int above = before & 0xffff, equal = before >> 16;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const bool gt = key[i] > last, eq = key[i] == last;
    node[i] = gt || (eq && equal < ties) ? 1 + above + min(equal, ties) : 0;
    above += gt ? 1 : 0;
    equal += eq ? 1 : 0;
    if (i < per && c0 + i < C) node_of[c0 + i] = (int16_t)node[i];
  }
  __syncthreads();
  const size_t o = (size_t)b * n;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int c = c0 + i, at = node[i];
    if (at == 0) continue;
    const int pc = par[i] < 0 || par[i] >= c ? -1 : par[i];  // a parent comes before its children, else: the root
    const int p = pc < 0 ? 0 : node_of[pc];  // a dropped parent (malformed scores) also maps to the root
    spar[at] = p;
    parent[o + at] = p;
    draft_ids[o + at] = tok[i];
    node_cand[o + at] = c;
    node_score[o + at] = score[i];
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
  auto kern = C <= 64    ? tree_finalize_kernel<1, 1>
              : C <= 128 ? tree_finalize_kernel<1, 2>
              : C <= 256 ? tree_finalize_kernel<1, 4>
              : C <= 512 ? tree_finalize_kernel<1, 8>
                         : tree_finalize_kernel<4, 16>;
  kern<<<B, C <= 512 ? 64 : 256, 0, s>>>(B, C, n, cand_score, cand_token, cand_parent, root_token, node_offset, parent, draft_ids,
                                         depth, anc, node_cand, node_score);
  return hipGetLastError();
}

}  // namespace hb
