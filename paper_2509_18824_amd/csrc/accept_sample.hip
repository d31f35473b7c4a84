// Sampling acceptance of a verified draft tree (speculative sampling with several candidates
// per position), in exact fixed-point integers so that every decision is reproducible.
//
// The tree is walked from the root.  At a node, the children are tried in
// index order: child with token x is accepted iff  u * q_x * S(p) < 2^32 * p_x * S(q)  (p, q:
// fix(.) = floor(. * 2^30) of the target's / the draft's distribution after the node, S = sum);
// a rejection replaces p by the residual  r_v = max(p_v S(q) - q_v S(p), 0)  rescaled to 2^30
// (r_v / max(S(r) >> 30, 1)) and removes x from q.  When no child
// is accepted the step's last token is the smallest v with p_0 + .. + p_v > (u_bonus S(p)) >> 32.
// Sums are integer sums, so they do not depend on the order in which the lanes add them up.
//
// Rejected tokens need no mask over q in the vocabulary passes: after its rejection round a token
// has p_x = 0 (rejection means q_x S(p) > p_x S(q)), so its residual is 0 whatever q_x is; only
// S(q) and the single look-ups of q_x honour the removals.
//
// Decomposition.  A node needs one pass over its two rows and every rejection two more (the
// residual's sum, then the rescaled residual and its sum), each depending on the sums of the one
// before.  One workgroup per sequence would read 1.2 MB per pass through one CU's memory path on 16
// of 256 CUs (5.3 ms for 16 sequences of 60 nodes over 152064 tokens, measured in that form).  Here
// the vocabulary of a sequence is dealt to wavefronts, 2560 consecutive tokens each, which read their
// range of a node's rows once and keep it in registers (40 values of p and of q per lane), so that a
// rejection touches no vocabulary in memory; what crosses wavefronts are the sums.  Every wavefront
// keeps p_x and q_x of the node's children in its lanes, updates them like any other value, and takes
// every decision itself: no barrier on the way.  16 sequences of 60 nodes over 152064 tokens: 80 us, the
// kernel that clears the slots included.  Vocabularies of up to 5120 tokens are one workgroup's per sequence (kAlone).
// What bounds it is the chain of the sequence with the most rejections (ten at the root: 73 us): per
// rejection two exchanges of 2 us each and 2.5 us of 64-bit integer work, per node visited 5 us for its
// rows.  Measured against 81 us in a form whose workgroups took their places by index: 20 values per lane
// (twice the wavefronts, twice the partners per exchange) 107 us; recomputing the residual for the division
// instead of keeping its 80 registers 88 us; sums by LDS permutes and workgroup barriers 95 us.
//
// Exchange: slot (k, w) holds wavefront w's partial sum of exchange k, bit 63 set; a slot is written
// once per launch (they are cleared by a kernel before it) and polled by the sequence's other
// wavefronts, the data being its own flag.
//
// The waits have to end whatever else runs on the chip, which holds one of these workgroups per CU.  A
// workgroup draws its place (sequence, share) from a counter when it starts, so the places held are
// always the lowest and of a launch that has begun only the last sequence can be waiting for workgroups
// that have not, at most 31 CUs of 256.  (By the workgroup's index two launches could each fill one XCD
// and wait there for the other's.)  Where even those few find no CU, under a CU mask or beside many such
// launches, a wavefront gives up after so many looks and says so in the sequence's leave word, which the
// others look at while they wait; every workgroup counts itself out there, and the last one, which has no
// partner left, does the whole sequence by itself (accept_alone).  The same way go sequences whose rows sum
// to 2 or more, which 32 bits do not hold.  Drawing cost that form 6 to
// 14 us for 240 workgroups, nothing measurable for 60; four counters instead of one the same, the
// workgroups of a sequence on one XCD 18 us: it is where a sequence's workgroups sit, not the counter.
#include "hb_internal.h"

namespace hb {

namespace {

constexpr int kThreads = 256;
constexpr int kFixBits = 30;

__device__ __forceinline__ uint32_t fix_prob(float p) {
  if (!(p > 0.f)) return 0u;            // negative, zero, NaN
  if (p >= 2.f) return 0x7fffffffu;     // clamp (also +inf)
  return (uint32_t)(p * 1073741824.f);  // exact scaling by 2^30, truncation
}

// a * b < c * d in 128 bits (all operands < 2^64)
__device__ __forceinline__ bool mul_less(unsigned long long a, unsigned long long b, unsigned long long c,
                                         unsigned long long d) {
  const unsigned long long lh = __umul64hi(a, b), ll = a * b;
  const unsigned long long rh = __umul64hi(c, d), rl = c * d;
  return lh < rh || (lh == rh && ll < rl);
}

typedef unsigned long long u64;

constexpr int kPer = 40;                       // vocabulary entries a lane keeps in registers
constexpr int kRange = kPer * 64;              // ... a wavefront (2560)
constexpr int kMaxWorkers = 127;               // wavefronts per sequence; beyond 325120 tokens the rest stays in memory
constexpr int kExchanges = 192;                // at most 64 nodes visited and two exchanges for each of 63 children
// Vocabularies up to here: one workgroup per sequence, alone, p and q of a node in LDS.  Dealt to wavefronts
// they pay 7 us a node for exchanges and registers that hardly hold anything (16 chains of 8 nodes, V = 100: 56 us
// dealt, 16 alone, 1000: 58 and 23, 3000: 66 and 40, 5000: 67 and 59; trees of 60 nodes 5000: 59 and 73, 7000: 66 and
// 103; one workgroup that read its rows from memory in every pass: 19, 29, 53, 72; 194, 271).
constexpr int kAlone = 2 * kRange;
constexpr u64 kPosted = 1ull << 63;
constexpr uint32_t kMost = 0x7fffffff;          // sums of rows and residuals stay below: nearly 2 in fixed point
constexpr uint32_t kGaveUp = 1u << 16;         // in a sequence's leave word: one for every wavefront that gave up ...
constexpr uint32_t kLeft = kGaveUp - 1;        // ... above the count of its workgroups that have left
constexpr int kBufferFlags = 0x00027000;       // untyped 32-bit elements

template <int CTRL>
__device__ __forceinline__ u64 dpp_add(u64 x) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
  return x + (((u64)hi << 32) | lo);
}
// sum over the wavefront, in every lane: inside a row of 16 lanes by data-parallel moves, across
// rows by the lane swaps (an LDS permute per step costs a memory round trip each)
__device__ __forceinline__ u64 wave_sum(u64 x) {
  x = dpp_add<0xB1>(x);   // lanes ^ 1
  x = dpp_add<0x4E>(x);   // lanes ^ 2
  x = dpp_add<0x141>(x);  // the other quad of eight
  x = dpp_add<0x140>(x);  // the other eight of sixteen
  typedef unsigned int swap2 __attribute__((ext_vector_type(2)));
  swap2 lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
  swap2 hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
  x = (((u64)hi[0] << 32) | lo[0]) + (((u64)hi[1] << 32) | lo[1]);
  lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
  return (((u64)hi[0] << 32) | lo[0]) + (((u64)hi[1] << 32) | lo[1]);
}

// the same of 32-bit values, 0xffffffff where it does not fit
__device__ __forceinline__ uint32_t add_sat(uint32_t x, uint32_t y) { return __builtin_elementwise_add_sat(x, y); }
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_add_sat(uint32_t x) {
  return add_sat(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t wave_sum_sat(uint32_t x) {
  x = dpp_add_sat<0xB1>(x);
  x = dpp_add_sat<0x4E>(x);
  x = dpp_add_sat<0x141>(x);
  x = dpp_add_sat<0x140>(x);
  typedef unsigned int swap2 __attribute__((ext_vector_type(2)));
  swap2 y = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = add_sat(y[0], y[1]);
  y = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return add_sat(y[0], y[1]);
}

// max(p S(q) - q S(p), 0); the sums of rows and of residuals are below 2^31
__device__ __forceinline__ u64 residual(uint32_t p, uint32_t q, uint32_t sp, uint32_t sq) {
  const u64 a = (u64)p * sq, b = (u64)q * sp;
  return a > b ? a - b : 0ull;
}

// r / max(S(r) >> 30, 1) by a 32-bit reciprocal: with 2^k <= div < 2^(k+1) the estimate
// ((r >> k) * floor(2^(32+k) / div)) >> 32 is at most two below the quotient (each factor loses less
// than one unit), and the remainder says by how much.  r <= S(r) keeps r >> k below 2^32.
struct Divisor {
  uint32_t div, recip;
  int k;
};
__device__ __forceinline__ Divisor make_divisor(u64 sr) {
  Divisor d;
  const u64 div = sr >> kFixBits;
  d.div = div ? (uint32_t)div : 1u;
  d.k = 31 - __builtin_clz(d.div);
  const u64 r = (1ull << (32 + d.k)) / d.div;
  d.recip = r > 0xffffffffull ? 0xffffffffu : (uint32_t)r;
  return d;
}
__device__ __forceinline__ uint32_t divide(u64 r, const Divisor &d) {
  uint32_t q = __umulhi((uint32_t)(r >> d.k), d.recip);
  const u64 rem = r - (u64)q * d.div;
  q += rem >= d.div ? 1u : 0u;
  q += rem >= 2ull * d.div ? 1u : 0u;
  return q;
}

__device__ __forceinline__ u64 *slots_of(uint32_t *work) { return (u64 *)(((uintptr_t)work + 7) & ~(uintptr_t)7); }

// A sequence's workspace: a word of control (low half: in the first sequence's the counter that places are
// drawn from; high half: the leave word), the slots of its exchanges, and what lies beyond the registers.
__global__ __launch_bounds__(256) void accept_sample_clear_kernel(int V, int workers, uint32_t *__restrict__ work_all) {
  u64 *control = slots_of(work_all + (size_t)blockIdx.x * V);
  for (int i = threadIdx.x; i < 1 + kExchanges * workers; i += 256) control[i] = 0ull;
}

struct Sequence {
  int n0, n;  // its nodes
  const int32_t *parent, *draft_ids;
  const float *p_target, *q_draft;
  const uint32_t *u_accept;
  uint32_t u_bonus;
  int V, max_path;
  int32_t *accept_len, *accept_path, *out_tokens, *bonus_id;
};

// One sequence by one workgroup, alone and waiting for nobody: every pass over the vocabulary reads the
// rows from memory, and a value's residual is worked out again from the node's rejections before it (their
// sums stay in LDS; the workspace still belongs to the launch).  Small vocabularies (KEEP) stay in LDS: p (the
// node's, or the residual) and q of a node in p_row and q_row.  Sums and products have 64 bits.
struct Rejection {
  u64 sp, sq, div;  // p <- max(p S(q) - q S(p), 0) / div
  Divisor d;        // where the sums fit it
  bool fits;
};
struct AloneShared {
  int32_t par[64], did[64], path[64], removed[64];
  Rejection rejections[64];
  u64 red[kThreads / 64], share[kThreads], q_token;
  int decision;
};

__device__ __forceinline__ u64 wide_residual(uint32_t p, uint32_t q, u64 sp, u64 sq) {
  const u64 a = p * sq, b = q * sp;
  return a > b ? a - b : 0ull;
}

template <bool KEEP>
__device__ __forceinline__ void accept_alone(const Sequence &s, AloneShared &sh, uint32_t *p_row, uint32_t *q_row) {
  const int tid = threadIdx.x;
  auto sum = [&](u64 x) {
    x = wave_sum(x);
    __syncthreads();  // red may still be read from the previous sum
    if ((tid & 63) == 0) sh.red[tid >> 6] = x;
    __syncthreads();
    return sh.red[0] + sh.red[1] + sh.red[2] + sh.red[3];
  };
  if (tid < 64) {
    int par = -1, did = 0;
    if (tid < s.n) {
      par = s.parent[s.n0 + tid];
      if (par >= tid || par < -1 || tid == 0) par = -1;  // malformed: never anybody's child
      did = s.draft_ids[s.n0 + tid];
    }
    sh.par[tid] = par;
    sh.did[tid] = did;
  }
  if (tid == 0) sh.path[0] = 0;
  __syncthreads();
  int cur = 0, len = 1, bonus = -1;
#pragma unroll 1
  for (;;) {
    const float *prow = s.p_target + (size_t)(s.n0 + cur) * s.V;
    const float *qrow = s.q_draft + (size_t)(s.n0 + cur) * s.V;
    int n_rejections = 0, n_removed = 0;
    auto q_at = [&](int v) { return KEEP ? q_row[v] : fix_prob(qrow[v]); };
    auto p_at = [&](int v) {
      if (KEEP) return p_row[v];
      uint32_t p = fix_prob(prow[v]);
      const uint32_t q = n_rejections ? fix_prob(qrow[v]) : 0u;
#pragma unroll 1
      for (int i = 0; i < n_rejections; ++i)
        p = sh.rejections[i].fits ? divide(residual(p, q, (uint32_t)sh.rejections[i].sp, (uint32_t)sh.rejections[i].sq), sh.rejections[i].d)
                                  : (uint32_t)(wide_residual(p, q, sh.rejections[i].sp, sh.rejections[i].sq) / sh.rejections[i].div);
      return p;
    };
    u64 sp = 0, sq = 0;
    for (int v = tid; v < s.V; v += kThreads) {
      const uint32_t p = fix_prob(prow[v]), q = fix_prob(qrow[v]);
      if (KEEP) {
        p_row[v] = p;
        q_row[v] = q;
      }
      sp += p;
      sq += q;
    }
    sp = sum(sp);
    sq = sum(sq);
    int taken = -1;
#pragma unroll 1
    for (int c = cur + 1; c < s.n && len < s.max_path; ++c) {
      if (sh.par[c] != cur) continue;  // uniform
      const int x = sh.did[c];
      const bool x_ok = x >= 0 && x < s.V;
      if (tid == 0) {
        const u64 px = x_ok ? p_at(x) : 0u;
        u64 qx = x_ok ? q_at(x) : 0u;
        for (int i = 0; i < n_removed; ++i) qx = sh.removed[i] == x ? 0ull : qx;
        const u64 u = s.u_accept[s.n0 + c];
        sh.decision = mul_less(u * qx, sp, px * sq, 1ull << 32) ? 1 : 0;
        sh.q_token = qx;
      }
      __syncthreads();
      const bool accept = sh.decision != 0;
      const u64 qx = sh.q_token;
      __syncthreads();
      if (accept) {
        taken = c;
        break;
      }
      u64 sr = 0;
      for (int v = tid; v < s.V; v += kThreads) sr += wide_residual(p_at(v), q_at(v), sp, sq);
      sr = sum(sr);
      if (sr != 0) {
        const u64 div = sr >> kFixBits;
        const bool fits = sp <= kMost && sq <= kMost;
        const Rejection r = {sp, sq, div ? div : 1ull, fits ? make_divisor(sr) : Divisor{}, fits};
        u64 snew = 0;
        if (KEEP) {
          for (int v = tid; v < s.V; v += kThreads) {
            const uint32_t p = p_row[v], q = q_row[v];
            const uint32_t x = fits ? divide(residual(p, q, (uint32_t)sp, (uint32_t)sq), r.d) : (uint32_t)(wide_residual(p, q, sp, sq) / r.div);
            p_row[v] = x;
            snew += x;
          }
        } else {
          if (tid == 0) sh.rejections[n_rejections] = r;
          __syncthreads();
          ++n_rejections;
          for (int v = tid; v < s.V; v += kThreads) snew += p_at(v);
        }
        sp = sum(snew);
      }
      if (tid == 0 && x_ok) sh.removed[n_removed] = x;
      n_removed += x_ok ? 1 : 0;
      sq -= qx;
      __syncthreads();
    }
    if (taken < 0) {
      // the last token: inverse CDF of the current p over consecutive shares of the vocabulary
      if (sp != 0) {
        const u64 t = (s.u_bonus * sp) >> 32;
        const int per = (s.V + kThreads - 1) / kThreads;
        const int v0 = min(s.V, tid * per), v1 = min(s.V, v0 + per);
        u64 mine = 0;
        for (int v = v0; v < v1; ++v) mine += p_at(v);
        __syncthreads();
        sh.share[tid] = mine;
        if (tid == 0) sh.decision = -1;  // sums that overflow 64 bits: nobody's share
        __syncthreads();
        u64 before = 0;
        for (int i = 0; i < tid; ++i) before += sh.share[i];
        if (before <= t && t < before + mine) {
          u64 upto = before;
          for (int v = v0; v < v1; ++v) {
            upto += p_at(v);
            if (upto > t) {
              sh.decision = v;
              break;
            }
          }
        }
        __syncthreads();
        bonus = sh.decision;
      }
      break;
    }
    if (tid == 0) sh.path[len] = taken;
    ++len;
    cur = taken;
    __syncthreads();
  }
  __syncthreads();
  for (int j = tid; j < s.max_path; j += kThreads) {
    s.accept_path[j] = j < len ? sh.path[j] : -1;
    s.out_tokens[j] = j + 1 < len ? sh.did[sh.path[j + 1]] : (j + 1 == len ? bonus : -1);
  }
  if (tid == 0) {
    *s.accept_len = len;
    *s.bonus_id = bonus;
  }
}

__global__ __launch_bounds__(kThreads) void tree_accept_sample_alone_kernel(
    int max_nodes, int V, const int32_t *__restrict__ node_offset, const int32_t *__restrict__ parent,
    const int32_t *__restrict__ draft_ids, const float *__restrict__ p_target, const float *__restrict__ q_draft,
    const uint32_t *__restrict__ u_accept, const uint32_t *__restrict__ u_bonus, int max_path,
    int32_t *__restrict__ accept_len, int32_t *__restrict__ accept_path, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ bonus_id) {
  __shared__ AloneShared sh;
  __shared__ uint32_t p_row[kAlone], q_row[kAlone];
  const int b = blockIdx.x;
  const int n0 = node_offset[b];
  int n = node_offset[b + 1] - n0;
  n = n < 0 ? 0 : (n > max_nodes ? max_nodes : n);
  int32_t *path_out = accept_path + (size_t)b * max_path, *tok_out = out_tokens + (size_t)b * max_path;
  if (n == 0) {  // nothing to verify: nothing is emitted
    for (int j = threadIdx.x; j < max_path; j += kThreads) { path_out[j] = -1; tok_out[j] = -1; }
    if (threadIdx.x == 0) { accept_len[b] = 0; bonus_id[b] = -1; }
    return;
  }
  accept_alone<true>({n0, n, parent, draft_ids, p_target, q_draft, u_accept, u_bonus[b], V, max_path, accept_len + b, path_out,
                      tok_out, bonus_id + b}, sh, p_row, q_row);
}

__global__ __launch_bounds__(kThreads) void tree_accept_sample_kernel(
    int polls, int max_nodes, int V, int workers, int groups, int chunk, const int32_t *__restrict__ node_offset, const int32_t *__restrict__ parent,
    const int32_t *__restrict__ draft_ids, const float *__restrict__ p_target, const float *__restrict__ q_draft,
    const uint32_t *__restrict__ u_accept, const uint32_t *__restrict__ u_bonus, int max_path,
    int32_t *__restrict__ accept_len, int32_t *__restrict__ accept_path, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ bonus_id, uint32_t *__restrict__ work_all) {
  __shared__ unsigned drawn;
  __shared__ uint32_t leave_mark;  // what this workgroup adds to the leave word
  __shared__ bool alone;
  __shared__ AloneShared alone_shared;
  if (threadIdx.x == 0) {
    drawn = groups > 1 ? atomicAdd((unsigned *)slots_of(work_all), 1u) : blockIdx.x;
    leave_mark = 1;
  }
  __syncthreads();
  const unsigned place = drawn;
  if (place >= gridDim.x) return;  // somebody else draws from this workspace: wrong, but inside the tensors
  const int b = __builtin_amdgcn_readfirstlane((int)(place / (unsigned)groups));
  const int w = __builtin_amdgcn_readfirstlane((int)(place % (unsigned)groups) * (kThreads / 64) + (int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int n0 = node_offset[b];
  int n = node_offset[b + 1] - n0;
  n = n < 0 ? 0 : (n > max_nodes ? max_nodes : n);
  int32_t *path_out = accept_path + (size_t)b * max_path;
  int32_t *tok_out = out_tokens + (size_t)b * max_path;
  if (n == 0) {  // nothing to verify: nothing is emitted
    if (w != 0) return;
    for (int j = lane; j < max_path; j += 64) { path_out[j] = -1; tok_out[j] = -1; }
    if (lane == 0) { accept_len[b] = 0; bonus_id[b] = -1; }
    return;
  }
  // the tree, one node per lane
  int par = -1, did = 0;
  uint32_t u_mine = 0;
  if (lane < n) {
    par = parent[n0 + lane];
    if (par >= lane || par < -1 || lane == 0) par = -1;  // malformed: never anybody's child
    did = draft_ids[n0 + lane];
    u_mine = u_accept[n0 + lane];
  }
  u64 *control = slots_of(work_all + (size_t)b * V), *slots = control + 1;
  uint32_t *leave = (uint32_t *)control + 1;
  const int v_begin = w * chunk, v_end = min(V, v_begin + chunk);  // this wavefront's range
  const int r_end = min(v_end, v_begin + kRange);                  // the part in registers
  // what lies beyond the registers keeps its residual behind the slots
  uint32_t *work = (uint32_t *)(slots + kExchanges * kMaxWorkers) + (long long)w * (chunk - kRange) - v_begin - kRange;
  int k = 0;

  // x of every wavefront of the sequence: lane i gets the shares of wavefronts i and i + 64.  Not ok:
  // a share did not come in time, or somebody has given up (lane 63, which has no share to look for,
  // looks at the leave word instead).  Few wavefronts have a loop of their own, and there is one way out:
  // with one loop for both the kernel spills 24 registers (16 trees of 60 nodes over 152064 tokens: 90 us),
  // with a return at each exit they take 85 us, this way 80.
  const bool wide = workers > 63;
  struct Shares {
    u64 s0, s1;
    bool ok;
  };
  auto exchange = [&](u64 x) -> Shares {
    u64 *slot = slots + k * workers;
    ++k;
    if (lane == 0) __hip_atomic_store(slot + w, x | kPosted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    u64 y0 = 0, y1 = 0;
    bool ok = false;
    if (!wide) {
      const u64 *at = lane == 63 ? control : slot + min(lane, workers - 1);
#pragma unroll 1
      for (int i = 0; i < polls; ++i) {
        y0 = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = __all(lane == 63 || (y0 & kPosted) != 0);
        if (ok || __any(lane == 63 && (uint32_t)(y0 >> 32) >= kGaveUp)) break;
      }
      y0 = lane < workers ? y0 & ~kPosted : 0ull;
    } else {
      const u64 *at0 = slot + lane, *at1 = lane == 63 ? control : slot + min(lane + 64, workers - 1);
#pragma unroll 1
      for (int i = 0; i < polls; ++i) {
        y0 = __hip_atomic_load(at0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        y1 = __hip_atomic_load(at1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = __all((y0 & kPosted) != 0 && (lane == 63 || (y1 & kPosted) != 0));
        if (ok || __any(lane == 63 && (uint32_t)(y1 >> 32) >= kGaveUp)) break;
      }
      y0 &= ~kPosted;
      y1 = lane + 64 < workers ? y1 & ~kPosted : 0ull;
    }
    return {y0, y1, ok};
  };

  auto walk = [&]() -> bool {
    int cur = 0, len = 1;
    int path = 0;  // lane i: node i of the path
    uint32_t sp = 0;
    uint32_t sp0 = 0, sp1 = 0;  // shares of S(p)
    uint32_t p[kPer], q[kPer];
    const float *prow, *qrow;
    bool in_work = false;  // beyond the registers: p is the target's row (false) or the residual in the workspace
#pragma unroll 1
    for (;;) {
      prow = p_target + (size_t)(n0 + cur) * V;
      qrow = q_draft + (size_t)(n0 + cur) * V;
      in_work = false;
      // lanes that hold a child of the node: p and q of its token
      const bool child = par == cur && len < max_path;
      const int tok = child && did >= 0 && did < V ? did : -1;
      float pf = 0.f, qf = 0.f;
      if (tok >= 0) {
        pf = prow[tok];
        qf = qrow[tok];
      }
      // The range's loads are all in flight before the first is used; buffer loads return zero beyond
      // the range and cost one address register for all of them.
      uint32_t a = 0, c = 0;  // this wavefront's shares of S(p) and S(q)
      {
        const int bytes = (r_end > v_begin ? r_end - v_begin : 0) * 4;
        const auto pr = __builtin_amdgcn_make_buffer_rsrc((void *)(prow + v_begin), 0, bytes, kBufferFlags);
        const auto qr = __builtin_amdgcn_make_buffer_rsrc((void *)(qrow + v_begin), 0, bytes, kBufferFlags);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          p[j] = __builtin_amdgcn_raw_buffer_load_b32(pr, lane * 4, j * 256, 0);
          q[j] = __builtin_amdgcn_raw_buffer_load_b32(qr, lane * 4, j * 256, 0);
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          p[j] = fix_prob(__uint_as_float(p[j]));
          q[j] = fix_prob(__uint_as_float(q[j]));
          a = add_sat(a, p[j]);
          c = add_sat(c, q[j]);
        }
        for (int v = v_begin + kRange + lane; v < v_end; v += 64) { a = add_sat(a, fix_prob(prow[v])); c = add_sat(c, fix_prob(qrow[v])); }
      }
      uint32_t px = fix_prob(pf), qx = fix_prob(qf), q_left = qx;  // q_left: 0 once the token has been removed from q
      // both in one exchange; a share that does not fit shows as kMost, and so the sum does not either
      a = wave_sum_sat(a);
      c = wave_sum_sat(c);
      const Shares both = exchange(((u64)min(a, kMost) << 32) | min(c, kMost));
      if (!both.ok) return false;
      sp0 = (uint32_t)(both.s0 >> 32);
      sp1 = (uint32_t)(both.s1 >> 32);
      sp = wave_sum_sat(sp0 + sp1);
      uint32_t sq = wave_sum_sat((uint32_t)both.s0 + (uint32_t)both.s1);
      if (sp >= kMost || sq >= kMost) return false;
      int taken = -1;
      u64 left = __ballot(child);
#pragma unroll 1
      while (left) {
        const int c = __builtin_amdgcn_readfirstlane(__builtin_ctzll(left));
        left &= left - 1;
        const uint32_t cp = __builtin_amdgcn_readlane(px, c), cq = __builtin_amdgcn_readlane(q_left, c);
        const uint32_t u = __builtin_amdgcn_readlane(u_mine, c);
        // u q_x S(p) < 2^32 p_x S(q)
        if (mul_less((u64)u * cq, sp, (u64)cp * sq, 1ull << 32)) { taken = c; break; }
        // the residual's sum, then the rescaled residual and its sum
        u64 sr = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          sr += residual(p[j], q[j], sp, sq);
        }
        for (int v = v_begin + kRange + lane; v < v_end; v += 64)
          sr += residual(in_work ? work[v] : fix_prob(prow[v]), fix_prob(qrow[v]), sp, sq);
        const Shares rs = exchange(wave_sum(sr));
        if (!rs.ok) return false;
        sr = wave_sum(rs.s0 + rs.s1);
        if (sr != 0) {
          const Divisor d = make_divisor(sr);
          u64 snew = 0;
#pragma unroll
          for (int j = 0; j < kPer; ++j) {
            p[j] = divide(residual(p[j], q[j], sp, sq), d);
            snew += p[j];
          }
          for (int v = v_begin + kRange + lane; v < v_end; v += 64) {
            const uint32_t x = divide(residual(in_work ? work[v] : fix_prob(prow[v]), fix_prob(qrow[v]), sp, sq), d);
            work[v] = x;
            snew += x;
          }
          px = divide(residual(px, qx, sp, sq), d);
          in_work = true;
          const Shares ps = exchange(wave_sum(snew));
          if (!ps.ok) return false;
          sp0 = (uint32_t)ps.s0;
          sp1 = (uint32_t)ps.s1;
          sp = wave_sum_sat(sp0 + sp1);
        }
        sq -= cq;
        const int cx = __builtin_amdgcn_readlane(tok, c);
        if (tok == cx) q_left = 0;
      }
      if (taken < 0) break;
      if (lane == len) path = taken;
      ++len;
      cur = taken;
    }

    // Last token: the wavefront whose share of p holds the bonus uniform's place finds it, and writes
    // the step's results; wavefront 0 does when p is all zero.
    int bonus = -1;
    if (sp == 0) {
      if (w != 0) return true;
    } else {
      u64 t = ((u64)u_bonus[b] * sp) >> 32;
      const u64 before = wave_sum((lane < w ? (u64)sp0 : 0ull) + (lane + 64 < w ? (u64)sp1 : 0ull));
      const u64 mine = wave_sum((lane == w ? (u64)sp0 : 0ull) + (lane + 64 == w ? (u64)sp1 : 0ull));
      if (t < before || t - before >= mine) return true;
      t -= before;
      // the row of 64 consecutive tokens that holds the place, then the token
      u64 acc = 0;
      auto look = [&](uint32_t x, int v) {
        const u64 row = wave_sum(x);
        if (bonus < 0 && t < acc + row) {
          u64 upto = x;  // inclusive prefix over the lanes
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const u64 y = __shfl_up(upto, off, 64);
            if (lane >= off) upto += y;
          }
          bonus = v + __builtin_ctzll(__ballot(acc + upto > t));
        }
        acc += row;
      };
#pragma unroll
      for (int j = 0; j < kPer; ++j) look(p[j], v_begin + j * 64);
      for (int v = v_begin + kRange; v < v_end; v += 64) {
        const int at = v + lane;
        look(at < v_end ? (in_work ? work[at] : fix_prob(prow[at])) : 0u, v);
      }
    }
    for (int j0 = 0; j0 < max_path; j0 += 64) {
      const int j = j0 + lane;
      const int node = j < len ? path : -1;
      const int next = j0 == 0 ? __shfl(path, lane < 63 ? lane + 1 : lane, 64) : 0;
      const int next_tok = __shfl(did, next, 64);
      if (j < max_path) {
        path_out[j] = j0 == 0 ? node : -1;
        tok_out[j] = j0 == 0 && j + 1 < len ? next_tok : (j + 1 == len ? bonus : -1);
      }
    }
    if (lane == 0) { accept_len[b] = len; bonus_id[b] = bonus; }
    return true;
  };

  if (w < workers && !walk() && lane == 0) {
    atomicAdd(leave, kGaveUp);  // partners need not wait any longer
    leave_mark = 1 + kGaveUp;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t word = leave_mark;
    if (groups > 1) word += atomicAdd(leave, leave_mark);
    alone = word >= kGaveUp && (word & kLeft) == (uint32_t)groups;  // the last of the sequence, and somebody gave up
  }
  __syncthreads();
  if (alone)
    accept_alone<false>({n0, n, parent, draft_ids, p_target, q_draft, u_accept, u_bonus[b], V, max_path, accept_len + b, path_out,
                         tok_out, bonus_id + b}, alone_shared, nullptr, nullptr);
}

}  // namespace

hipError_t launch_tree_accept_sample(int32_t B, int32_t max_nodes, int32_t V, const int32_t *node_offset,
                                     const int32_t *parent, const int32_t *draft_ids, const float *p_target,
                                     const float *q_draft, const uint32_t *u_accept, const uint32_t *u_bonus,
                                     int32_t max_path, int32_t *accept_len, int32_t *accept_path,
                                     int32_t *out_tokens, int32_t *bonus_id, uint32_t *work, int32_t polls, hipStream_t s) {
  if (V <= kAlone) {
    tree_accept_sample_alone_kernel<<<(unsigned)B, kThreads, 0, s>>>(max_nodes, V, node_offset, parent, draft_ids, p_target, q_draft,
                                                                    u_accept, u_bonus, max_path, accept_len, accept_path,
                                                                    out_tokens, bonus_id);
    return hipGetLastError();
  }
  // as few wavefronts as hold the vocabulary in registers: fewer partners per exchange
  int workers = (int)(((int64_t)V + kRange - 1) / kRange);
  if (workers > kMaxWorkers) workers = kMaxWorkers;
  const int chunk = workers < kMaxWorkers ? kRange : (int)(((int64_t)V + workers - 1) / workers);
  const int groups = (workers + kThreads / 64 - 1) / (kThreads / 64);
  accept_sample_clear_kernel<<<(unsigned)B, 256, 0, s>>>(V, workers, work);
  const int64_t grid = (int64_t)B * groups;
  tree_accept_sample_kernel<<<(unsigned)grid, kThreads, 0, s>>>(
      polls, max_nodes, V, workers, groups, chunk, node_offset, parent, draft_ids, p_target, q_draft, u_accept, u_bonus, max_path,
      accept_len, accept_path, out_tokens, bonus_id, work);
  return hipGetLastError();
}

}  // namespace hb
