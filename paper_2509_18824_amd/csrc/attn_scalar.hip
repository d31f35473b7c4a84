// Scalar tree-verify attention: one workgroup per (node, query head, KV chunk), fp32 arithmetic
// whatever the storage type.  It is the kernel for fp32 inputs and for shapes the MFMA kernel does
// not take, and it defines the semantics the fast kernel must match: keys are the prefix positions
// of the chunk, plus (chunk 0 only) the tree nodes on the node's own root path.  Also holds the
// split-K merge kernel.
//
// What bounds it at the sizes it is used for is latency: memory round trips in a row and chains of
// dependent instructions, not bytes.  The four wavefronts of a workgroup deal out blocks of 64 keys;
// a block is a handful of round trips (page ids, K, the V rows 16 at a time) and one softmax update
// whatever the number of keys in it.  4 nodes x 4 heads of 64 over 256 float32 positions: 12 us (7.7 by the kernel of few
// workgroups below);
// one wavefront that took the keys one by one, each with a sum across lanes and two exponentials,
// 138 us.
#include "hb_internal.h"

#include <algorithm>

namespace hb {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kRowsInFlight = 16;  // V rows requested before the first is used

__device__ inline float wave_max(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
  return x;
}
__device__ inline float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// eight consecutive elements, 16-byte aligned (head_dim % 8 == 0, tensors 16-byte aligned)
__device__ inline void load8(const float *p, float (&x)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[e] = a[e];
    x[4 + e] = b[e];
  }
}
__device__ inline void load8(const bf16_t *p, float (&x)[8]) {
  const u32x4 a = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[2 * e] = __uint_as_float(a[e] << 16);
    x[2 * e + 1] = __uint_as_float(a[e] & 0xffff0000u);
  }
}

// A lane's E elements of a row of V.  float32: every 64th, a load of 256 bytes each (two or four neighbours
// in one load: 28/4 heads of 128, 60-node trees over 4 x 500 positions 261 -> 300 us).  bf16: E neighbours in one
// load (every 64th, 128 bytes each: 8/8 heads of 256, 16 x 200 positions 461 us, in one load 212).
template <typename T, int E>
__device__ inline int dim_of(int lane, int e) { return sizeof(T) == 2 ? E * lane + e : lane + 64 * e; }
template <int E>
__device__ inline void load_row(const bf16_t *row, int lane, int D, float (&x)[E]) {
  if (E * lane >= D) return;  // head_dim % 8 == 0: all of them or none
  uint32_t a[E / 2];
  __builtin_memcpy(a, __builtin_assume_aligned(row + E * lane, 2 * E), 2 * E);
#pragma unroll
  for (int e = 0; e < E / 2; ++e) {
    x[2 * e] = __uint_as_float(a[e] << 16);
    x[2 * e + 1] = __uint_as_float(a[e] & 0xffff0000u);
  }
}

template <int E>
struct OnlineSoftmax {
  float m, l;     // reference exponent; this lane's share of the sum
  float acc[E];   // head dimensions dim_of(lane, 0), ...
};

// Up to 64 keys, one per lane: `live` marks the lanes that hold one, `off` is the key's offset in
// k and v.  A lane takes the whole dot product of its key, so the block needs one maximum and no
// sum across lanes; then the lanes spread over the head dimension and the V rows of the live keys
// are added up, kRowsInFlight of them requested at a time.
template <typename T, int E>
__device__ inline void absorb_keys(OnlineSoftmax<E> &st, const float *q_lds, const T *k, const T *v, size_t off,
                                   unsigned long long live, int D, int lane, float scale) {
  if (live == 0) return;
  const bool mine = (live >> lane) & 1;
  float s = -__builtin_huge_valf();
  if (mine) {
    float part[4] = {0.f, 0.f, 0.f, 0.f};
    const T *row = k + off;
#pragma unroll 8
    for (int d = 0; d < D; d += 8) {
      float x[8];
      load8(row + d, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) part[e & 3] = fmaf(q_lds[d + e], x[e], part[e & 3]);
    }
    s = ((part[0] + part[1]) + (part[2] + part[3])) * scale;
  }
  const float m_new = fmaxf(st.m, wave_max(s));
  // scores of -inf weigh nothing, also where there is nothing else yet to weigh them against
  const float m_ref = fmaxf(m_new, -__FLT_MAX__);
  const float corr = expf(st.m - m_ref);  // exp(-inf) = 0 on the first keys
  const float p = mine ? expf(s - m_ref) : 0.f;
  st.l = st.l * corr + p;
  st.m = m_new;
#pragma unroll
  for (int e = 0; e < E; ++e) st.acc[e] *= corr;
  const uint32_t off_lo = (uint32_t)off, off_hi = (uint32_t)(off >> 32);
  while (live) {
    float w[kRowsInFlight], x[kRowsInFlight][E];
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u) {
      w[u] = 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e) x[u][e] = 0.f;
      if (live) {  // uniform
        const int j = __builtin_amdgcn_readfirstlane(__builtin_ctzll(live));
        live &= live - 1;
        w[u] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p), j));
        const size_t o = (size_t)(uint32_t)__builtin_amdgcn_readlane(off_lo, j) |
                         ((size_t)(uint32_t)__builtin_amdgcn_readlane(off_hi, j) << 32);
        if constexpr (sizeof(T) == 2 && E > 1) {
          load_row<E>(v + o, lane, D, x[u]);
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e)
            if (lane + 64 * e < D) x[u][e] = load_f32(v + o + lane + 64 * e);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u)
#pragma unroll
      for (int e = 0; e < E; ++e) st.acc[e] = fmaf(w[u], x[u][e], st.acc[e]);
  }
}

// E: head dimensions per lane (D <= 64 E).  Eight wavefronts per SIMD where the compiler would use a few scalar
// registers too many for them (float32, 28/4 heads of 128, one 60-node tree over 64 positions 24.5 -> 19.4 us).
template <typename T, int E>
__global__ __launch_bounds__(kThreads, E == 4 || (E == 1 && sizeof(T) == 2) ? 4 : 8) void attn_scalar_kernel(
    hb_attn_desc d, int splits, int chunk_tokens, const T *__restrict__ q, const T *__restrict__ k_tree,
    const T *__restrict__ v_tree, const T *__restrict__ k_pool, const T *__restrict__ v_pool,
    const int32_t *__restrict__ block_table, const int32_t *__restrict__ prefix_len,
    const int32_t *__restrict__ node_offset, const int32_t *__restrict__ parent, T *__restrict__ out,
    float *__restrict__ lse, float *__restrict__ part_o, float *__restrict__ part_ml, ClearArgs clear) {
  if (blockIdx.y == 0) clear_words(clear, blockIdx.x, gridDim.x, threadIdx.x, kThreads);
  __shared__ float q_lds[64 * E];
  __shared__ float acc_lds[kWaves][64 * E];
  __shared__ float ml_lds[kWaves][2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row = blockIdx.x;  // node * Hq + head
  const int c = blockIdx.y;
  const int node = row / d.num_q_heads;
  const int h = row - node * d.num_q_heads;
  const int g = h / (d.num_q_heads / d.num_kv_heads);
  const int D = d.head_dim;

  for (int i = threadIdx.x; i < D; i += kThreads) q_lds[i] = load_f32(q + (size_t)row * D + i);
  // sequence of this node: largest b with node_offset[b] <= node
  int lo = 0, hi = d.batch;  // invariant: node_offset[lo] <= node < node_offset[hi] (if well formed)
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (node_offset[mid] <= node) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int n0 = node_offset[b];
  int n_nodes = node_offset[b + 1] - n0;
  if (n_nodes > d.max_nodes_per_tree) n_nodes = d.max_nodes_per_tree;
  int L = prefix_len[b];
  const int cap = d.max_blocks_per_seq * d.page_size;
  L = L < 0 ? 0 : (L > cap ? cap : L);
  __syncthreads();

  OnlineSoftmax<E> st;
  st.m = -__builtin_huge_valf();
  st.l = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) st.acc[e] = 0.f;

  const int begin = c * chunk_tokens;
  const int end = (c == splits - 1) ? L : min(L, begin + chunk_tokens);
  const size_t page_stride = (size_t)d.num_kv_heads * d.page_size * D;
  for (int p0 = begin + 64 * wave; p0 < end; p0 += 64 * kWaves) {
    const int n = min(64, end - p0);
    const int p = p0 + min(lane, n - 1);
    int blk = block_table[(size_t)b * d.max_blocks_per_seq + p / d.page_size];
    blk = blk < 0 ? 0 : (blk >= d.num_blocks ? d.num_blocks - 1 : blk);
    const size_t off = (size_t)blk * page_stride + ((size_t)g * d.page_size + p % d.page_size) * D;
    absorb_keys<T, E>(st, q_lds, k_pool, v_pool, off, n < 64 ? (1ull << n) - 1 : ~0ull, D, lane, d.softmax_scale);
  }
  if (c == 0 && wave == kWaves - 1) {  // the wavefront that has the least prefix when it is short
    // walk up from the node to the root through the parents held by the lanes; every visited node
    // is on the node's own path
    const int last = d.total_nodes - 1;
    const int at = max(0, min(n0 + lane, last));
    const int par = parent[at];
    unsigned long long live = 0;
    int x = __builtin_amdgcn_readfirstlane(node - n0);
    if (x >= n_nodes) x = -1;
    for (int guard = 0; x >= 0 && guard < 64; ++guard) {
      live |= 1ull << x;
      const int px = __builtin_amdgcn_readlane(par, x);
      x = (px < x) ? px : -1;  // a malformed parent ends the walk
    }
    const size_t off = ((size_t)at * d.num_kv_heads + g) * D;
    absorb_keys<T, E>(st, q_lds, k_tree, v_tree, off, live, D, lane, d.softmax_scale);
  }

  // the wavefronts' results are combined through LDS; one without keys has l = 0 and no weight
  const float l_wave = wave_sum(st.l);
#pragma unroll
  for (int e = 0; e < E; ++e) acc_lds[wave][dim_of<T, E>(lane, e)] = st.acc[e];
  if (lane == 0) {
    ml_lds[wave][0] = st.m;
    ml_lds[wave][1] = l_wave;
  }
  __syncthreads();
  float m = ml_lds[0][0], l = 0.f, w[kWaves];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) m = fmaxf(m, ml_lds[i][0]);
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const float li = ml_lds[i][1];
    w[i] = li == 0.f ? 0.f : expf(ml_lds[i][0] - m);
    l += w[i] * li;
  }
  // keys, but every score is -inf: NaN, or a chunk that is there and has no weight beside others
  if (l == 0.f && (end > begin || (c == 0 && node - n0 < n_nodes))) l = splits == 1 ? __builtin_nanf("") : 1.f;
  const float inv = l == 0.f ? 0.f : 1.f / l;
  const size_t slot = (size_t)row * splits + c;
  for (int i = threadIdx.x; i < D; i += kThreads) {
    float o = 0.f;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) o += w[u] * acc_lds[u][i];
    if (splits == 1)
      store_f32(out + (size_t)row * D + i, o * inv);
    else
      part_o[slot * D + i] = o;
  }
  if (threadIdx.x == 0) {
    if (splits == 1) {
      if (lse) lse[row] = m + logf(l);
    } else {
      part_ml[slot * 2 + 0] = m;
      part_ml[slot * 2 + 1] = l;
    }
  }
}

// ---- float32 rows of up to 64 values, few workgroups: as few memory round trips in a row as there can be -------------
// Four nodes or forty leave most of the chip idle, and what a workgroup does is wait: for the sequence's bounds, the page
// ids, K, four times for 16 rows of V, and in its last wavefront for the parents and the tree's keys after all that.  Here
// the bounds of all sequences come in one load, K and V of a block of 64 keys are in flight together (a load of V is four
// rows, four values a lane), the prefix has seven wavefronts and the tree one of its own.  That takes 200 registers a lane
// and a CU per workgroup: 4 nodes x 4 heads of 64 over 256 positions 12.0 -> 7.7 us, 8 nodes over 1024 15.5 -> 11.0.
constexpr int kEagerWaves = 7, kEagerThreads = 64 * (kEagerWaves + 1);
// What it takes: one round of the 256 CUs, and a little more where rows are cut into chunks (us, general and this: 160 rows in
// two chunks 256 positions 14.3 and 12.0, 400 18.9 and 13.5).  Whole rows on more than that are short, and a second round costs
// more than it saves (272 rows, 31 positions 9.1 and 11.0, 192 11.7 and 11.9).  Nor does it pay for hardly any keys (16 rows, 16
// positions 5.5 and 5.8, 31 6.5 and 5.9, 64 8.8 and 5.8).
constexpr int kEagerOnce = 256, kEagerMost = 320;  // workgroups
constexpr int kEagerLeast = 16;                    // positions that the prefixes may exceed
bool eager_takes(const hb_attn_desc &d, int64_t workgroups, int splits) {
  int64_t span = (int64_t)d.page_size * d.max_blocks_per_seq;
  if (d.max_prefix_len_hint > 0) span = std::min(span, (int64_t)d.max_prefix_len_hint);
  return d.dtype == HB_F32 && d.head_dim <= 64 && d.batch < 64 && span > kEagerLeast && workgroups <= (splits > 1 ? kEagerMost : kEagerOnce);
}

struct EagerSoftmax {
  float m, l;  // reference exponent; this lane's share of the sum
  f32x4 acc;   // of values 4 (lane % 16) ..., over the keys whose place in their block is lane / 16 more than a multiple of 4
};

// Up to 64 keys, one per lane, as absorb_keys takes them.
__device__ __forceinline__ void absorb_eagerly(EagerSoftmax &st, const float *q_lds, const float *k, const float *v, size_t off,
                                               unsigned long long live, int D, int lane, float scale) {
  if (live == 0) return;
  const bool mine = (live >> lane) & 1;
  const int d4 = min(4 * (lane & 15), D - 4), g = lane >> 4;
  const unsigned long long live_g = live >> g;
  f32x4 kx[16], vx[16];
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (4 * i < D) kx[i] = *reinterpret_cast<const f32x4 *>(k + off + 4 * i);
  const uint32_t off_lo = (uint32_t)off, off_hi = (uint32_t)(off >> 32);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    // a lane without a key has the address of one, and what it loads is not used
    const size_t o = (size_t)(uint32_t)__shfl((int)off_lo, 4 * i + g, 64) | ((size_t)(uint32_t)__shfl((int)off_hi, 4 * i + g, 64) << 32);
    vx[i] = *reinterpret_cast<const f32x4 *>(v + o + d4);
  }
  f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (4 * i < D) {
      const f32x4 qv = *reinterpret_cast<const f32x4 *>(q_lds + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) part[e] = fmaf(qv[e], kx[i][e], part[e]);
    }
  const float s = mine ? ((part[0] + part[1]) + (part[2] + part[3])) * scale : -__builtin_huge_valf();
  const float m_new = fmaxf(st.m, wave_max(s));
  // scores of -inf weigh nothing, also where there is nothing else yet to weigh them against
  const float m_ref = fmaxf(m_new, -__FLT_MAX__);
  const float corr = expf(st.m - m_ref);  // exp(-inf) = 0 on the first keys
  const float p = mine ? expf(s - m_ref) : 0.f;
  st.l = st.l * corr + p;
  st.m = m_new;
#pragma unroll
  for (int e = 0; e < 4; ++e) st.acc[e] *= corr;
#pragma unroll
  for (int i = 0; i < 16; ++i)
  {
    const float w = __shfl(p, 4 * i + g, 64);
    const bool has = (live_g >> (4 * i)) & 1;
#pragma unroll
    for (int e = 0; e < 4; ++e) st.acc[e] = fmaf(w, has ? vx[i][e] : 0.f, st.acc[e]);
  }
}

__global__ __launch_bounds__(kEagerThreads) void attn_scalar_eager_kernel(
    hb_attn_desc d, int splits, int chunk_tokens, const float *__restrict__ q, const float *__restrict__ k_tree,
    const float *__restrict__ v_tree, const float *__restrict__ k_pool, const float *__restrict__ v_pool,
    const int32_t *__restrict__ block_table, const int32_t *__restrict__ prefix_len,
    const int32_t *__restrict__ node_offset, const int32_t *__restrict__ parent, float *__restrict__ out,
    float *__restrict__ lse, float *__restrict__ part_o, float *__restrict__ part_ml, ClearArgs clear) {
  if (blockIdx.y == 0) clear_words(clear, blockIdx.x, gridDim.x, threadIdx.x, kEagerThreads);
  __shared__ __align__(16) float q_lds[64];
  __shared__ __align__(16) float acc_lds[kEagerWaves + 1][64];
  __shared__ float ml_lds[kEagerWaves + 1][2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row = blockIdx.x;  // node * Hq + head
  const int c = blockIdx.y;
  const int node = row / d.num_q_heads;
  const int h = row - node * d.num_q_heads;
  const int g = h / (d.num_q_heads / d.num_kv_heads);
  const int D = d.head_dim;

  // the sequence of this node: the largest b with node_offset[b] <= node; at most 63 of them, one per lane
  const int offset_mine = node_offset[min(lane, d.batch)], len_mine = prefix_len[min(lane, max(d.batch - 1, 0))];
  if (threadIdx.x < D) q_lds[threadIdx.x] = q[(size_t)row * D + threadIdx.x];
  const unsigned long long begun = __ballot(lane < d.batch && offset_mine <= node);
  const int b = begun ? 63 - __builtin_clzll(begun) : 0;
  const int n0 = __builtin_amdgcn_readlane(offset_mine, b);
  int n_nodes = __builtin_amdgcn_readlane(offset_mine, b + 1) - n0;
  if (n_nodes > d.max_nodes_per_tree) n_nodes = d.max_nodes_per_tree;
  int L = __builtin_amdgcn_readlane(len_mine, b);
  const int cap = d.max_blocks_per_seq * d.page_size;
  L = L < 0 ? 0 : (L > cap ? cap : L);

  EagerSoftmax st = {-__builtin_huge_valf(), 0.f, {0.f, 0.f, 0.f, 0.f}};
  const int begin = c * chunk_tokens;
  const int end = (c == splits - 1) ? L : min(L, begin + chunk_tokens);
  const size_t page_stride = (size_t)d.num_kv_heads * d.page_size * D;
  const int32_t *pages = block_table + (size_t)b * d.max_blocks_per_seq;
  const int at = max(0, min(n0 + lane, d.total_nodes - 1));
  const bool tree = wave == kEagerWaves;
  int p0 = begin + 64 * wave, blk = 0;
  auto place = [&] { return p0 + min(lane, end - p0 - 1); };
  if (!tree && p0 < end) blk = pages[place() / d.page_size];
  const int par = tree && c == 0 ? parent[at] : -1;
  __syncthreads();
  if (!tree) {
    for (; p0 < end; p0 += 64 * kEagerWaves) {
      const int n = min(64, end - p0), p = place();
      const int page = blk < 0 ? 0 : (blk >= d.num_blocks ? d.num_blocks - 1 : blk);
      const size_t off = (size_t)page * page_stride + ((size_t)g * d.page_size + p % d.page_size) * D;
      const int next = p0 + 64 * kEagerWaves;
      if (next < end) blk = pages[(next + min(lane, end - next - 1)) / d.page_size];
      absorb_eagerly(st, q_lds, k_pool, v_pool, off, n < 64 ? (1ull << n) - 1 : ~0ull, D, lane, d.softmax_scale);
    }
  } else if (c == 0) {
    // as above: up from the node to the root through the parents held by the lanes
    unsigned long long live = 0;
    int x = __builtin_amdgcn_readfirstlane(node - n0);
    if (x >= n_nodes) x = -1;
    for (int guard = 0; x >= 0 && guard < 64; ++guard) {
      live |= 1ull << x;
      const int px = __builtin_amdgcn_readlane(par, x);
      x = (px < x) ? px : -1;  // a malformed parent ends the walk
    }
    absorb_eagerly(st, q_lds, k_tree, v_tree, ((size_t)at * d.num_kv_heads + g) * D, live, D, lane, d.softmax_scale);
  }

  // the wavefronts' results are combined through LDS; one without keys has l = 0 and no weight
  const float l_wave = wave_sum(st.l);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    st.acc[e] += __shfl_xor(st.acc[e], 16, 64);
    st.acc[e] += __shfl_xor(st.acc[e], 32, 64);
  }
  if (lane < 16) *reinterpret_cast<f32x4 *>(&acc_lds[wave][4 * lane]) = st.acc;
  if (lane == 0) {
    ml_lds[wave][0] = st.m;
    ml_lds[wave][1] = l_wave;
  }
  __syncthreads();
  if (wave) return;
  float m = ml_lds[0][0], l = 0.f, o = 0.f;
#pragma unroll
  for (int i = 1; i <= kEagerWaves; ++i) m = fmaxf(m, ml_lds[i][0]);
#pragma unroll
  for (int i = 0; i <= kEagerWaves; ++i) {
    const float li = ml_lds[i][1];
    const float w = li == 0.f ? 0.f : expf(ml_lds[i][0] - m);
    l += w * li;
    o += w * acc_lds[i][lane];
  }
  // keys, but every score is -inf: NaN, or a chunk that is there and has no weight beside others
  if (l == 0.f && (end > begin || (c == 0 && node - n0 < n_nodes))) l = splits == 1 ? __builtin_nanf("") : 1.f;
  const float inv = l == 0.f ? 0.f : 1.f / l;
  const size_t slot = (size_t)row * splits + c;
  if (lane < D) {
    if (splits == 1)
      out[(size_t)row * D + lane] = o * inv;
    else
      part_o[slot * D + lane] = o;
  }
  if (lane == 0) {
    if (splits == 1) {
      if (lse) lse[row] = m + logf(l);
    } else {
      part_ml[slot * 2 + 0] = m;
      part_ml[slot * 2 + 1] = l;
    }
  }
}

// out[row] = sum_c O_c e^{m_c - m} / sum_c l_c e^{m_c - m}; chunks with l_c == 0 are empty and
// their O_c was never written.  One thread per four consecutive d of a row (D / 4 threads per
// row, 16-byte loads and stores); every thread reads its row's (m_c, l_c) pairs itself (they are
// a few cached bytes), and the loads of up to kMergeBatch chunks are issued together before any
// arithmetic, so the kernel runs at memory rate instead of one chunk latency at a time.
constexpr int kMergeBatch = 8;
typedef float merge_f32x4 __attribute__((ext_vector_type(4)));
typedef float merge_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t merge_u32x2 __attribute__((ext_vector_type(2)));

__device__ inline void store_row4(float *p, merge_f32x4 v) { *reinterpret_cast<merge_f32x4 *>(p) = v; }
__device__ inline void store_row4(bf16_t *p, merge_f32x4 v) {
  merge_u32x2 w;
  w.x = (uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16);
  w.y = (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16);
  *reinterpret_cast<merge_u32x2 *>(p) = w;
}

// l plus chunk c's sum of weights, rounded the same in both kernels below whatever the compiler makes of the code around it:
// a row is the same bits whichever of them has it.  The first of a batch is fused, as is every product with the values.
__device__ inline float add_weights(float l, float sum, float w, int c) {
#pragma clang fp contract(off)
  return c % kMergeBatch == 0 ? __builtin_fmaf(sum, w, l) : l + sum * w;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_merge_kernel(int rows, int D, int splits,
                                                         const float *__restrict__ part_o,
                                                         const float *__restrict__ part_ml,
                                                         T *__restrict__ out, float *__restrict__ lse) {
  const int tpr = D >> 2;  // threads per row (D % 4 == 0)
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const int row = (int)(gid / tpr);
  const int piece = (int)(gid - (long)row * tpr);
  if (row >= rows) return;
  const merge_f32x2 *ml = reinterpret_cast<const merge_f32x2 *>(part_ml) + (size_t)row * splits;
  // Chunks are filled from slot 0 on and empty ones only follow non-empty ones (a chunk that
  // holds any key has l > 0), so the first empty slot ends the list; producers need to mark
  // only that one.
  // Slots are read kMergeBatch at a time (independent loads: one round trip per batch instead
  // of one per slot).
  float m = -__builtin_huge_valf();
  int live = 0;
  bool open = true;
  for (int c0 = 0; c0 < splits && open; c0 += kMergeBatch) {
    merge_f32x2 x[kMergeBatch];
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      x[i] = (merge_f32x2){0.f, 0.f};
      if (c0 + i < splits) x[i] = ml[c0 + i];
    }
    if (c0 == 0 && x[0].y < 0.f) return;  // the attention kernel wrote this row out itself (row sums are never negative)
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      open = open && x[i].y > 0.f;
      m = open ? fmaxf(m, x[i].x) : m;
      live += open ? 1 : 0;
    }
  }
  const merge_f32x4 *po = reinterpret_cast<const merge_f32x4 *>(part_o) + (size_t)row * splits * tpr + piece;
  float l = 0.f;
  merge_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < live; c0 += kMergeBatch) {
    float w[kMergeBatch];
    merge_f32x4 o[kMergeBatch];
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const int c = c0 + i;
      merge_f32x2 x = {0.f, 0.f};
      if (c < live) x = ml[c];
      const bool ok = c < live;
      w[i] = ok ? expf(x.x - m) : 0.f;
      l = ok ? add_weights(l, x.y, w[i], i) : l;
      merge_f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (ok) v = po[(size_t)c * tpr];  // an empty chunk's slot is never read
      o[i] = v;
    }
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(o[i][e], w[i], acc[e]);
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
  store_row4(out + (size_t)row * D + piece * 4, acc * inv);
  if (lse && piece == 0) lse[row] = m + logf(l);
}

// The same for few partial results: those of all slots are requested with the (m, l) pairs, whether there is a chunk in
// them or not (what a slot without one holds is not used), so that a row takes one round trip instead of two.
// Up to 16 slots and 8 MB: the attention call for one 8-node chain over 2048 positions 16.5 -> 15.9 us, one 60-node tree 26.7
// -> 26.1; more bytes lose by the empty slots that they read (eight 30-node trees 30.8 -> 33.2).
constexpr int kEagerSlots = 16;
constexpr size_t kEagerBytes = 8 << 20;
template <typename T>
__global__ __launch_bounds__(256) void attn_merge_eager_kernel(int rows, int D, int splits, const float *__restrict__ part_o,
                                                               const float *__restrict__ part_ml, T *__restrict__ out,
                                                               float *__restrict__ lse) {
  const int tpr = D >> 2;  // threads per row (D % 4 == 0)
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const int row = (int)(gid / tpr);
  const int piece = (int)(gid - (long)row * tpr);
  if (row >= rows) return;
  const merge_f32x2 *ml = reinterpret_cast<const merge_f32x2 *>(part_ml) + (size_t)row * splits;
  const merge_f32x4 *po = reinterpret_cast<const merge_f32x4 *>(part_o) + (size_t)row * splits * tpr + piece;
  merge_f32x2 x[kEagerSlots];
  merge_f32x4 o[kEagerSlots];
#pragma unroll
  for (int c = 0; c < kEagerSlots; ++c) {
    x[c] = (merge_f32x2){0.f, 0.f};
    if (c < splits) x[c] = ml[c];
  }
#pragma unroll
  for (int c = 0; c < kEagerSlots; ++c)
    if (c < splits) o[c] = po[(size_t)c * tpr];
  if (x[0].y < 0.f) return;  // the attention kernel wrote this row out itself
  float m = -__builtin_huge_valf(), l = 0.f;
  int live = 0;  // the first empty slot ends the list
#pragma unroll
  for (int c = 0; c < kEagerSlots; ++c) {
    if (live == c && x[c].y > 0.f) {
      m = fmaxf(m, x[c].x);
      live = c + 1;
    }
  }
  merge_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kEagerSlots; ++c) {
    if (c < live) {
      const float w = expf(x[c].x - m);
      l = add_weights(l, x[c].y, w, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(o[c][e], w, acc[e]);
    }
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
  store_row4(out + (size_t)row * D + piece * 4, acc * inv);
  if (lse && piece == 0) lse[row] = m + logf(l);
}

}  // namespace

hipError_t launch_attn_scalar(const hb_attn_desc &d, const AttnPlan &plan, const void *q,
                              const void *k_tree, const void *v_tree, const void *k_pool,
                              const void *v_pool, const int32_t *block_table,
                              const int32_t *prefix_len, const int32_t *node_offset,
                              const int32_t *parent, void *out, float *lse, float *part_o,
                              float *part_ml, ClearArgs clear, hipStream_t s) {
  dim3 grid((unsigned)(d.total_nodes * d.num_q_heads), (unsigned)plan.splits);
#define HB_ATTN_SCALAR(T_, E_)                                                                                  \
  attn_scalar_kernel<T_, E_><<<grid, kThreads, 0, s>>>(d, plan.splits, plan.chunk_tokens, (const T_ *)q,        \
      (const T_ *)k_tree, (const T_ *)v_tree, (const T_ *)k_pool, (const T_ *)v_pool, block_table, prefix_len,  \
      node_offset, parent, (T_ *)out, lse, part_o, part_ml, clear)
  if (eager_takes(d, (int64_t)grid.x * grid.y, plan.splits)) {
    attn_scalar_eager_kernel<<<grid, kEagerThreads, 0, s>>>(d, plan.splits, plan.chunk_tokens, (const float *)q, (const float *)k_tree,
                                                            (const float *)v_tree, (const float *)k_pool, (const float *)v_pool,
                                                            block_table, prefix_len, node_offset, parent, (float *)out, lse, part_o,
                                                            part_ml, clear);
    return hipGetLastError();
  }
  const int e = d.head_dim <= 64 ? 1 : d.head_dim <= 128 ? 2 : 4;  // head dimensions per lane
  if (d.dtype == HB_F32) {
    if (e == 1) HB_ATTN_SCALAR(float, 1);
    else if (e == 2) HB_ATTN_SCALAR(float, 2);
    else HB_ATTN_SCALAR(float, 4);
  } else {
    if (e == 1) HB_ATTN_SCALAR(bf16_t, 1);
    else if (e == 2) HB_ATTN_SCALAR(bf16_t, 2);
    else HB_ATTN_SCALAR(bf16_t, 4);
  }
#undef HB_ATTN_SCALAR
  return hipGetLastError();
}

hipError_t launch_attn_merge(const hb_attn_desc &d, const AttnPlan &plan, const float *part_o,
                             const float *part_ml, void *out, float *lse, hipStream_t s) {
  int rows = d.total_nodes * d.num_q_heads;
  long threads = (long)rows * (d.head_dim / 4);
  dim3 grid((unsigned)((threads + 255) / 256));
  if (plan.splits <= kEagerSlots && (size_t)rows * plan.splits * d.head_dim * sizeof(float) <= kEagerBytes) {
    if (d.dtype == HB_F32)
      attn_merge_eager_kernel<float><<<grid, 256, 0, s>>>(rows, d.head_dim, plan.splits, part_o, part_ml, (float *)out, lse);
    else
      attn_merge_eager_kernel<bf16_t><<<grid, 256, 0, s>>>(rows, d.head_dim, plan.splits, part_o, part_ml, (bf16_t *)out, lse);
    return hipGetLastError();
  }
  if (d.dtype == HB_F32)
    attn_merge_kernel<float><<<grid, 256, 0, s>>>(rows, d.head_dim, plan.splits, part_o, part_ml, (float *)out, lse);
  else
    attn_merge_kernel<bf16_t><<<grid, 256, 0, s>>>(rows, d.head_dim, plan.splits, part_o, part_ml, (bf16_t *)out, lse);
  return hipGetLastError();
}

}  // namespace hb
