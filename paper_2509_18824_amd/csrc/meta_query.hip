// Target-feature aggregation with meta queries (the paper, Section 3.1.1, Eq. 1): for every token,
// Q learnable queries attend over the L layer features of that token (multi-head, H heads of size
// d = D / H) and the Q outputs are flattened.
//
// The queries do not depend on the token, so the key projection is folded into them once:
//   score(q, h, l) = (f_q W_q^T)_{q,h} . (f_i[l] W_k^T)_h / sqrt(d) = A[h Q + q] . f_i[l],
//   A[h Q + q] = (f_q W_q^T)_{q,h} W_k[h d .. (h + 1) d, :] / sqrt(d)          (a D-vector)
// which removes the L x D x D key projection per token: the scores are one small dense product
// [H Q, D] x [D, L] per token, on the matrix cores.  A is kept as the sum of two bf16 matrices
// (value rounded to bf16 plus the rounded remainder), so that folding costs the scores no
// accuracy against projecting keys in fp32.
//
// meta_scores_kernel: the scores of all tokens are one dense product A [H Q, D] x feats^T
// [D, S L].  A workgroup takes eight tokens and a range of D, 64 features at a time: the tokens'
// features and both halves of A go from memory to LDS directly, features two steps and A one step ahead
// of the matrix instructions (16x16x32); four pairs of wavefronts take two tokens each and half of the
// rows of A.  With few tokens D is spread over several workgroups, which write partial scores (fp32) to
// a workspace.  2048 tokens, 28 layers, D = 3584: 110 us with W_v's rearrangement (411 MB of features and
// nearly as much of A through the L2s); 122 with features one step ahead, 183 with features loaded in
// fragment order, four rows per four lanes.
// meta_mix_kernel, one workgroup per token (and per 4096 features): sums the partial scores, one thread per (head, query)
// row does the softmax over the L layers, and every thread then mixes the token's projected values
// (v_proj = f_i W_v^T, a plain linear layer run beforehand) for eight feature columns of all Q
// queries:  pre[q, c] = sum_l P[head(c) Q + q, l] v_proj[l, c].
// meta_project_kernel, meta_project_wide_kernel: the features are mixed first and W_v is applied to the mixture.  Where tokens in
// sixteens leave CUs idle, workgroups share D: meta_softmax_kernel makes the probabilities once, meta_sum_kernel adds the shares.
// The output projection and the skip connection (Section 3.1.2) are a linear layer with residual
// run afterwards on pre; the mixing kernel also copies the residual rows f_i[residual_layers[q]].
#include "hb_internal.h"

#include <algorithm>
#include <type_traits>

namespace hb {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;       // the two set-up kernels
constexpr int kWaves = 4;
constexpr int kScoreWaves = 8;      // wavefronts of meta_scores_kernel
constexpr int kScoreThreads = 64 * kScoreWaves;
constexpr int kTokPerWave = 2;      // tokens whose scores one wavefront accumulates
constexpr int kTokPerGroup = 8;
constexpr int kSlice = 256;         // features: the unit in which D is dealt to workgroups
constexpr int kMixThreads = 512;      // meta_mix_kernel: one thread per eight feature columns
constexpr int kBufferFlags = 0x00027000;  // untyped 32-bit elements
constexpr int kMaxParts = 16;         // workgroup columns of the score kernel
constexpr int kMaxRowTiles = 6;   // H * Q <= 96
constexpr int kMaxRows = 16 * kMaxRowTiles;
constexpr int kMaxL = 32;
constexpr int kLdsL = kMaxL + 1;    // row stride of the score tables in LDS: one thread per row reads without bank conflicts
constexpr int kMaxQ = 4;

// qproj[q, n] = sum_c f_q[q, c] w_q[n, c]: one wavefront per output
__global__ __launch_bounds__(kThreads) void meta_qproj_kernel(int Q, int D, const bf16_t *__restrict__ f_q,
                                                              const bf16_t *__restrict__ w_q,
                                                              float *__restrict__ qproj) {
  const int out = blockIdx.x * kWaves + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (out >= Q * D) return;
  const int q = out / D, n = out - q * D;
  float acc = 0.f;
  for (int c = lane; c < D; c += 64) acc += bf16_to_f32(f_q[(size_t)q * D + c]) * bf16_to_f32(w_q[(size_t)n * D + c]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) qproj[out] = acc;
}

// A[h Q + q, c] = scale * sum_j qproj[q, h d + j] w_k[h d + j, c], split into two bf16 matrices;
// rows from H * Q up to rows_pad are zero
__global__ __launch_bounds__(kThreads) void meta_fold_kernel(int Q, int D, int H, int rows_pad, float scale,
                                                             const float *__restrict__ qproj,
                                                             const bf16_t *__restrict__ w_k,
                                                             bf16_t *__restrict__ a_hi, bf16_t *__restrict__ a_lo) {
  const int c = blockIdx.x * kThreads + threadIdx.x;
  const int r = blockIdx.y;
  if (c >= D) return;
  float acc = 0.f;
  if (r < H * Q) {
    const int h = r / Q, q = r - h * Q, d = D / H;
    for (int j = 0; j < d; ++j) acc += qproj[(size_t)q * D + h * d + j] * bf16_to_f32(w_k[(size_t)(h * d + j) * D + c]);
    acc *= scale;
  }
  const bf16_t hi = f32_to_bf16(acc);
  a_hi[(size_t)r * D + c] = hi;
  a_lo[(size_t)r * D + c] = f32_to_bf16(acc - bf16_to_f32(hi));
}

struct ResidualLayers {
  int32_t layer[kMaxQ];
  int32_t on;
};

// The first pack_wgs workgroups rearrange W_v for meta_project_kernel, where that follows.
__device__ void pack_values(int wave, int waves, int D, const u32x4 *__restrict__ w_v, u32x4 *__restrict__ packed);

constexpr int kScoreFeatRows = kTokPerGroup * kMaxL;                    // LDS rows of 64 features per stage
constexpr int kScoreFeatStage = kScoreFeatRows * 8, kScoreAStage = 2 * kMaxRows * 8;                       // pieces
constexpr int kScoreFeatLoads = kScoreFeatRows / 8 / kScoreWaves, kScoreALoads = 2 * kMaxRows / 8 / kScoreWaves;  // of a wavefront per step
constexpr size_t kScoreLds = (3 * (size_t)kScoreFeatStage + 2 * (size_t)kScoreAStage) * sizeof(u32x4);

// part[p][s][row][l] (row stride 32): the scores of token s summed over the slices that
// workgroup column p covers
__global__ __launch_bounds__(kScoreThreads) void meta_scores_kernel(int S, int L, int D, int row_tiles,
                                                                    int slices_per_wg, int token_groups, int pack_wgs,
                                                                    const u32x4 *__restrict__ w_v, u32x4 *__restrict__ packed,
                                                                    const u32x4 *__restrict__ feats,
                                                                    const u32x4 *__restrict__ a_fold,
                                                                    float *__restrict__ part) {
  // Features come from memory and have three stages, requested two steps ahead; A comes from the L2s, one step ahead.
  extern __shared__ u32x4 meta_a_lds[];  // [3][features of 8 x 32 rows][8 pieces], [2][A: values, then remainders][8]
  u32x4 *lds_a = meta_a_lds + 3 * kScoreFeatStage;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x < pack_wgs) {
    pack_values(blockIdx.x * kScoreWaves + wave, pack_wgs * kScoreWaves, D, w_v, packed);
    return;
  }
  const int id = blockIdx.x - pack_wgs;
  const int token_group = id % token_groups, column = id / token_groups;
  const int rows_pad = 16 * row_tiles;
  const int j16 = lane & 15, kq = lane >> 4;
  const int row_bytes = D * 2;
  const int tok0 = token_group * kTokPerGroup;
  const int slices = D / kSlice;
  const int sl_begin = column * slices_per_wg;
  const int sl_end = sl_begin + slices_per_wg < slices ? sl_begin + slices_per_wg : slices;
  const int k_begin = sl_begin * (kSlice / 64), steps = (sl_end - sl_begin) * (kSlice / 64);

  // Loads of eight rows of 128 bytes, pieces swizzled on the source side; rows past the tokens' or past
  // A's are out of range and arrive as zeros.  Layers past L are the next token's (their scores are
  // written and not read).
  typedef __attribute__((address_space(3))) void *lptr_t;
  const auto f_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(feats + (size_t)tok0 * L * (row_bytes / 16)), 0,
                                                        min(kTokPerGroup, S - tok0) * L * row_bytes, kBufferFlags);
  const auto a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)a_fold, 0, 2 * rows_pad * row_bytes, kBufferFlags);
  const int r8 = lane >> 3;
  auto swz = [](int r, int c) { return r * 8 + (c ^ (r & 7)); };
  const int src = (wave * 8 + r8) * row_bytes + ((lane & 7) ^ r8) * 16;
  auto issue_feats = [&](int t, int stage) {
#pragma unroll
    for (int i = 0; i < kScoreFeatLoads; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(f_rsrc, (lptr_t)(meta_a_lds + stage * kScoreFeatStage + (wave + i * kScoreWaves) * 64), 16,
                                               src + i * kScoreWaves * 8 * row_bytes, (k_begin + min(t, steps - 1)) * 128, 0, 0);
  };
  auto issue_a = [&](int t) {
#pragma unroll
    for (int i = 0; i < kScoreALoads; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lptr_t)(lds_a + (t & 1) * kScoreAStage + (wave + i * kScoreWaves) * 64), 16,
                                               src + i * kScoreWaves * 8 * row_bytes, (k_begin + min(t, steps - 1)) * 128, 0, 0);
  };
  const int tw = (wave & 3) * kTokPerWave;   // first token
  const int mt0 = (wave >> 2) * (kMaxRowTiles / 2);
  f32x4 acc[kMaxRowTiles / 2][kTokPerWave][2];
#pragma unroll
  for (int mt = 0; mt < kMaxRowTiles / 2; ++mt)
#pragma unroll
    for (int t = 0; t < kTokPerWave; ++t)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) acc[mt][t][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
  issue_a(0);
  issue_feats(0, 0);
  issue_feats(1, 1);
  issue_a(1);
  issue_feats(2, 2);
  int stage = 0;
#pragma unroll 1
  for (int st = 0; st < steps; ++st) {
    // This step's loads have landed; in flight stay the features of the next two steps and the next A.
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * kScoreFeatLoads + kScoreALoads) : "memory");
    const u32x4 *f = meta_a_lds + stage * kScoreFeatStage, *ah = lds_a + (st & 1) * kScoreAStage, *al = ah + rows_pad * 8;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 x[kTokPerWave][2];
#pragma unroll
      for (int t = 0; t < kTokPerWave; ++t)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) x[t][ct] = __builtin_bit_cast(bf16x8, f[swz((tw + t) * L + 16 * ct + j16, 4 * ks + kq)]);
#pragma unroll
      for (int mt = 0; mt < kMaxRowTiles / 2; ++mt) {
        if (mt0 + mt < row_tiles) {
          const int at = swz(16 * (mt0 + mt) + j16, 4 * ks + kq);
          const bf16x8 h8 = __builtin_bit_cast(bf16x8, ah[at]);
          const bf16x8 l8 = __builtin_bit_cast(bf16x8, al[at]);
          // values for all, then remainders for all: neighbours do not wait for each other's sums
#pragma unroll
          for (int t = 0; t < kTokPerWave; ++t)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[mt][t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h8, x[t][ct], acc[mt][t][ct], 0, 0, 0);
#pragma unroll
          for (int t = 0; t < kTokPerWave; ++t)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[mt][t][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l8, x[t][ct], acc[mt][t][ct], 0, 0, 0);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // everybody has read the stages
    issue_a(st + 2);
    issue_feats(st + 3, stage);
    stage = stage == 2 ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may land in LDS that belongs to somebody else
  // lane (j16, kq) holds rows 16 mt + 4 kq + r of layer 16 ct + j16
#pragma unroll
  for (int t = 0; t < kTokPerWave; ++t) {
    if (tok0 + tw + t < S) {
      float *dst = part + ((size_t)column * S + tok0 + tw + t) * rows_pad * kMaxL;
#pragma unroll
      for (int mt = 0; mt < kMaxRowTiles / 2; ++mt) {
        if (mt0 + mt < row_tiles) {
#pragma unroll
          for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[(16 * (mt0 + mt) + 4 * kq + r) * kMaxL + 16 * ct + j16] = acc[mt][t][ct][r];
        }
      }
    }
  }
}

__global__ __launch_bounds__(kMixThreads) void meta_mix_kernel(int S, int L, int D, int H, int Q, int rows_pad,
                                                               int parts, const float *__restrict__ part,
                                                               const u32x4 *__restrict__ feats,
                                                               const u32x4 *__restrict__ v_proj, ResidualLayers res,
                                                               u32x4 *__restrict__ pre, u32x4 *__restrict__ res_out) {
  __shared__ float prob[kMaxRows][kLdsL];
  const int s = blockIdx.x;
  const int tid = threadIdx.x;
  const int dp = D / 8;                       // 16-byte pieces per feature row
  const u32x4 *f_tok = feats + (size_t)s * L * dp;
  const u32x4 *g_tok = v_proj + (size_t)s * L * dp;
  const int rows = H * Q;

  // Everything the token needs from memory is requested up front, in one round: the projected
  // values of this thread's eight columns for all layers, the residual rows, the partial scores.
  const int d8 = (D / H) / 8;  // 16-byte pieces per head
  const int cg = blockIdx.y * kMixThreads + tid;  // this thread's 16-byte column group
  const bool mixer = cg < dp;
  u32x4 g[kMaxL], rr[kMaxQ];
#pragma unroll
  for (int l = 0; l < kMaxL; ++l)
    if (mixer && l < L) g[l] = g_tok[(size_t)l * dp + cg];
#pragma unroll
  for (int q = 0; q < kMaxQ; ++q)
    if (mixer && res.on && q < Q) rr[q] = f_tok[(size_t)res.layer[q] * dp + cg];

  // ---- the token's scores: sum over the workgroup columns of the score kernel ----------------
  const int n4 = rows_pad * kMaxL / 4;  // float4 pieces of one partial table
  const f32x4 *part4 = reinterpret_cast<const f32x4 *>(part);
#pragma unroll
  for (int it = 0; it < (kMaxRows * kMaxL / 4 + kMixThreads - 1) / kMixThreads; ++it) {
    const int i = tid + it * kMixThreads;
    if (i < n4) {
      f32x4 v[kMaxParts];
#pragma unroll
      for (int p = 0; p < kMaxParts; ++p)
        if (p < parts) v[p] = part4[((size_t)p * S + s) * n4 + i];
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kMaxParts; ++p)
        if (p < parts) t += v[p];
      const int row = i / (kMaxL / 4), c4 = i % (kMaxL / 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) prob[row][4 * c4 + e] = t[e];
    }
  }
  __syncthreads();

  // ---- softmax over the layers, one thread per (head, query) row -----------------------------
  if (tid < rows) {
    float sc[kMaxL];
    float mx = -__builtin_huge_valf();
#pragma unroll
    for (int l = 0; l < kMaxL; ++l) {
      sc[l] = prob[tid][l];
      if (l < L) mx = fmaxf(mx, sc[l]);
    }
    float sum = 0.f;
#pragma unroll
    for (int l = 0; l < kMaxL; ++l) {
      sc[l] = l < L ? __expf(sc[l] - mx) : 0.f;
      sum += sc[l];
    }
    const float inv = 1.f / sum;
#pragma unroll
    for (int l = 0; l < kMaxL; ++l) prob[tid][l] = sc[l] * inv;
  }
  __syncthreads();

  // ---- mix the projected values: eight feature columns per thread, all queries ---------------
  if (!mixer) return;
  const int h = cg / d8;
  float o[kMaxQ][8];
#pragma unroll
  for (int q = 0; q < kMaxQ; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) o[q][e] = 0.f;
#pragma unroll
  for (int l = 0; l < kMaxL; ++l) {
    if (l < L) {
      float gv[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        gv[2 * e] = __uint_as_float(g[l][e] << 16);
        gv[2 * e + 1] = __uint_as_float(g[l][e] & 0xffff0000u);
      }
#pragma unroll
      for (int q = 0; q < kMaxQ; ++q) {
        if (q < Q) {
          const float p = prob[h * Q + q][l];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[q][e] += p * gv[e];
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kMaxQ; ++q) {
    if (q < Q) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = (uint32_t)f32_to_bf16(o[q][2 * e]) | ((uint32_t)f32_to_bf16(o[q][2 * e + 1]) << 16);
      pre[((size_t)s * Q + q) * dp + cg] = w;
      if (res.on) res_out[((size_t)s * Q + q) * dp + cg] = rr[q];
    }
  }
}

// ---- values projected after the mixing -------------------------------------------------------
// pre[i, q, head h] = sum_l P[i, h, q, l] (f_i[l] W_v^T)_h = (sum_l P[i, h, q, l] f_i[l]) W_v,h^T:
// mixing the features first leaves Q rows per token and head to project instead of L rows per
// token, L / Q times less matrix work (28 layers, 3 queries: 9 times).  The mixed features, H Q
// vectors of D per token, would be three times the features in memory; here a workgroup makes them
// slice by slice in LDS and uses them up at once.
//
// Workgroup: 4 or 16 tokens and up to eight heads (their hq rows: head-major, the queries of a head
// together).  It walks D:
//   mixing   feats^T P^T on the matrix cores per token (features as rows, the transposing LDS read
//            supplies them; P^T of a wavefront's tokens stays in registers for the whole kernel).
//            The two 16-feature tiles of 32 features are interleaved in fours, so that a lane holds
//            eight consecutive features of one hq row and stores them as one piece.
//   product  W_v slice (straight from memory in fragment layout) times the mixed features of the
//            wavefront's head: accumulators for all of the workgroup's tokens.
// P and the mixed features are each a bf16 value plus the bf16 remainder (two products, about 2^-17
// relative): what was float32 when values were projected first stays better than bf16.
// With 4 tokens (meta_project_kernel) mixing and product of 64 features follow each other, each covering the other's loads:
// the first half of a slice's weights is requested among the matrix instructions of the product before it, the second half
// during its own mixing, the next slice's features (global -> LDS) among those of its product.
//
// What bounds it: with 4 tokens the path L2 -> CU (every 4 tokens read all of W_v once); with 16 (see
// meta_project_wide_kernel) matrix work 43 % of the clocks, LDS reads behind the barriers, features from memory at 1.7 TB/s.
// 2048 tokens, 28 layers, D = 3584, 28 heads, 3 queries: 460 us (530 with 64 features between barriers); the
// value projection of all layers and the mixing of its results took 1478 + 161 us.  96 tokens 62 us against 76 + 15 (40 + 12 by
// workgroups of 16 that share D, as they now do).
constexpr int kMpThreads = 512;
constexpr int kMpWaves = 8;
constexpr int kMpHq = 24;           // hq rows of a workgroup at most (16 tokens: 48 KB of mixed features beside 96 to 112 KB of features)
constexpr int kMpHeadDim = 128;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// W_v in fragment order, made on every call by workgroups of the score kernel's launch: 16 rows x 32
// columns are 1 KB in the order of the lanes, [32 columns][16 rows][lane]: all that the workgroups want of a slice of
// features is in one piece, spread over all channels of the L2s (with the columns inside the rows every head's part of a
// slice began a multiple of 2 KB from the others').  Read
// from the matrix itself, four neighbouring lanes of a fragment load touch four rows and a load takes
// 64 clocks instead of 16 (measured: 34 GB/s per CU, and 2.5 times the time for the whole kernel).
__device__ void pack_values(int wave, int waves, int D, const u32x4 *__restrict__ w_v, u32x4 *__restrict__ packed) {
  const int lane = threadIdx.x & 63;
  const int dp = D / 8, steps = D / 64;
  constexpr int kBatch = 4;
  const int tiles = D / 16 * steps;  // 16 rows x 64 columns: 2 KB
  for (int t0 = wave * kBatch; t0 < tiles; t0 += waves * kBatch) {
    u32x4 x[kBatch][2];  // lane -> row lane / 8 (+ 8), piece lane % 8
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int t = min(t0 + i, tiles - 1);
      const u32x4 *src = w_v + (size_t)(t / steps * 16 + (lane >> 3)) * dp + t % steps * 8 + (lane & 7);
      x[i][0] = src[0];
      x[i][1] = src[(size_t)8 * dp];
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int t = min(t0 + i, tiles - 1);
      u32x4 *dst = packed + ((size_t)(2 * (t % steps) + ((lane & 7) >> 2)) * (D / 16) + t / steps) * 64 + (lane & 3) * 16 + (lane >> 3);
      dst[0] = x[i][0];
      dst[8] = x[i][1];
    }
  }
}

// value = bf16 (truncated) + bf16 remainder; two values per word
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &hi, uint32_t &lo) {
  const uint32_t ua = __float_as_uint(a) & 0xffff0000u, ub = __float_as_uint(b) & 0xffff0000u;
  hi = (ua >> 16) | ub;
  const f32x2 r = {a - __uint_as_float(ua), b - __uint_as_float(ub)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
}

// Four transposing reads of 8 bytes per lane.  Inline asm with its own wait: before the builtin the
// compiler waits for every load in flight, taking it for a reader of the features on their way.
__device__ __forceinline__ void tr_fragments(uint32_t at0, uint32_t at1, bf16x8 (&a)[2]) {
  bf16x4 x0, x1, y0, y1;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4\n\t"
      "ds_read_b64_tr_b16 %1, %5\n\t"
      "ds_read_b64_tr_b16 %2, %4 offset:8\n\t"
      "ds_read_b64_tr_b16 %3, %5 offset:8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x0), "=&v"(x1), "=&v"(y0), "=&v"(y1)
      : "v"(at0), "v"(at1)
      : "memory");
  a[0] = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
  a[1] = __builtin_shufflevector(y0, y1, 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same for two tokens.
__device__ __forceinline__ void tr_fragments(uint32_t at0, uint32_t at1, uint32_t at2, uint32_t at3, bf16x8 (&a)[2][2]) {
  bf16x4 x[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %9\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:8\n\t"
      "ds_read_b64_tr_b16 %3, %9 offset:8\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\t"
      "ds_read_b64_tr_b16 %5, %11\n\t"
      "ds_read_b64_tr_b16 %6, %10 offset:8\n\t"
      "ds_read_b64_tr_b16 %7, %11 offset:8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
      : "v"(at0), "v"(at1), "v"(at2), "v"(at3)
      : "memory");
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 2; ++i) a[t][i] = __builtin_shufflevector(x[4 * t + 2 * i], x[4 * t + 2 * i + 1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// Softmax over the layers of row row0 + hq of token tok0 + t; to entry at of tab[2][n][4 pieces], values and remainders.
__device__ __forceinline__ void softmax_layers(int at, int t, int hq, int n, int S, int L, int tok0, int row0, int rows_pad,
                                               int parts, const float *__restrict__ part, u32x4 *tab) {
  const int s = min(tok0 + t, S - 1);
  const f32x4 *src = reinterpret_cast<const f32x4 *>(part + ((size_t)s * rows_pad + row0 + hq) * kMaxL);
  const size_t stride = (size_t)S * rows_pad * (kMaxL / 4);
  f32x4 sc[kMaxL / 4];
#pragma unroll
  for (int i = 0; i < kMaxL / 4; ++i) sc[i] = src[i];
  for (int p = 1; p < parts; ++p)
#pragma unroll
    for (int i = 0; i < kMaxL / 4; ++i) sc[i] += src[p * stride + i];
  float mx = -__builtin_huge_valf();
#pragma unroll
  for (int l = 0; l < kMaxL; ++l)
    if (l < L) mx = fmaxf(mx, sc[l >> 2][l & 3]);
  float sum = 0.f;
#pragma unroll
  for (int l = 0; l < kMaxL; ++l) {
    const float e = l < L ? __expf(sc[l >> 2][l & 3] - mx) : 0.f;
    sc[l >> 2][l & 3] = e;
    sum += e;
  }
  const float inv = 1.f / sum;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u32x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int l = 8 * i + 2 * e;
      uint32_t a, b;
      split_pair(sc[l >> 2][l & 3] * inv, sc[(l + 1) >> 2][(l + 1) & 3] * inv, a, b);
      hi[e] = a;
      lo[e] = b;
    }
    tab[at * 4 + i] = hi;
    tab[(n + at) * 4 + i] = lo;
  }
}

// 4 tokens: a head's rows are one tile, row = q * 4 + token.  NT: 16-column tiles of a head per wavefront; 8 / NT
// wavefronts share a head.
template <int NT>
__global__ __launch_bounds__(kMpThreads) void meta_project_kernel(
    int S, int L, int D, int H, int Q, int hg, int rows_pad, int parts, const float *__restrict__ part,
    const u32x4 *__restrict__ feats, const u32x4 *__restrict__ packed, ResidualLayers res, bf16_t *__restrict__ pre,
    u32x4 *__restrict__ res_out) {
  constexpr int kWavesPerHead = 8 / NT;
  constexpr int TG = 4, NS = 2;            // tokens; slices of features in LDS
  constexpr int FI = 2;                    // feature loads of a wavefront per slice
  extern __shared__ u32x4 meta_a_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j16 = lane & 15, kq = lane >> 4;
  const int dp = D / 8;
  const int tok0 = blockIdx.x * TG, h0 = blockIdx.y * hg;
  const int heads = min(hg, H - h0);        // >= 1
  const int hq_rows = heads * Q;
  const int frows = min(TG, S - tok0) * L;  // feature rows of the workgroup, consecutive in memory
  u32x4 *lds_f = meta_a_lds;                // [NS][FI * 8 wavefronts * 8 rows][8]
  constexpr int kStagePieces = FI * kMpWaves * 64;
  u32x4 *lds_m = meta_a_lds + NS * kStagePieces;  // [2][mixed rows][8]: values, remainders
  const int mixed = hg * 16;

  // Features: 64 rows per round of the wavefronts, lane -> row lane / 8 of its wavefront's eight,
  // piece swizzled on the source side; rows past the workgroup's are out of the buffer's range and
  // arrive as zeros.  Always FI loads (the waits below count them): a repeated slice changes nothing.
  typedef __attribute__((address_space(3))) void *lptr_t;
  const int steps = D / 64;
  const auto f_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(feats + (size_t)tok0 * L * dp), 0, frows * dp * 16, kBufferFlags);
  const int f_src = (wave * 8 + (lane >> 3)) * dp * 16 + ((lane & 7) ^ (((wave * 8 + (lane >> 3)) >> 1) & 7)) * 16;
  auto issue_feat = [&](int kt, int i) {
    const int k = min(kt, steps - 1);
    u32x4 *stage = lds_f + (kt % NS) * kStagePieces + wave * 64;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(f_rsrc, (lptr_t)(stage + i * kMpWaves * 64), 16,
                                             f_src + i * kMpWaves * 8 * dp * 16, k * 128, 0, 0);
  };
  auto issue_feats = [&](int kt) {
#pragma unroll
    for (int i = 0; i < FI; ++i) issue_feat(kt, i);
  };
  issue_feats(0);

  // ---- softmax over the layers, one thread per (token, hq row); P goes through LDS ------------
  const int t = wave >> 1, g = wave & 1;    // the token whose mixing this wavefront does, and the half of the slice
  bf16x8 p_hi[2], p_lo[2];
  {
    u32x4 *tab = lds_m;  // [2][TG * hq_rows][4 pieces]
    const int n = TG * hq_rows;
    if (tid < n) {
      softmax_layers(tid, tid / hq_rows, tid % hq_rows, n, S, L, tok0, h0 * Q, rows_pad, parts, part, tab);
    }
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int hq = 16 * ct + j16;
      const int at = t * hq_rows + min(hq, hq_rows - 1);
      const u32x4 zero = {0u, 0u, 0u, 0u};
      p_hi[ct] = __builtin_bit_cast(bf16x8, hq < hq_rows ? tab[at * 4 + kq] : zero);
      p_lo[ct] = __builtin_bit_cast(bf16x8, hq < hq_rows ? tab[(n + at) * 4 + kq] : zero);
    }
  }

  // the residual rows of the workgroup's columns
  if (res.on) {
    const int cols = heads * (kMpHeadDim / 8), n = TG * Q * cols;
    for (int i = tid; i < n; i += kMpThreads) {
      const int row = i / cols, c = h0 * (kMpHeadDim / 8) + i - row * cols;
      const int t = row / Q, q = row - t * Q;
      if (tok0 + t < S) res_out[((size_t)(tok0 + t) * Q + q) * dp + c] = feats[((size_t)(tok0 + t) * L + res.layer[q]) * dp + c];
    }
  }

  // transposing reads of the mixing: lane -> layer row and 8-byte half piece.  Layers past L repeat
  // the last one (their probabilities are zero).
  const uint32_t f_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4 *)lds_f;
  uint32_t f_off[2];  // by half of the lane group's eight layers; ^ 64 for the slice's second 32 features
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    const int r = t * L + min(8 * kq + 4 * hf + (j16 >> 2), L - 1);
    f_off[hf] = (f_lds + r * 128 + ((j16 & 3) ^ ((r >> 1) & 7)) * 16) ^ (64 * g);
  }

  const bool active = wave / kWavesPerHead < heads;        // a wavefront too many repeats the last head
  const int hl = min(wave / kWavesPerHead, heads - 1);     // this wavefront's head
  const int n0 = (wave % kWavesPerHead) * NT * 16;         // its first column in the head
  const int w_step = D / 16 * 1024;  // bytes of 32 columns
  const auto w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(packed + (size_t)((h0 + hl) * 8 + n0 / 16) * 64), 0,
                                                        (2 * steps - 1) * w_step + NT * 1024, kBufferFlags);
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

  bf16x8 w[2][NT];
  auto issue_weight = [&](int kt, int ks, int nt) {
    const int k = min(kt, steps - 1);
    w[ks][nt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane * 16, (2 * k + ks) * w_step + nt * 1024, 0));
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the count below starts here
  issue_feats(1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) issue_weight(0, 0, nt);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
  for (int kt = 0; kt < steps; ++kt) {
    // The slice's features have landed (newer loads: with two stages the next slice's features; the first
    // half of the slice's weights); everybody is done with the previous mixed features.
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 1) * FI + NT) : "memory");
    const uint32_t stage = (uint32_t)(kt % NS) * (uint32_t)(kStagePieces * 16);
    // the second half of the slice's weights
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) issue_weight(kt, 1, nt);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a[2];
    tr_fragments(stage + f_off[0], stage + f_off[1], a);
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      if (16 * ct >= hq_rows) break;
      f32x4 c[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], p_hi[ct], (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], p_lo[ct], c[i], 0, 0, 0);
      }
      const int hq = 16 * ct + j16;
      u32x4 hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t x, y;
        split_pair(c[e >> 1][2 * (e & 1)], c[e >> 1][2 * (e & 1) + 1], x, y);
        hi[e] = x;
        lo[e] = y;
      }
      if (hq < hq_rows) {
        const int row = (hq / Q) * 16 + (hq % Q) * 4 + t;
        const int at = row * 8 + ((4 * g + kq) ^ ((row + hq) & 7));
        lds_m[at] = hi;
        lds_m[mixed * 8 + at] = lo;
      }
    }
    // the mixed features are complete; everybody is done with the slice's features
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // The slice's weights are waited for before the next features are requested: the compiler's wait
    // at their first use would include the newer loads.
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(w[ks][nt]));
    // The next slice's features and then the first half of its weights are requested among the matrix instructions: in
    // front of them and behind them the address unit had every wavefront wait.
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int row = hl * 16 + j16, hq = hl * Q + (j16 >> 2);
      const int at = row * 8 + ((4 * ks + kq) ^ ((row + hq) & 7));
      const bf16x8 hi = __builtin_bit_cast(bf16x8, lds_m[at]);
      const bf16x8 lo = __builtin_bit_cast(bf16x8, lds_m[mixed * 8 + at]);
#pragma unroll
      for (int nt = 0; nt < NT; nt += 2) {  // two columns in turn: neighbours do not wait for each other's sums
        acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt], hi, acc[nt], 0, 0, 0);
        acc[nt + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt + 1], hi, acc[nt + 1], 0, 0, 0);
        acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt], lo, acc[nt], 0, 0, 0);
        acc[nt + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][nt + 1], lo, acc[nt + 1], 0, 0, 0);
        const int loads = ks ? NT : FI;
#pragma unroll
        for (int i = nt * loads / NT; i < (nt + 2) * loads / NT; ++i) {
          if (ks) issue_weight(kt + 1, 0, i);
          else issue_feat(kt + NS, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // lane (j16, kq) holds columns 16 nt + 4 kq .. + 3 of row j16
  if (!active) return;
  const int q = j16 >> 2, s = tok0 + (j16 & 3);
  if (q >= Q || s >= S) return;
  bf16_t *dst = pre + ((size_t)s * Q + q) * D + (h0 + hl) * kMpHeadDim + n0 + 4 * kq;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    *(u32x2 *)(dst + nt * 16) = (u32x2){(uint32_t)f32_to_bf16(acc[nt][0]) | ((uint32_t)f32_to_bf16(acc[nt][1]) << 16),
                                        (uint32_t)f32_to_bf16(acc[nt][2]) | ((uint32_t)f32_to_bf16(acc[nt][3]) << 16)};
  }
}

// Where several workgroups share D (see there), their probabilities are made once, from all rows of a token: eight lanes a
// row.  probs[2][S][rows][4 pieces of eight layers], values, then remainders.
constexpr int kSoftmaxThreads = 256;
__global__ __launch_bounds__(kSoftmaxThreads) void meta_softmax_kernel(int S, int L, int rows, int rows_pad, int parts,
                                                                       const f32x4 *__restrict__ part, uint32_t *__restrict__ probs) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const int s = blockIdx.x, c4 = threadIdx.x & 7;
  const size_t stride = (size_t)S * rows_pad * (kMaxL / 4);
  for (int row = threadIdx.x >> 3; row < rows; row += kSoftmaxThreads / 8) {  // the eight lanes of a row go together
    const f32x4 *src = part + ((size_t)s * rows_pad + row) * (kMaxL / 4) + c4;
    f32x4 v[kMaxParts];
#pragma unroll
    for (int p = 0; p < kMaxParts; ++p)
      if (p < parts) v[p] = src[p * stride];
    f32x4 sc = v[0];
#pragma unroll
    for (int p = 1; p < kMaxParts; ++p)
      if (p < parts) sc += v[p];
    float mx = -__builtin_huge_valf();
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * c4 + e < L) mx = fmaxf(mx, sc[e]);
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = 4 * c4 + e < L ? __expf(sc[e] - mx) : 0.f;
      sum += sc[e];
    }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    const float inv = 1.f / sum;
    u32x2 hi, lo;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      uint32_t a, b;
      split_pair(sc[2 * e] * inv, sc[2 * e + 1] * inv, a, b);
      hi[e] = a;
      lo[e] = b;
    }
    const size_t at = (((size_t)s * rows + row) * 8 + c4) * 2;
    *(u32x2 *)(probs + at) = hi;
    *(u32x2 *)(probs + (size_t)S * rows * 16 + at) = lo;
  }
}

// The sum over D's parts, in order, of four values, and the residual rows.
__global__ __launch_bounds__(256) void meta_sum_kernel(int S, int L, int D, int Q, int parts, const f32x4 *__restrict__ sums,
                                                       const uint2 *__restrict__ feats, ResidualLayers res, uint2 *__restrict__ pre,
                                                       uint2 *__restrict__ res_out) {
  const size_t n4 = (size_t)S * Q * (D / 4), i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  uint2 r;
  if (res.on) {
    const int d4 = D / 4, col = (int)(i % d4), row = (int)(i / d4), t = row / Q;
    r = feats[((size_t)t * L + res.layer[row - t * Q]) * d4 + col];
  }
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
  for (int p0 = 0; p0 < parts; p0 += 8) {
    f32x4 v[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) v[p] = sums[(size_t)min(p0 + p, parts - 1) * n4 + i];
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p0 + p < parts) x += v[p];
  }
  pre[i] = make_uint2((uint32_t)f32_to_bf16(x[0]) | ((uint32_t)f32_to_bf16(x[1]) << 16),
                      (uint32_t)f32_to_bf16(x[2]) | ((uint32_t)f32_to_bf16(x[3]) << 16));
  if (res.on) res_out[i] = r;
}

// The same for 16 tokens a workgroup: a head's rows are Q tiles of 16 tokens.  A step is 32 features.  The product of a step
// and the mixing of the next one do not depend on each other, so a wavefront does both in one stream of instructions: it
// reads the operands of both from LDS, and between the matrix instructions of the product the mixed values are split and
// stored.  Features arrive in slices of 64 (whole lines: with 32 the kernel waited for memory, 480 us), two of them in LDS,
// requested almost three steps ahead.
constexpr int kMwTok = 16;
constexpr int mw_loads(int L) { return L <= 24 ? 6 : L <= 28 ? 7 : 8; }  // feature loads of a wavefront per slice: 64 rows each
// More than 28 layers with three queries: two slices of 64 leave LDS for five heads only (six groups of 28 heads instead
// of four: 900 tokens 302 -> 345 us), so slices are of 32 features and there are three, requested two steps ahead.
constexpr bool mw_short(int qt, int nt, int fi) { return qt == 3 && nt == 8 && fi == 8; }
constexpr int mw_stage(int fi, bool half) { return (half ? fi / 2 : fi) * kMpWaves * 64; }  // 16-byte pieces of a slice's features

template <int QT, int NT, int FI>
__global__ __launch_bounds__(kMpThreads) void meta_project_wide_kernel(
    int S, int L, int D, int H, int Q, int hg, int rows_pad, int parts, const float *__restrict__ part,
    const u32x4 *__restrict__ feats, const u32x4 *__restrict__ packed, ResidualLayers res, bf16_t *__restrict__ pre,
    u32x4 *__restrict__ res_out, int share, const u32x4 *__restrict__ probs, float *__restrict__ sums) {
  constexpr int kWavesPerHead = 8 / NT;
  constexpr int CT = QT * 8 > 16 && NT == 8 ? 2 : 1;  // tiles of 16 hq rows (NT 4: at most 16 rows)
  extern __shared__ u32x4 meta_a_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j16 = lane & 15, kq = lane >> 4;
  const int dp = D / 8;
  const int tok0 = blockIdx.x * kMwTok, h0 = blockIdx.y * hg;
  const int heads = min(hg, H - h0);  // >= 1
  const int hq_rows = heads * Q;
  const int frows = min(kMwTok, S - tok0) * L;  // feature rows of the workgroup, consecutive in memory
  constexpr bool kShort = mw_short(QT, NT, FI);
  constexpr int kStage = mw_stage(FI, kShort), kStages = kShort ? 3 : 2;
  constexpr int kRow = kShort ? 4 : 8;           // 16-byte pieces of a feature row in a slice
  constexpr int kLoads = kShort ? FI / 2 : FI;   // of a wavefront per slice
  u32x4 *lds_f = meta_a_lds;                     // [kStages][16 L rows][kRow]
  u32x4 *lds_m = meta_a_lds + kStages * kStage;  // [values, remainders][token][hq][4]
  const int mixed = kMwTok * hq_rows * 4;       // pieces

  // Features: 64 rows per round of the wavefronts, lane -> row lane / 8 of its wavefront's eight, piece swizzled on the
  // source side; rows past the workgroup's are out of the buffer's range and arrive as zeros.  Always kLoads loads (the
  // waits below count them): a repeated slice changes nothing.
  typedef __attribute__((address_space(3))) void *lptr_t;
  const int first = (int)blockIdx.z * share, mine = min(share, D / 64 - first);  // of D, in slices of 64
  const int steps = 2 * mine, slices = kShort ? 2 * mine : mine;
  const auto f_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(feats + (size_t)tok0 * L * dp), 0, frows * dp * 16, kBufferFlags);
  constexpr int kRows = 64 / kRow;  // of a load
  const int f_row = wave * kRows + lane / kRow;
  const int f_src = f_row * dp * 16 + (kShort ? lane & 3 : (lane & 7) ^ ((f_row >> 1) & 7)) * 16;
  auto issue_feats = [&](int slice, int slot) {
    const int k = min(slice, slices - 1);
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(f_rsrc, (lptr_t)(lds_f + slot * kStage + (wave + i * kMpWaves) * 64), 16,
                                               f_src + i * kMpWaves * kRows * dp * 16, first * 128 + k * kRow * 16, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < kStages; ++i) issue_feats(i, i);

  // ---- softmax over the layers, one thread per (token, hq row); P goes through LDS ------------
  // Of tokens 2 wave and 2 wave + 1, hq rows in tiles of 16.  Lanes past the last row repeat one of the first tile and store
  // the same values there again.
  auto row_of = [&](int ct) { return 16 * ct + j16 < hq_rows ? 16 * ct + j16 : j16 % hq_rows; };
  bf16x8 p_hi[2][CT], p_lo[2][CT];
  if (probs) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const u32x4 *at = probs + ((size_t)min(tok0 + 2 * wave + tt, S - 1) * (H * Q) + h0 * Q + row_of(ct)) * 4 + kq;
        p_hi[tt][ct] = __builtin_bit_cast(bf16x8, at[0]);
        p_lo[tt][ct] = __builtin_bit_cast(bf16x8, at[(size_t)S * H * Q * 4]);
      }
  } else {
    u32x4 *tab = lds_m;  // [2][16 * hq_rows][4 pieces]
    const int n = kMwTok * hq_rows;
    if (tid < n) softmax_layers(tid, tid / hq_rows, tid % hq_rows, n, S, L, tok0, h0 * Q, rows_pad, parts, part, tab);
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int at = (2 * wave + tt) * hq_rows + row_of(ct);
        p_hi[tt][ct] = __builtin_bit_cast(bf16x8, tab[at * 4 + kq]);
        p_lo[tt][ct] = __builtin_bit_cast(bf16x8, tab[(n + at) * 4 + kq]);
      }
  }

  // the residual rows of the workgroup's columns, kBatch loads in flight (one after the other they took 15 us)
  if (res.on && !sums) {
    constexpr int kBatch = 6;
    const int cols = heads * (kMpHeadDim / 8), n = min(kMwTok, S - tok0) * Q * cols;
    for (int i0 = tid; i0 < n; i0 += kBatch * kMpThreads) {
      u32x4 x[kBatch];
      size_t to[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int i = min(i0 + b * kMpThreads, n - 1);  // past the end: the last one again
        const int row = i / cols, c = h0 * (kMpHeadDim / 8) + i - row * cols;
        const int t = row / Q, q = row - t * Q;
        x[b] = feats[((size_t)(tok0 + t) * L + res.layer[q]) * dp + c];
        to[b] = ((size_t)(tok0 + t) * Q + q) * dp + c;
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) res_out[to[b]] = x[b];
    }
  }

  // Transposing reads of the mixing: lane -> layer row and 8-byte half piece.  Layers past L repeat the last one (their
  // probabilities are zero).
  const uint32_t f_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u32x4 *)lds_f;
  uint32_t f_off[2][2];  // by token and half of the lane group's eight layers; ^ 64 for the second 32 features of 64
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const int r = (2 * wave + tt) * L + min(8 * kq + 4 * hf + (j16 >> 2), L - 1);
      f_off[tt][hf] = f_lds + r * kRow * 16 + ((j16 & 3) ^ (kShort ? 0 : (r >> 1) & 7)) * 16;
    }

  // Mixed features of (token t, row hq): 64 bytes.  The mixing writes 16 rows of one token at a time, the product reads
  // one row of 16 tokens.  With rows of 64 bytes an odd number apart and piece p of every other four of them at p ^ 2, 16-byte
  // reads run at 4 clocks and writes at 9.4 (8 in a row; without the exchange 6 and 17.5); an even number of rows is
  // rotated by the token.
  auto mixed_at = [&](int t, int hq, int p) {
    const int r = hq_rows & 1 ? hq : (hq + (t & 3)) % hq_rows;
    return (t * hq_rows + r) * 4 + (p ^ (((t >> 2) ^ (hq >> 2)) & 1) * 2);
  };
  const bool active = wave / kWavesPerHead < heads;     // a wavefront too many repeats the last head
  const int hl = min(wave / kWavesPerHead, heads - 1);  // this wavefront's head
  const int n0 = (wave % kWavesPerHead) * NT * 16;      // its first column in the head
  int m_write[2][CT], m_read[QT];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) m_write[tt][ct] = mixed_at(2 * wave + tt, row_of(ct), kq);
#pragma unroll
  for (int q = 0; q < QT; ++q) m_read[q] = mixed_at(j16, hl * Q + q, kq);

  const int w_step = D / 16 * 1024;  // bytes of a slice
  const auto w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(packed + (size_t)((h0 + hl) * 8 + n0 / 16) * 64), 0,
                                                        (D / 32 - 1) * w_step + NT * 1024, kBufferFlags);
  f32x4 acc[QT][NT];
#pragma unroll
  for (int q = 0; q < QT; ++q)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[q][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  bf16x8 w[NT];
  auto issue_weight = [&](int kt, int nt) {
    const int k = 2 * first + min(kt, steps - 1);
    w[nt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, lane * 16, k * w_step + nt * 1024, 0));
  };

  // the mixing of one tile of hq rows for both tokens: features x P
  bf16x8 a[2][2];
  f32x4 c[2][2];
  auto mix_products = [&](int ct) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        c[tt][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[tt][i], p_hi[tt][ct], (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 2; ++i) c[tt][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[tt][i], p_lo[tt][ct], c[tt][i], 0, 0, 0);
  };
  u32x4 mix_hi, mix_lo;
  auto split_one = [&](int ct, int n) {  // n: token, pair; the fourth pair completes a piece
    const int tt = n >> 2, e = n & 3;
    uint32_t x, y;
    split_pair(c[tt][e >> 1][2 * (e & 1)], c[tt][e >> 1][2 * (e & 1) + 1], x, y);
    mix_hi[e] = x;
    mix_lo[e] = y;
    if (e == 3) {
      lds_m[m_write[tt][ct]] = mix_hi;
      lds_m[mixed + m_write[tt][ct]] = mix_lo;
    }
  };
  auto read_features = [&](int slot, uint32_t half) {
    const uint32_t at = (uint32_t)slot * (uint32_t)(kStage * 16), x = half * 64;
    tr_fragments(at + (f_off[0][0] ^ x), at + (f_off[0][1] ^ x), at + (f_off[1][0] ^ x), at + (f_off[1][1] ^ x), a);
  };

  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // P is read, the first slices are there
  read_features(0, 0);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    mix_products(ct);
#pragma unroll
    for (int n = 0; n < 8; ++n) split_one(ct, n);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) issue_weight(0, nt);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  // the first weights are there, so that in the loop the compiler counts only what the loop requests
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(w[nt]));
  constexpr int kChunks = 2 * NT, kPairs = 8 * CT;
  // step kt: product of its 32 features, mixing of the 32 after them (the first half of a slice in odd steps); the last step
  // mixes what nobody reads
  int slot = 1;  // of three: the one of step kt + 1
  auto step = [&](int kt, auto odd) {
    constexpr bool kOdd = decltype(odd)::value;
    bf16x8 hi[QT], lo[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      hi[q] = __builtin_bit_cast(bf16x8, lds_m[m_read[q]]);
      lo[q] = __builtin_bit_cast(bf16x8, lds_m[mixed + m_read[q]]);
    }
    if (kShort) read_features(slot, 0);
    else read_features(((kt + 1) >> 1) & 1, !kOdd);
    asm volatile("s_barrier" ::: "memory");  // everybody has read: the mixed features may be replaced, and a slice's stage
#pragma unroll
    for (int n = 0; n < kChunks; ++n) {
      const int nt = n >> 1;
      if (n % (kChunks / CT) == 0) mix_products(n / (kChunks / CT));
#pragma unroll
      for (int q = 0; q < QT; ++q) acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nt], n & 1 ? lo[q] : hi[q], acc[q][nt], 0, 0, 0);
      // every weight fragment is requested for the next step right behind its last use, then the features
      if (n & 1) issue_weight(kt + 1, nt);
#pragma unroll
      for (int i = n * kPairs / kChunks; i < (n + 1) * kPairs / kChunks; ++i) split_one(i / 8, i % 8);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The mixed features are complete, and the next slice's features have landed, where the next step begins it: newer are,
    // with slices of 64, two steps' weights and the features just requested, with slices of 32 one step's weights and these.
    if (kShort) {
      issue_feats(kt + 3, slot ? slot - 1 : 2);  // where this step's were
      slot = slot == 2 ? 0 : slot + 1;
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NT + kLoads) : "memory");
    } else if (kOdd) {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
      issue_feats((kt >> 1) + 2, (kt >> 1) & 1);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * NT + kLoads) : "memory");
    }
  };
#pragma unroll 1
  for (int kt = 0; kt < steps; kt += kShort ? 1 : 2) {
    step(kt, std::false_type());
    if (!kShort) step(kt + 1, std::true_type());
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // lane (j16, kq) holds columns 16 nt + 4 kq .. + 3 of token j16
  if (!active || tok0 + j16 >= S) return;
  if (sums) {
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      float *dst = sums + (((size_t)blockIdx.z * S + tok0 + j16) * Q + q) * D + (h0 + hl) * kMpHeadDim + n0 + 4 * kq;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) *(f32x4 *)(dst + nt * 16) = acc[q][nt];
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    bf16_t *dst = pre + ((size_t)(tok0 + j16) * Q + q) * D + (h0 + hl) * kMpHeadDim + n0 + 4 * kq;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      *(u32x2 *)(dst + nt * 16) = (u32x2){(uint32_t)f32_to_bf16(acc[q][nt][0]) | ((uint32_t)f32_to_bf16(acc[q][nt][1]) << 16),
                                          (uint32_t)f32_to_bf16(acc[q][nt][2]) | ((uint32_t)f32_to_bf16(acc[q][nt][3]) << 16)};
    }
  }
}

}  // namespace

int32_t meta_rows_pad(int32_t H, int32_t Q) { return (H * Q + 15) / 16 * 16; }

hipError_t launch_meta_fold(int32_t Q, int32_t D, int32_t H, const void *f_q, const void *w_q, const void *w_k,
                            void *a_fold, float *qproj, hipStream_t s) {
  const int rows_pad = meta_rows_pad(H, Q);
  meta_qproj_kernel<<<(Q * D + kWaves - 1) / kWaves, kThreads, 0, s>>>(Q, D, (const bf16_t *)f_q, (const bf16_t *)w_q,
                                                                      qproj);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  bf16_t *a_hi = (bf16_t *)a_fold, *a_lo = a_hi + (size_t)rows_pad * D;
  const float scale = 1.f / sqrtf((float)(D / H));
  meta_fold_kernel<<<dim3((D + kThreads - 1) / kThreads, rows_pad), kThreads, 0, s>>>(Q, D, H, rows_pad, scale, qproj,
                                                                                      (const bf16_t *)w_k, a_hi, a_lo);
  return hipGetLastError();
}

// Workgroup columns of the score kernel: one workgroup per CU, as many as that leaves room for (with
// 512 wanted, 2048 tokens took 8 us more, 300 tokens 19 us more for the layer).  Beside the rearrangement of W_v up to 320
// tokens leave half of the CUs to that: with columns on all of them half of the scores came behind it (28 layers x 3584, the
// whole call, 96 tokens 79.2 -> 74.6 us, 128 83.4 -> 77.9, 192 97 -> 93; 400 tokens 173 -> 182).
constexpr int kPackWorkgroups = 128;
static void score_split(int32_t S, int32_t D, int *slices_per_wg, int *parts, bool packs = false) {
  const int slices = D / kSlice;
  const int groups = (S + kTokPerGroup - 1) / kTokPerGroup;
  int p = (packs && S <= 320 ? 256 - kPackWorkgroups : 256) / groups;
  if (p > slices) p = slices;
  if (p > kMaxParts) p = kMaxParts;
  if (p < 1) p = 1;
  *slices_per_wg = (slices + p - 1) / p;
  *parts = (slices + *slices_per_wg - 1) / *slices_per_wg;
}

size_t meta_attn_workspace_bytes(int32_t S, int32_t D, int32_t H, int32_t Q) {
  int spw, parts;
  score_split(S, D, &spw, &parts);
  return (size_t)parts * S * meta_rows_pad(H, Q) * kMaxL * sizeof(float);
}

// scores of all tokens to part, its workgroup columns in *parts; w_v rearranged into packed if given
static hipError_t launch_scores(int32_t S, int32_t L, int32_t D, int32_t rows_pad, const void *feats, const void *a_fold,
                                const void *w_v, void *packed, float *part, int *parts, hipStream_t s) {
  int spw;
  score_split(S, D, &spw, parts, packed != nullptr);
  hipError_t e = hipFuncSetAttribute((const void *)meta_scores_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kScoreLds);
  if (e != hipSuccess) return e;
  const int groups = (S + kTokPerGroup - 1) / kTokPerGroup, work = groups * *parts;
  const int pack_wgs = !packed ? 0 : std::max(kPackWorkgroups, 256 - work);
  meta_scores_kernel<<<pack_wgs + work, kScoreThreads, kScoreLds, s>>>(
      S, L, D, rows_pad / 16, spw, groups, pack_wgs, (const u32x4 *)w_v, (u32x4 *)packed, (const u32x4 *)feats,
      (const u32x4 *)a_fold, part);
  return hipGetLastError();
}

static ResidualLayers residuals(int32_t Q, const int32_t *residual_layers, const void *res_out) {
  ResidualLayers res = {};
  if (residual_layers && res_out) {
    res.on = 1;
    for (int q = 0; q < Q; ++q) res.layer[q] = residual_layers[q];
  }
  return res;
}

hipError_t launch_meta_attn(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, const void *feats, const void *v_proj,
                            const void *a_fold, const int32_t *residual_layers, void *pre, void *res_out,
                            float *part, hipStream_t s) {
  const int rows_pad = meta_rows_pad(H, Q);
  int parts;
  hipError_t e = launch_scores(S, L, D, rows_pad, feats, a_fold, nullptr, nullptr, part, &parts, s);
  if (e != hipSuccess) return e;
  meta_mix_kernel<<<dim3(S, (D / 8 + kMixThreads - 1) / kMixThreads), kMixThreads, 0, s>>>(
      S, L, D, H, Q, rows_pad, parts, part, (const u32x4 *)feats, (const u32x4 *)v_proj, residuals(Q, residual_layers, res_out),
      (u32x4 *)pre, (u32x4 *)res_out);
  return hipGetLastError();
}

bool meta_project_supports(int32_t D, int32_t H) { return D == H * kMpHeadDim; }

// the partial scores, then W_v in fragment order
static size_t meta_packed_offset(int32_t S, int32_t D, int32_t H, int32_t Q) {
  return (meta_attn_workspace_bytes(S, D, H, Q) + 255) / 256 * 256;
}
// behind them, where workgroups share D: the probabilities, and the sums of D's parts (as many as there may be)
static size_t meta_probs_bytes(int32_t S, int32_t H, int32_t Q) { return (size_t)S * H * Q * 128; }
static int project_most_shares(int32_t S, int32_t D, int32_t H, int32_t Q);
size_t meta_project_least_bytes(int32_t S, int32_t D, int32_t H, int32_t Q) {
  return meta_packed_offset(S, D, H, Q) + (size_t)D * D * sizeof(bf16_t);
}
size_t meta_project_workspace_bytes(int32_t S, int32_t D, int32_t H, int32_t Q) {
  const int most = project_most_shares(S, D, H, Q);
  const size_t shared = most > 1 ? meta_probs_bytes(S, H, Q) + (size_t)most * S * Q * D * sizeof(float) : 0;
  return meta_project_least_bytes(S, D, H, Q) + shared;
}

namespace {

template <int NT>
hipError_t launch_project(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, int hg, int parts, const void *feats,
                          const void *packed, const ResidualLayers &res, void *pre, void *res_out, const float *part,
                          hipStream_t s) {
  const size_t lds = ((size_t)2 * 2 * kMpWaves * 64 + 2 * (size_t)hg * 16 * 8) * sizeof(u32x4);  // two slices, mixed features
  auto kern = meta_project_kernel<NT>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  kern<<<dim3((S + 3) / 4, (H + hg - 1) / hg), kMpThreads, lds, s>>>(
      S, L, D, H, Q, hg, meta_rows_pad(H, Q), parts, part, (const u32x4 *)feats, (const u32x4 *)packed, res, (bf16_t *)pre,
      (u32x4 *)res_out);
  return hipGetLastError();
}

template <int QT, int NT, int FI>
hipError_t launch_project_wide(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, int hg, int parts, const void *feats,
                               const void *packed, const ResidualLayers &res, void *pre, void *res_out, const float *part,
                               int share, const void *probs, float *sums, hipStream_t s) {
  if (FI > mw_loads(L)) {
    if constexpr (FI > 6)
      return launch_project_wide<QT, NT, FI - 1>(S, L, D, H, Q, hg, parts, feats, packed, res, pre, res_out, part, share, probs, sums, s);
  }
  constexpr bool kShort = mw_short(QT, NT, FI);
  constexpr size_t kStages = (size_t)(kShort ? 3 : 2) * mw_stage(FI, kShort);
  constexpr int kMostRows = NT == 4 ? 4 * QT : 8 * QT < kMpHq ? 8 * QT : kMpHq;  // of project_plan
  static_assert((kStages + 2 * kMostRows * kMwTok * 4) * sizeof(u32x4) <= 160 * 1024, "more LDS than a CU has");
  if (hg * Q > kMostRows) return hipErrorInvalidValue;
  const size_t lds = (kStages + 2 * (size_t)hg * Q * kMwTok * 4) * sizeof(u32x4);
  auto kern = meta_project_wide_kernel<QT, NT, FI>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  kern<<<dim3((S + kMwTok - 1) / kMwTok, (H + hg - 1) / hg, (D / 64 + share - 1) / share), kMpThreads, lds, s>>>(
      S, L, D, H, Q, hg, meta_rows_pad(H, Q), parts, part, (const u32x4 *)feats, (const u32x4 *)packed, res, (bf16_t *)pre,
      (u32x4 *)res_out, share, (const u32x4 *)probs, sums);
  return hipGetLastError();
}

}  // namespace

// Which form, by the time a slice of 64 features takes (microseconds, fitted to 759 drawn calls of 16 to 2100 tokens, 8 to
// 32 heads, 12 to 32 layers, 1 to 4 queries): 4 tokens and 2 heads per workgroup where all workgroups run at once; 4 tokens
// and 4 heads by the workgroups, every one of which reads its heads' part of W_v; 16 tokens by rounds of 256 workgroups, by
// the queries and by the share of the CUs at work.  What it takes is 0.2 % slower in the mean than the fastest form of 981
// other calls, 10 % at most; one time a round, 3.0 for 4 heads and 5.0 for more, was 1.1 % and 36 % (480 tokens, 21 layers,
// 16 heads, 3 queries: 4 tokens a workgroup 78 us, 16 tokens 95; 1247, 15, 28, 1: 16 tokens and 7 heads 280, 4 heads 344).
struct ProjectPlan {
  int tg, nt, hg;
  int ds = 1;  // workgroups that share D
  double us = 0;  // what they are expected to take
};
static int split_heads(int H, int most) {  // heads per workgroup, evenly
  const int groups = (H + most - 1) / most;
  return (H + groups - 1) / groups;
}
// Workgroups that share D: where 16 tokens a workgroup occupy a part of the CUs only, each takes a share of D, the
// probabilities are made once in front of them and the float32 sums of the shares are added up behind them.
// us before and now (scores included): 28 layers x 3584, 28 heads, 3 queries 16 tokens 61 -> 44, 64 67 -> 59, 96 85 -> 75, 192 126 ->
// 93; 24 x 4096, 32 heads, 2 queries 64 tokens 74 -> 60, 256 158 -> 97; 16 x 2048, 16 heads, 1 query 400 tokens 67 -> 48.  Which
// form and how many shares: rounds of 256 workgroups, by times fitted to 480 measurements (30 shapes of 8 to 600 tokens, 2 to
// 14 shares; 3 % rms).  The forms below keep three queries of more than 320 tokens (400 tokens 175 and 178, 600 240 and 229),
// one or two of more than 640 of 4096 features or as many values of more (600 of 5120 255 and 240), and short D, where a share is hardly longer than its start (1024, 2 queries 416 tokens 30 and 36, 3 queries 210 24 and 31;
// 2048, 3 queries 96 38 and 42; but 1 query 20 tokens x 1024 22.3 and 20.6).  Of 70 drawn calls of 9 to 640 tokens those it takes
// are 1.35 times as fast.  Fewer than 10 tokens are left to values projected first (meta_project_pays), which also says from how many
// layers on it is worth it.
constexpr int kMostShares = 16;
static ProjectPlan shared_plan(int32_t S, int32_t D, int32_t H, int32_t Q) {
  ProjectPlan best = {0, 0, 0, 1};
  const int short_d = Q == 3 ? (S <= 48 ? 2048 : 3072) : Q == 2 ? 2048 : S <= 128 ? 1024 : 2048;
  if (S < 10 || Q > 3 || D < short_d || (int64_t)S * std::max(D, 4096) > (Q <= 2 ? 640 : 320) * 4096) return best;
  double best_us = 1e30;
  for (int nt : {4, 8}) {
    const int hg = split_heads(H, nt == 4 ? 4 : std::min(8, kMpHq / Q));
    const int64_t per = (int64_t)((S + 15) / 16) * ((H + hg - 1) / hg);
    for (int ds = 2; ds <= kMostShares && ds * 2 <= D / 64; ++ds) {
      const int share = (D / 64 + ds - 1) / ds, parts = (D / 64 + share - 1) / share;
      const double us = (double)((per * parts + 255) / 256) * (share * (nt == 4 ? 1.3 + 0.2 * Q : 1.6 + 0.5 * Q) + 6) + 2e-6 * parts * S * Q * D;
      if (us < best_us) {
        best_us = us;
        best = {16, nt, hg, parts, us};
      }
    }
  }
  return best;
}
static int project_most_shares(int32_t S, int32_t D, int32_t H, int32_t Q) { return shared_plan(S, D, H, Q).ds; }
static ProjectPlan project_plan(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, bool may_share) {
  const ProjectPlan shared = may_share ? shared_plan(S, D, H, Q) : ProjectPlan{0, 0, 0, 1};
  const int64_t g4 = (S + 3) / 4, g16 = (S + 15) / 16;
  auto groups = [&](int hg) { return (int64_t)(H + hg - 1) / hg; };
  if (g4 * groups(2) <= 256) return shared.ds > 1 ? shared : ProjectPlan{4, 2, split_heads(H, 2)};
  const int wide = split_heads(H, std::min(8, kMpHq / Q)), narrow = split_heads(H, 4);
  const double layers = L > 24 ? 1.0 + 0.0044 * (L - 24) : 1.0;  // more features to load
  auto rounds_us = [&](int hg, double round, double share) {
    const int64_t wgs = g16 * groups(hg);
    return layers * ((double)((wgs + 255) / 256) * round + share * (double)wgs / 256);
  };
  const double four_us = 0.6 + 0.81 * (double)(g4 * groups(narrow)) / 256, narrow_us = rounds_us(narrow, 1.87 + 0.06 * Q, 0.34);
  static const double kWide[4] = {0, 2.15, 2.7, 3.09};
  // four queries: accumulators for 4 heads only
  const double wide_us = Q <= 3 ? rounds_us(wide, kWide[Q] + (L < 24 ? 0.02 * (24 - L) : 0.0), 0.47) : 1e30;
  // The probabilities and the sum of the shares are 8 us of launches on top.  Where a form below has a round that just fits, its
  // whole rows are ahead (24 layers x 3584, 2 queries, 540 tokens 154 us and by shares 178, 500 tokens 152 and 132; of 1156 calls 0.1 %
  // slower than the faster in the mean).
  if (shared.ds > 1 && shared.us + 8 < std::min(std::min(wide_us, narrow_us), four_us) * (D / 64)) return shared;
  if (wide_us < narrow_us && wide_us < four_us) return {16, 8, wide};
  return narrow_us < four_us ? ProjectPlan{16, 4, narrow} : ProjectPlan{4, 4, narrow};
}

// Against values projected first: L rows per token through the product (0.85 PFLOP/s, 20 us at least) and the mixing of the
// projected values (2.6 TB/s, 5 us at least), which round the values to bf16 on the way.  The line is where slices of 0.65 to
// 1 us with 4 tokens, 3.0 with 16 tokens and 4 heads and 5.0 with more heads, longer than they take, put it: what it sends
// this way is 1.5 to 3 % slower in the mean of 1100 drawn calls than the faster of both orders (28 layers, 3 queries, D =
// 3584, up to fc1: 16 tokens 92 us values first and 95 this way, 48 tokens 117 and 103, 2048 tokens 2082 and 860), and lines
// closer to it would round the values of calls that have none rounded.
//
// Where workgroups share D, this way is also taken where it is expected to be ahead: the product of the S L rows (up to 128 of them
// few rows' tiles, beyond them the 256-row tiles' one round at least) and the mixing against the shares, the rearrangement of W_v
// and the two launches around them, fitted to 800 calls of 10 to 700 tokens and 1 to 32 layers.  The fewer layers, the more tokens
// it takes and the wider D may not be (3584, 3 queries, without the products behind, us, values first and this way: 16 tokens of 3 layers 28 and 38, of
// 12 47 and 39, of 28 51 and 41; 128 tokens 52 and 67, 71 and 69, 114 and 76; 320 tokens 69 and 116, 125 and 119, 236 and 133).  Of 844 calls what
// it chooses is 0.7 % slower than the faster in the mean, shares wherever they may be had were 14 %.
bool meta_project_pays(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q) {
  if (!meta_project_supports(D, H)) return false;
  const ProjectPlan shared = shared_plan(S, D, H, Q);
  if (shared.ds > 1) {
    const double k = D / 1e3, kk = k * k, rows = (double)S * L;
    const double rows_us = rows <= 128 ? (0.99 + 0.0058 * rows) * kk - 8.1 : std::max(15.5 * k - 0.85 * kk - 20.2, 0.0016 * rows * kk);
    if (0.71 * shared.us + 1.34 * kk + 0.0044 * S * k - 10.7 < rows_us + 0.00143 * S * Q * k) return true;
  }
  const double product = 2.0 * S * L * D * (double)D / 0.85e9, mixing = 2.0 * S * L * (double)D / 2.6e6;
  const double first = (product < 20 ? 20 : product) + (mixing < 5 ? 5 : mixing);
  const int64_t g4 = (S + 3) / 4, g16 = (S + 15) / 16;
  auto groups = [&](int most) { return (int64_t)(H + split_heads(H, most) - 1) / split_heads(H, most); };
  double slice_us = 0.65;
  if (g4 * ((H + 1) / 2) > 256) {
    slice_us = std::max(1.0, (double)(g4 * H) * kMpHeadDim * 128 / 9.2e6);
    slice_us = std::min(slice_us, 3.0 * (double)((g16 * groups(4) + 255) / 256));
    if (Q <= 3) slice_us = std::min(slice_us, 5.0 * (double)((g16 * groups(std::min(8, kMpHq / Q)) + 255) / 256));
  }
  return 5 + slice_us * (D / 64) < first;
}

hipError_t launch_meta_attn_project(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, const void *feats,
                                    const void *a_fold, const void *w_v, const int32_t *residual_layers, void *pre,
                                    void *res_out, float *part, size_t part_bytes, hipStream_t s) {
  int parts;
  void *packed = (char *)part + meta_packed_offset(S, D, H, Q);
  hipError_t e = launch_scores(S, L, D, meta_rows_pad(H, Q), feats, a_fold, w_v, packed, part, &parts, s);
  if (e != hipSuccess) return e;
  const ResidualLayers res = residuals(Q, residual_layers, res_out);
  // a workspace that was enough before workgroups shared D (sized for more tokens, say) takes the forms that don't
  const ProjectPlan plan = project_plan(S, L, D, H, Q, part_bytes >= meta_project_workspace_bytes(S, D, H, Q));
  if (plan.tg == 4)
    return plan.nt == 2 ? launch_project<2>(S, L, D, H, Q, plan.hg, parts, feats, packed, res, pre, res_out, part, s)
                        : launch_project<4>(S, L, D, H, Q, plan.hg, parts, feats, packed, res, pre, res_out, part, s);
  const int share = plan.ds > 1 ? (D / 64 + plan.ds - 1) / plan.ds : D / 64, shares = (D / 64 + share - 1) / share;
  char *more = (char *)packed + (size_t)D * D * sizeof(bf16_t);
  void *probs = plan.ds > 1 ? more : nullptr;
  float *sums = plan.ds > 1 ? (float *)(more + meta_probs_bytes(S, H, Q)) : nullptr;
  if (probs) {
    meta_softmax_kernel<<<S, kSoftmaxThreads, 0, s>>>(S, L, H * Q, meta_rows_pad(H, Q), parts, (const f32x4 *)part, (uint32_t *)probs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  auto project = [&] {
#define HB_MP(QT_, NT_) return launch_project_wide<QT_, NT_, 8>(S, L, D, H, Q, plan.hg, parts, feats, packed, res, pre, res_out, part, share, probs, sums, s)
  if (plan.nt == 4) {
    switch (Q) {
      case 1: HB_MP(1, 4);
      case 2: HB_MP(2, 4);
      case 3: HB_MP(3, 4);
      default: HB_MP(4, 4);
    }
  }
  switch (Q) {
    case 1: HB_MP(1, 8);
    case 2: HB_MP(2, 8);
    default: HB_MP(3, 8);
  }
#undef HB_MP
  };
  if ((e = project()) != hipSuccess || !sums) return e;
  const size_t n4 = (size_t)S * Q * D / 4;
  meta_sum_kernel<<<(unsigned)((n4 + 255) / 256), 256, 0, s>>>(S, L, D, Q, shares, (const f32x4 *)sums, (const uint2 *)feats, res,
                                                               (uint2 *)pre, (uint2 *)res_out);
  return hipGetLastError();
}

}  // namespace hb
