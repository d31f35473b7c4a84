// The target's projections around the tree-verify attention, on the bf16 matrix cores:
//   * fused query/key/value projection + bias + rotary embedding, written straight into the
//     layouts hb_tree_verify_attn reads (q [T, Hq, D], k_tree / v_tree [T, Hkv, D]);
//   * output projection (a plain  out = x W^T (+ residual)  in bf16 with fp32 accumulation);
//   * the gated-SiLU half of the feed-forward block, out = silu(x Wg^T) * (x Wu^T), gate and up
//     projection in one pass (the down projection is the plain one with the residual);
//   * root-mean-square normalisation of the rows;
//   * the two small kernels that give every tree node its position (prefix length + depth) and
//     the cosine / sine table of those positions.
// The matrix work is the tile loop of the LM head (mfma_gemm_tile.inc: C^T = W H^T, weight rows
// as the MFMA "A" operand, so a lane's accumulators of a 16x16 tile are four output features of ONE
// token).  For the rotary embedding the 256 weight rows of a tile are not taken in memory order:
// a tile holds two heads, and the rows are arranged so that the two accumulators a lane holds at
// the same position of its two 32-row halves are the pair (d, d + 64) of one head, which is
// what the rotate-half convention rotates together: the rotation costs no exchange at all.  The
// gated projection uses the same device: a tile holds 128 features, the gate rows in the first
// 32-row sub-tile of every wavefront row and the matching up rows in the second, so silu(gate) * up
// is one lane's own two accumulators.
#include "mfma_gemm_tile.h"

#include <cmath>

namespace hb {

namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kHeadDim = 128;
constexpr int64_t kUncached = (int64_t)1 << 27;  // weights: 256 MB, the size of the last-level cache

// Workgroup ids go round-robin to the XCDs.  Of the units 0 .. units - 1, numbered so that neighbours share a
// weight tile, every XCD gets one run of equal length: neighbours find the shared tile in its L2, and no XCD
// gets more units than its 32 CUs hold while others idle (18 weight tiles x 11 hidden tiles, whole weight tiles
// dealt: 33 units on two of them, 2048 tokens x 3584 x 4608 113 us; so 67).
__device__ inline int deal_unit(int units) {
  const int per = (units + kXcds - 1) / kXcds, slot = (int)blockIdx.x / kXcds;
  const int unit = (int)blockIdx.x % kXcds * per + slot;
  return slot < per && unit < units ? unit : -1;
}
inline unsigned deal_grid(long units) { return (unsigned)((units + kXcds - 1) / kXcds * kXcds); }

struct QkvArgs {
  const bf16_t *bias;      // [(Hq + 2 Hkv) * 128] or null
  const float *cos, *sin;  // [M, 64]
  bf16_t *q, *k, *v;       // [M, Hq, 128], [M, Hkv, 128], [M, Hkv, 128]
  int Hq, Hkv;
};
struct StoreArgs {
  const bf16_t *residual;  // [M, N] or null
  bf16_t *out;             // [M, N]
  const bf16_t *hidden2, *weight2;  // of K's second half (proj_pair.hip and proj_few.hip), or null
};
struct NormArgs {  // of the rows that a plain projection gives; weight null: none
  const bf16_t *weight;  // [N]
  bf16_t *out;           // [M, N]
  float eps;
};
// A row of these is normalised in the launch that sums the parts of K: a workgroup per token, eight values a thread.  Of
// more than 128 tokens a short row leaves the workgroup's threads idle, and one just longer than the workgroup asks for a
// second round trip for a few values; two launches are ahead there (us, two launches and one: 619 x 17600 x 232 25.8 and
// 32.9, 536 x 12544 x 512 27.4 and 29.7, 528 x 4992 x 4136 43.6 and 45.0; on the other side
// 300 x 3584 x 1100 4 %, x 4000 5 %, x 6500 1.5 % for one; 500 calls).
inline bool norm_fits(const NormArgs &n, int M, int N) {
  if (!n.weight || N % 8 || N > 8192) return false;
  return M <= 128 || (N >= 1024 && !(M > 256 && N > 4096 && N < 5120));
}

// ROPE: query/key/value projection with rotary embedding (V = (Hq + 2 Hkv) * 128 weight rows),
// else plain projection.  One workgroup per (weight tile, hidden tile), dealt by deal_unit.
// WNT: the weight loads carry the non-temporal hint.  It pays where one hidden tile means that nobody shares
// them and they exceed the last-level cache (gated 3584 x 37888, 272 MB: 192 tokens 77.5 -> 73.6 us, 256 85.9 -> 82.6;
// 4096 x 34816 at 160 84.3 -> 80.0; 5120 x 27648 and 8192 x 20480 82 and 104 both).  Weights that the cache holds lose
// (4096 x 28672, 235 MB, read again and again: 40 -> 62; 512 x 2048 9.7 -> 11.8).
template <int MT, bool ROPE, bool GLU, bool WNT>
__global__ __launch_bounds__(512) void proj_mfma_kernel(int M, int K, int V, int m_tiles, int v_tiles,
                                                        const u32x4 *__restrict__ hidden,
                                                        const u32x4 *__restrict__ weight, QkvArgs qa, StoreArgs sa) {
  constexpr int TM = 64 * MT;
  extern __shared__ u32x4 lds[];
  u32x4 *lw = lds;
  u32x4 *lh = lds + 3 * TV * CH;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wv = wave >> 1;
  const int wm = wave & 1;
  const int unit = deal_unit(v_tiles * m_tiles);
  if (unit < 0) return;
  const int v_tile = unit / m_tiles, m_tile = unit % m_tiles;
  const int m0 = m_tile * TM;
  const int v0 = v_tile * TV;
  const int kp = K / 8;

  // Tile row t (wavefront row wv = t / 64, sub-tile i = (t % 64) / 32, rr = t % 32) holds, for the
  // rotary variant, feature  (wv / 2) * 128 + (wv % 2) * 32 + 64 i + rr  of the tile's two heads.
  // ... and for the gated projection (V = 2 F weight rows: F gate rows, then F up rows) feature
  // v0 / 2 + 32 wv + rr of the gate (i = 0) or of the up projection (i = 1).
#define HB_GEMM_W_ROW(t_) (ROPE ? v0 + (((t_) >> 7) << 7) + ((((t_) >> 6) & 1) << 5) + ((((t_) >> 5) & 1) << 6) + ((t_) & 31) \
                           : GLU ? (((t_) >> 5) & 1) * (V >> 1) + (v0 >> 1) + (((t_) >> 6) << 5) + ((t_) & 31)                  \
                                 : v0 + (t_))
#include "mfma_gemm_tile.inc"
#undef HB_GEMM_W_ROW

  // Epilogue.  Accumulator e of lane l in tile (i, j): tile row wv*64 + i*16 + 4 (l / 16) + e,
  // token m0 + wm*32*MT + j*16 + l % 16.
#pragma unroll
  for (int j = 0; j < JT; ++j) {
    const int m = m0 + wm * 32 * MT + j * 16 + frag_row;
    if (m >= M) continue;
    if (ROPE) {
      const int head = (v0 >> 7) + (wv >> 1);
      if (head >= qa.Hq + 2 * qa.Hkv) continue;  // second half of the last tile when the heads are odd in number
      const bool rotate = head < qa.Hq + qa.Hkv;
      bf16_t *dst = head < qa.Hq ? qa.q + ((size_t)m * qa.Hq + head) * kHeadDim
                    : head < qa.Hq + qa.Hkv ? qa.k + ((size_t)m * qa.Hkv + (head - qa.Hq)) * kHeadDim
                                            : qa.v + ((size_t)m * qa.Hkv + (head - qa.Hq - qa.Hkv)) * kHeadDim;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int d = (wv & 1) * 32 + i * 16 + 4 * frag_k;  // d .. d + 3 and d + 64 .. d + 67
        f32x4 x1 = acc[i][j], x2 = acc[i + 2][j];
        if (qa.bias) {
          const u32x2 b1 = *(const u32x2 *)(qa.bias + head * kHeadDim + d);
          const u32x2 b2 = *(const u32x2 *)(qa.bias + head * kHeadDim + d + 64);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x1[e] += __uint_as_float((e & 1) ? (b1[e >> 1] & 0xffff0000u) : (b1[e >> 1] << 16));
            x2[e] += __uint_as_float((e & 1) ? (b2[e >> 1] & 0xffff0000u) : (b2[e >> 1] << 16));
          }
        }
        if (rotate) {
          const f32x4 cs = *(const f32x4 *)(qa.cos + (size_t)m * 64 + d);
          const f32x4 sn = *(const f32x4 *)(qa.sin + (size_t)m * 64 + d);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float a1 = x1[e] * cs[e] - x2[e] * sn[e];
            const float a2 = x2[e] * cs[e] + x1[e] * sn[e];
            x1[e] = a1;
            x2[e] = a2;
          }
        }
        *(u32x2 *)(dst + d) = (u32x2){pack_bf16(x1[0], x1[1]), pack_bf16(x1[2], x1[3])};
        *(u32x2 *)(dst + d + 64) = (u32x2){pack_bf16(x2[0], x2[1]), pack_bf16(x2[2], x2[3])};
      }
    } else if (GLU) {
      const int F = V >> 1;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int f = (v0 >> 1) + wv * 32 + i * 16 + 4 * frag_k;  // f .. f + 3, F % 4 == 0
        if (f >= F) continue;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[i][j][e];
          y[e] = g / (1.f + __expf(-g)) * acc[i + 2][j][e];
        }
        *(u32x2 *)(sa.out + (size_t)m * F + f) = (u32x2){pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = v0 + wv * 64 + i * 16 + 4 * frag_k;  // n .. n + 3, V % 4 == 0
        if (n >= V) continue;
        f32x4 x = acc[i][j];
        if (sa.residual) {
          const u32x2 r = *(const u32x2 *)(sa.residual + (size_t)m * V + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] += __uint_as_float((e & 1) ? (r[e >> 1] & 0xffff0000u) : (r[e >> 1] << 16));
        }
        *(u32x2 *)(sa.out + (size_t)m * V + n) = (u32x2){pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
      }
    }
  }
}

template <int MT, bool ROPE, bool GLU>
hipError_t launch(int M, int K, int V, const void *hidden, const void *weight, const QkvArgs &qa, const StoreArgs &sa,
                  hipStream_t s) {
  constexpr int TM = 64 * MT;
  const int m_tiles = (M + TM - 1) / TM;
  const int v_tiles = (V + TV - 1) / TV;
  const size_t lds_bytes = tile_lds_bytes(MT);
  auto kern = proj_mfma_kernel<MT, ROPE, GLU, false>;
  if constexpr (GLU)
    if (m_tiles == 1 && (int64_t)K * V >= kUncached) kern = proj_mfma_kernel<MT, ROPE, GLU, true>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  kern<<<deal_grid((long)v_tiles * m_tiles), 512, lds_bytes, s>>>(M, K, V, m_tiles, v_tiles, (const u32x4 *)hidden, (const u32x4 *)weight, qa, sa);
  return hipGetLastError();
}

// ---- few tokens: split K ---------------------------------------------------------------------
// With few tokens a projection is a stream of its weight matrix from HBM, and one workgroup per
// 256-row weight tile and hidden tile would give work to a few dozen CUs only.  Here the K range
// of every tile is cut into `ks` parts, one workgroup per (weight tile, K part, hidden tile); the
// workgroups that differ in the hidden tile only, which read the same weights, get neighbouring
// slots of one XCD.  A workgroup runs the same tile loop over its part and stores its fp32
// accumulators to the caller's workspace as part[kpart][token][weight row] (a lane holds four
// consecutive weight rows of one token).  proj_reduce_kernel then sums the parts in order and
// applies the epilogue (bias, rotary embedding, residual).
template <int MT>
__global__ __launch_bounds__(512) void proj_splitk_kernel(int M, int Kfull, int V, int ks, int v_pad, int m_tiles,
                                                          int m_pad, int units,
                                                          const u32x4 *__restrict__ hidden_full,
                                                          const u32x4 *__restrict__ weight_full,
                                                          float *__restrict__ part) {
  constexpr bool WNT = false;  // measured: the non-temporal hint costs 10-25 % here, also with a single hidden tile
  constexpr int TM = 64 * MT;
  extern __shared__ u32x4 lds[];
  u32x4 *lw = lds;
  u32x4 *lh = lds + 3 * TV * CH;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wv = wave >> 1;
  const int wm = wave & 1;
  const int index = deal_unit(units * m_tiles);
  if (index < 0) return;
  const int unit = index / m_tiles;  // (weight tile, K part)
  const int v_tile = unit / ks, kpart = unit % ks;
  const int m0 = (index % m_tiles) * TM;
  const int v0 = v_tile * TV;
  const int K = Kfull / ks;          // this workgroup's share
  const int kp = Kfull / 8;          // row stride in 16-byte pieces
  const u32x4 *hidden = hidden_full + (size_t)kpart * (K / 8);
  const u32x4 *weight = weight_full + (size_t)kpart * (K / 8);
#define HB_GEMM_W_ROW(t_) (v0 + (t_))
#include "mfma_gemm_tile.inc"
#undef HB_GEMM_W_ROW
  float *dst = part + ((size_t)kpart * m_pad + m0) * v_pad + v0;
#pragma unroll
  for (int j = 0; j < JT; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wv * 64 + i * 16 + 4 * frag_k, token = wm * 32 * MT + j * 16 + frag_row;
      *(f32x4 *)(dst + (size_t)token * v_pad + row) = acc[i][j];
    }
}

// The sum over the K parts, in order, of four consecutive weight rows of one token; eight loads in flight.
__device__ inline f32x4 sum_parts(const float *__restrict__ src, int ks, size_t stride) {
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < ks; k0 += 8) {
    f32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = *(const f32x4 *)(src + (size_t)(k0 + i < ks ? k0 + i : ks - 1) * stride);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (k0 + i < ks) x += v[i];
  }
  return x;
}

// One thread per token and group of four features (rotary variant: four (d, d + 64) pairs), groups
// in neighbouring lanes: partials and results move in whole lines.
template <bool ROPE, bool GLU>
__global__ __launch_bounds__(256) void proj_reduce_kernel(int M, int V, int ks, int v_pad, int m_pad, int groups,
                                                          const float *__restrict__ part, QkvArgs qa, StoreArgs sa) {
  const int g = (int)blockIdx.x * 256 + (int)threadIdx.x, m = (int)blockIdx.y;
  if (g >= groups) return;
  const size_t stride = (size_t)m_pad * v_pad;
  const float *row = part + (size_t)m * v_pad;
  if (ROPE) {
    const int head = g >> 4, d = (g & 15) * 4;
    f32x4 x1 = sum_parts(row + head * kHeadDim + d, ks, stride);
    f32x4 x2 = sum_parts(row + head * kHeadDim + 64 + d, ks, stride);
    if (qa.bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x1[e] += bf16_to_f32(qa.bias[head * kHeadDim + d + e]);
        x2[e] += bf16_to_f32(qa.bias[head * kHeadDim + 64 + d + e]);
      }
    }
    const bool rotate = head < qa.Hq + qa.Hkv;
    bf16_t *dst = head < qa.Hq ? qa.q + ((size_t)m * qa.Hq + head) * kHeadDim
                  : head < qa.Hq + qa.Hkv ? qa.k + ((size_t)m * qa.Hkv + (head - qa.Hq)) * kHeadDim
                                          : qa.v + ((size_t)m * qa.Hkv + (head - qa.Hq - qa.Hkv)) * kHeadDim;
    if (rotate) {
      const f32x4 cs = *(const f32x4 *)(qa.cos + (size_t)m * 64 + d);
      const f32x4 sn = *(const f32x4 *)(qa.sin + (size_t)m * 64 + d);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = x1[e] * cs[e] - x2[e] * sn[e];
        const float b = x2[e] * cs[e] + x1[e] * sn[e];
        x1[e] = a;
        x2[e] = b;
      }
    }
    *(u32x2 *)(dst + d) = (u32x2){pack_bf16(x1[0], x1[1]), pack_bf16(x1[2], x1[3])};
    *(u32x2 *)(dst + d + 64) = (u32x2){pack_bf16(x2[0], x2[1]), pack_bf16(x2[2], x2[3])};
  } else if (GLU) {
    const int F = V >> 1, f = g * 4;
    const f32x4 xg = sum_parts(row + f, ks, stride), xu = sum_parts(row + F + f, ks, stride);
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = xg[e] / (1.f + __expf(-xg[e])) * xu[e];
    *(u32x2 *)(sa.out + (size_t)m * F + f) = (u32x2){pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
  } else {
    const int n = g * 4;
    f32x4 x = sum_parts(row + n, ks, stride);
    if (sa.residual) {
      const u32x2 r = *(const u32x2 *)(sa.residual + (size_t)m * V + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] += __uint_as_float((e & 1) ? (r[e >> 1] & 0xffff0000u) : (r[e >> 1] << 16));
    }
    *(u32x2 *)(sa.out + (size_t)m * V + n) = (u32x2){pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
  }
}

// The scale of a row of K values; ss: this thread's sum of squares, WAVES wavefronts to a row.
template <int WAVES>
__device__ __forceinline__ float rms_scale(float ss, int K, float eps, float (&red)[WAVES]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float all = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
  for (int w = 4; w < WAVES; w += 4) all += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
  return rsqrtf(all / (float)K + eps);
}
__device__ __forceinline__ float sum_squares(u32x4 v, float ss) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a = __uint_as_float(v[e] << 16), b = __uint_as_float(v[e] & 0xffff0000u);
    ss += a * a + b * b;
  }
  return ss;
}
__device__ __forceinline__ u32x4 rms_piece(u32x4 v, u32x4 w, float scale) {
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a = __uint_as_float(v[e] << 16) * scale * __uint_as_float(w[e] << 16);
    const float b = __uint_as_float(v[e] & 0xffff0000u) * scale * __uint_as_float(w[e] & 0xffff0000u);
    o[e] = pack_bf16(a, b);
  }
  return o;
}
constexpr int kKeep = 4;  // 16-byte pieces of a row that a thread keeps: 4 * 256 * 8 = 8192 values

// out[t, :] = x[t, :] / sqrt(mean(x[t, :]^2) + eps) * weight: one workgroup per row, the row is
// read once (16-byte loads, K % 8 == 0) and kept in registers between the two passes when it
// fits (K <= 8192), otherwise read again; its weights are requested with it (8 x 3584 3.6 -> 3.4 us)
__global__ __launch_bounds__(256) void rmsnorm_kernel(int K, const bf16_t *__restrict__ x,
                                                      const bf16_t *__restrict__ weight, float eps,
                                                      bf16_t *__restrict__ out) {
  __shared__ float red[4];
  const int t = blockIdx.x, tid = threadIdx.x;
  const int pieces = K / 8;
  const u32x4 *row = (const u32x4 *)(x + (size_t)t * K);
  const u32x4 *wv = (const u32x4 *)weight;
  u32x4 *dst = (u32x4 *)(out + (size_t)t * K);
  u32x4 keep[kKeep], gain[kKeep];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kKeep; ++i) {
    const int p = tid + i * 256;
    keep[i] = row[p < pieces ? p : pieces - 1];
  }
#pragma unroll
  for (int i = 0; i < kKeep; ++i) {
    const int p = tid + i * 256;
    gain[i] = wv[p < pieces ? p : pieces - 1];
  }
#pragma unroll
  for (int i = 0; i < kKeep; ++i)
    if (tid + i * 256 < pieces) ss = sum_squares(keep[i], ss);
  for (int p = tid + kKeep * 256; p < pieces; p += 256) ss = sum_squares(row[p], ss);
  const float scale = rms_scale(ss, K, eps, red);
#pragma unroll
  for (int i = 0; i < kKeep; ++i)
    if (tid + i * 256 < pieces) dst[tid + i * 256] = rms_piece(keep[i], gain[i], scale);
  for (int p = tid + kKeep * 256; p < pieces; p += 256) dst[p] = rms_piece(row[p], wv[p], scale);
}

// The sum over the K parts with the residual, and the row's root-mean-square normalisation, in one launch: a workgroup per
// token, which rounds as proj_reduce_kernel does and normalises what it rounded.  512 threads: a row of 3584 is one piece a
// thread, and the loads of its parts are one round trip (with 256 the launch saved was lost again: eight layers of 16 chains
// 1578 us by two launches, 1575, and 1564 with 512).  128 tokens: 3584 x 3584 19.7 -> 18.0 us, 18944 x 3584 41.5 -> 40.2, and with
// residual and weights requested in front of the parts 17.4 and 40.0.
constexpr int kNormThreads = 512;
__global__ __launch_bounds__(kNormThreads) void proj_reduce_norm_kernel(int V, int ks, int v_pad, int m_pad, const float *__restrict__ part,
                                                               StoreArgs sa, NormArgs norm) {
  __shared__ float red[kNormThreads / 64];
  const int m = blockIdx.x, tid = threadIdx.x, pieces = V / 8;
  const size_t stride = (size_t)m_pad * v_pad;
  const float *row = part + (size_t)m * v_pad;
  const u32x4 *res = (const u32x4 *)(sa.residual ? sa.residual + (size_t)m * V : nullptr);
  constexpr int kMine = 8192 / 8 / kNormThreads;
  const u32x4 *w = (const u32x4 *)norm.weight;
  u32x4 keep[kMine], gain[kMine];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kMine; ++i) {
    if (i * kNormThreads >= pieces) break;
    const int p = min(tid + i * kNormThreads, pieces - 1);
    gain[i] = w[p];
    const u32x4 r = res ? res[p] : (u32x4){0u, 0u, 0u, 0u};
    f32x4 x = sum_parts(row + p * 8, ks, stride), y = sum_parts(row + p * 8 + 4, ks, stride);
    if (res) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] += __uint_as_float((e & 1) ? (r[e >> 1] & 0xffff0000u) : (r[e >> 1] << 16));
        y[e] += __uint_as_float((e & 1) ? (r[2 + (e >> 1)] & 0xffff0000u) : (r[2 + (e >> 1)] << 16));
      }
    }
    keep[i] = (u32x4){pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
    if (tid + i * kNormThreads < pieces) {
      ((u32x4 *)(sa.out + (size_t)m * V))[p] = keep[i];
      ss = sum_squares(keep[i], ss);
    }
  }
  const float scale = rms_scale(ss, V, norm.eps, red);
  u32x4 *dst = (u32x4 *)(norm.out + (size_t)m * V);
#pragma unroll
  for (int i = 0; i < kMine; ++i)
    if (tid + i * kNormThreads < pieces) dst[tid + i * kNormThreads] = rms_piece(keep[i], gain[i], scale);
}

// Hidden tile height (64 mt rows) of the unsplit kernel: rounds of 256 workgroups, one per CU, times
// a workgroup's clocks, read inside the kernel: 3800 until the first tile is there, a K step, the results.
int plain_tile_height(int M, int K, int v_tiles) {
  static const double kStep[5] = {0, 1500, 1750, 2130, 2560}, kStore[5] = {0, 3800, 8200, 12700, 17000};
  int mt = 1;
  double best = 1e30;
  for (int t = 1; t <= 4; ++t) {
    const long units = (long)v_tiles * ((M + 64 * t - 1) / (64 * t));
    const double cost = (double)((units + 255) / 256) * (3800 + (K / BK) * kStep[t] + kStore[t]);
    if (cost < best) { best = cost; mt = t; }
  }
  return mt;
}

// The split over K: hidden tile height (64 mt rows) and K parts (a divisor of the K steps, at
// least kMinSteps steps per part, all workgroups resident at once), by a cost model (microseconds, weights too
// many to stay in the last-level cache):
//   split:  6 + steps / ks * (0.70 | 0.86 | 1.15 | 1.45 for mt = 1 .. 4) + partial bytes written and read / 4 TB/s
//   plain:  3 + steps * 0.75 per round of 256 workgroups of 64 tokens, whatever height the unsplit kernel takes (at most
//           512 tokens)
//           3 + steps * (0.72 | 0.95 | 1.15 | 1.4 for the unsplit kernel's mt) per round (more tokens)
// Up to 512 tokens the tile is 64 or 128 rows high; from there to kSplitMaxM tokens 128 to 256 rows,
// and the split must win by 10 % (it does for long K: 960 x 18944 -> 3584 takes 124 us in 4 parts of 256-row tiles, 196
// unsplit; with K = 3584 the unsplit kernel stays).  ks = 1 means: do not split.
// The constants were fitted to a slower tile loop: the split now takes 7 % less than they say in the mean (960 x 18944 ->
// 3584 143 expected), and gated 240 x 3584 -> 37888 unsplit 83 where they say 129.  What they choose holds: of 89 calls of
// 129 to 1024 tokens that are split the unsplit kernel takes more than 2 % less in one (640 x 2048 -> 2048, 19.4 against 20.5).
constexpr int kSplitMaxM = 1024;
constexpr int kMinSteps = 4;
struct SplitPlan {
  int ks, mt;
};
SplitPlan split_plan(int M, int K, int V) {
  SplitPlan best = {1, 1};
  if (M > kSplitMaxM || K % BK) return best;
  const int steps = K / BK, v_tiles = (V + TV - 1) / TV;
  const bool few = M <= 512;
  static const double kStepSplit[5] = {0, 0.70, 0.86, 1.15, 1.45}, kStepPlain[5] = {0, 0.72, 0.95, 1.15, 1.4};
  double best_cost;
  if (few) {
    const long plain_units = (long)v_tiles * ((M + 63) / 64);
    best_cost = 3.0 + steps * 0.75 * (double)((plain_units + 255) / 256);
  } else {
    const int pm = plain_tile_height(M, K, v_tiles);
    const long plain_units = (long)v_tiles * ((M + 64 * pm - 1) / (64 * pm));
    best_cost = 0.9 * (3.0 + steps * kStepPlain[pm] * (double)((plain_units + 255) / 256));
  }
  for (int mt = few ? 1 : 2; mt <= (few ? 2 : 4); ++mt) {
    const int m_tiles = (M + 64 * mt - 1) / (64 * mt);
    for (int d = 2; d <= steps; ++d) {
      if (steps % d || steps / d < kMinSteps || (long)v_tiles * m_tiles * d > 256) continue;
      const double bytes = 8.0 * d * v_tiles * TV * m_tiles * 64 * mt;
      const double cost = 6.0 + (double)(steps / d) * kStepSplit[mt] + bytes / 4e6;
      if (cost < best_cost - 1e-9) {
        best_cost = cost;
        best = {d, mt};
      }
    }
  }
  return best;
}

size_t split_bytes(SplitPlan plan, int M, int V) {
  if (plan.ks <= 1) return 0;
  const size_t v_pad = (size_t)((V + TV - 1) / TV) * TV;
  const size_t tm = 64 * plan.mt, m_pad = (M + tm - 1) / tm * tm;
  return (size_t)plan.ks * v_pad * m_pad * sizeof(float);
}

constexpr int kFewLeast = 17, kFewMost = 128;  // tokens
inline int few_m_pad(int M) { return M <= 64 ? 64 : 128; }

// 17 to 128 tokens: rows of a tile and parts of K of proj_few.hip, one round of workgroups (rows = 0: there is
// no such division).  Microseconds fitted to 250 measurements (18 shapes of 2048 to 18944 x 2048 to 37888, 40 to
// 128 tokens, weights too many to stay in the last-level cache; 7 % rms), a K step's part by the rows and by the
// share of the CUs at work.  What it takes is within 1 % of the fastest of them in the mean, and 19 % faster
// than the split into 256-row tiles (128 tokens, split and reduction against this: 3584 x 3584 18.4 -> 16.2,
// 18944 x 3584 49 -> 40, 2048 x 2048 13.7 -> 8.8; gated 3584 x 37888 73.5 -> 58.9, 4096 x 24576 62 -> 51).
// Gated weights are not split (tiles of pairs, and never few); 16-row tiles only where K is whole.
// workspace: the bytes that a caller was told to bring, for split_plan.
FewPlan few_plan(int M, int K, int V, StreamKind kind, size_t workspace) {
  FewPlan best = {0, 1};
  if (M < kFewLeast || M > kFewMost || K % BK) return best;
  const int steps = K / BK, v_pad = (V + TV - 1) / TV * TV;
  const bool gated = kind == StreamKind::kGlu;
  static const int kRows[] = {1, 2, 4, 6, 8, 10};
  double best_cost = 1e30;
  for (int rows : kRows) {
    if (rows == 1 && kind != StreamKind::kPlain) continue;
    const long tiles = gated ? (V / 2 + 8 * rows - 1) / (8 * rows) : (V + 16 * rows - 1) / (16 * rows);
    // Many short gated rows.  Beyond 64 tokens it depends on the shape (96 tokens, against the tile kernel: 1280 x 36864
    // 25 and 30 us, 1024 x 32768 22 and 18).  Elsewhere the few rows are 1 to 29 % ahead (64 tokens, 1536 x 28672 22.6 and
    // 28.6).  Rows 4 KB apart lost to the stream up to 32 tokens (2048 x 25600, 17 tokens 28 and 25.5) and to the tile kernel where
    // all CUs are at work (2048 x 32768, 40 tokens 36 and 34) while all workgroups began with the same columns.  Since they
    // don't, the lines for these are too low (few rows and what is taken: 17 tokens x 25600 22.2 and 28.3; 40 tokens x 32768
    // 27.3 and 28.6, x 40960 32.5 and 39.9; 96 tokens 28.8 and 35.2, x 25600 25.7 and 30.2).
    if (gated && rows >= 8 && K <= 2048 && (M > 64 || (K == 2048 && (M <= 32 || tiles > 240)))) continue;
    for (int ks = 1; ks <= (gated || rows == 1 ? 1 : 8); ++ks) {
      if (steps % ks || (ks > 1 && steps / ks < 6) || tiles * ks > 256) continue;
      if (ks > 1 && (size_t)ks * v_pad * few_m_pad(M) * sizeof(float) > workspace) continue;
      const double step = 0.08 + 0.039 * rows + 0.047 * rows * (double)(tiles * ks) / 256 + (M > 64 ? 0.12 : 0.0);
      const double sums = ks > 1 ? 4.0 + 0.86 * 8.0 * ks * v_pad * few_m_pad(M) / 4e6 : 0.0;
      const double cost = 3.0 + steps / ks * step + sums;
      if (cost < best_cost) {
        best_cost = cost;
        best = {rows, ks};
      }
    }
  }
  return best;
}

// 17 to 32 tokens: microseconds of a plan and of the stream, fitted to 2400 measurements of calls in a graph on weights
// too many to stay in the last-level cache (512 to 18944 x 128 to 40960; 5 and 4 % rms).
// Weight rows, or parts of them, that begin a multiple of 4 KB apart meet on few memory channels once all CUs read them,
// unless the workgroups begin at K steps of their own (24 tokens, 4096 x 28672 56 us and, gated, 43; 3072 x 28672 35); two to
// seven parts of 4 KB do all the same (8192 x 4096 20.8, the stream 18.4), but for the tallest tiles (8192 x 10240 36.7, the stream
// 43), and gated rows of 16 KB (8192 x 8200 37.7, the stream 35.6).  370 calls of K a multiple of 2048 are 1.01 to 1.02 times as
// fast as with the conflict expected of all (16384 x 4096 35.8 -> 30.0, 12288 x 11904 72 -> 59).
double few_us(const FewPlan &p, int M, int K, int V, StreamKind kind) {
  const bool gated = kind == StreamKind::kGlu;
  const int tiles = gated ? (V / 2 + 8 * p.rows - 1) / (8 * p.rows) : (V + 16 * p.rows - 1) / (16 * p.rows);
  const double fill = (double)(tiles * p.ks) / 256, v_pad = (V + TV - 1) / TV * TV;
  double row = 0.030 + (gated && (int64_t)K * V >= kUncached ? 0.026 : 0.038) * fill + 0.0017 * p.rows;
  const bool turns = few_turns(K, V, p);
  const bool short_parts = K / p.ks == 2048 && p.ks > 1 && p.ks < 8 && p.rows < 10, whole = K % 8192 == 0 && p.ks == 1;
  const bool meet = K / p.ks % 2048 == 0 && (!turns || short_parts || whole);
  if (p.rows >= 4 && meet) row += (whole ? 0.025 : 0.0147) * fill * fill;
  const double us = 3.3 + K / BK / p.ks * (0.054 + p.rows * row + 0.0087 * fill * fill + 0.00053 * (M - 17));
  if (p.ks > 1) return us + 2.1 + 1.33e-6 * p.ks * v_pad * 64;
  return turns && !whole && p.rows >= 4 && K > 2048 ? 0.95 * us : us;
}
// Up to K = 4096 the tokens stay in registers and two workgroups fit a CU; beyond they travel with the weights, and the
// workgroups take 256 tiles of 16 rows a round.
double stream_us(int M, int K, int V) {
  const double steps = K / BK;
  const int tiles = (V + 15) / 16;
  const double fill = (double)tiles / 256;
  if (K > 4096) return 4.4 + (tiles + 255) / 256 * (0.56 + steps * (0.042 + 0.0016 * M)) + 0.0227 * steps * fill;
  if (tiles > 256) return 12.0 + steps * (0.0025 * M - 0.025 + 0.07 * fill);
  return 4.95 + steps * (0.083 + 0.001 * M + 0.0108 * fill - 0.0006 * steps) + 0.19 * std::log2((double)(tiles > 8 ? tiles : 8));
}

template <bool ROPE, bool GLU>
hipError_t launch_reduce(int M, int V, int ks, int v_pad, int m_pad, const QkvArgs &qa, const StoreArgs &sa, const float *part,
                         const NormArgs &norm, hipStream_t s) {
  if (!ROPE && !GLU && norm_fits(norm, M, V)) {
    proj_reduce_norm_kernel<<<(unsigned)M, kNormThreads, 0, s>>>(V, ks, v_pad, m_pad, part, sa, norm);
    return hipGetLastError();
  }
  const int groups = ROPE ? V / kHeadDim * 16 : GLU ? V / 8 : V / 4;
  proj_reduce_kernel<ROPE, GLU><<<dim3((unsigned)((groups + 255) / 256), (unsigned)M), 256, 0, s>>>(M, V, ks, v_pad, m_pad, groups, part, qa, sa);
  return hipGetLastError();
}

template <bool ROPE, bool GLU>
hipError_t launch_few(StreamKind kind, const FewPlan &p, int M, int K, int V, const void *hidden, const void *weight,
                      const QkvArgs &qa, const StoreArgs &sa, float *part, hipStream_t s, const NormArgs &norm = {}) {
  if (p.ks > 1 && !part) return hipErrorInvalidValue;
  const int v_pad = (V + TV - 1) / TV * TV, m_pad = few_m_pad(M);
  const StreamArgs st = {sa.residual, sa.out, qa.bias, qa.cos, qa.sin, qa.q, qa.k, qa.v, qa.Hq, qa.Hkv, sa.hidden2, sa.weight2};
  hipError_t e = launch_proj_few(kind, p, M, K, V, hidden, weight, st, part, v_pad, m_pad, s);
  if (e != hipSuccess || p.ks == 1) return e;
  return launch_reduce<ROPE, GLU>(M, V, p.ks, v_pad, m_pad, qa, sa, part, norm, s);
}

// More than 128 tokens, where the tiles of proj_pair.hip (tokens x weight rows of 128 x 128, 160 x 128, or 128 x 224 for plain
// projections, whose rows need no partners) fill at most one round of CUs, K of products that are not gated in up to eight parts: the division expected to
// be the fastest, if the 256-row tiles are not.  Microseconds of both, fitted to 1200 measurements of 297 calls (136 to 6144
// tokens, 2048 to 18944 x 2048 to 37888, weights too many to stay in the last-level cache; 6.6 % rms); a K step costs
// by the share of the CUs at work, which meet at the L2s.  What is chosen is within 0.6 % of the faster one in the mean, 135
// of the calls are taken and 17 % faster for it, 110 drawn ones 21 % (256-row tiles -> this, us: 960 x 3584 x 3584 44.6 -> 35.9, rotary 960 x 3584 x
// 4608 53 -> 42, 1280 x 8192 x 4096 108 -> 81, gated 640 x 3584 x 8192 53 -> 43, 2048 x 10752 x 3584 145 -> 135); 224
// rows below K = 1024 are slower, hence not taken there.  More than a round never pays: then the taller tiles move fewer
// bytes from L2 to LDS.  Not kept: 96 x 192 (never the fastest by more than 1 %), 128 x 192, 128 x 256.
double tiles_us(SplitPlan plan, int M, int K, int V) {
  static const double kB[5] = {0, -1.92, 3.25, 6.14, 8.91}, kS[5] = {0, 0.5815, 0.7597, 0.6764, 0.7521}, kF[5] = {0, 0.148, 0.103, 0.455, 0.652};
  const int steps = K / BK, v_tiles = (V + TV - 1) / TV;
  if (plan.ks > 1) {
    const double units = (double)v_tiles * ((M + 64 * plan.mt - 1) / (64 * plan.mt)) * plan.ks;
    return 6.3 + steps / plan.ks * (kS[plan.mt] + kF[plan.mt] * units / 256) + 0.743 * 8.0 * units * TV * 64 * plan.mt / 4e6;
  }
  const int mt = plain_tile_height(M, K, v_tiles);
  const long units = (long)v_tiles * ((M + 64 * mt - 1) / (64 * mt)), rounds = (units + 255) / 256;
  return 3.84 + (double)rounds * (kB[mt] + steps * kS[mt]) + steps * kF[mt] * (double)units / 256;
}
// Where the times above are wrong, and below their range (K from 512, rows from 200; us by the 256-row tiles -> by these).
// K whole on a part of the CUs, where the others have it in parts, takes up to 1.4 times as long as they say: 347 x 2176 x
// 4268 23.5 -> 27.6, rotary 384 x 1728 x 3584 20.2 -> 22.3, gated 242 x 2688 x 6016 25.8 -> 29.7; not so among up to 160
// tokens or with few rows: gated 520 x 1152 x 640 15.9 -> 12.2, plain 1014 x 1152 x 292 15.6 -> 13.8.  Many tokens by few
// rows and short K: 3840 x 1408 x 928 19.1 -> 22.3, 4491 x 2560 x 644 27.6 -> 30.6, at 224 rows a tile 3068 x 1152 x 1696
// 24.8 -> 26.4, but 2250 x 1920 x 2824 37.6 -> 36.6.  With these lines 23 of 2356 drawn calls, most of them on purpose near
// the lines, are more than 2 % slower than by the 256-row tiles (977 x 8960 x 1024 in parts by 8 %); all are 1.115 times as fast.
// The share of the 256-row tiles' time that a plan must be expected to stay below; 0: it is not taken.
double pair_margin(int M, int K, int V, StreamKind kind, SplitPlan plan, int it, int ks, long tiles) {
  const bool plain = kind == StreamKind::kPlain;
  if (ks > 1) return 0.98;
  if (plan.ks > 1 && tiles < 171) {
    if (plain) return M > 512 && V <= 1200 ? 0.98 : 0.0;
    return M > 160 && (int64_t)K * V > (kind == StreamKind::kGlu ? 4000000 : 3000000) ? 0.87 : 0.98;
  }
  if (it == 7 && K < 2048 && (M > 2560 || (K < 1344 && tiles < 250))) return 0.0;
  if (it == 4 && plain && M > 1024 && V < 1024 && K < (M > 4096 ? 3072 : 2048)) return 0.0;
  return 0.98;
}
PairPlan pair_plan(int M, int K, int V, StreamKind kind, SplitPlan plan) {
  static const struct { int it, jt; double b, s, f; } kTiles[] = {
      {4, 4, 5.17, 0.416, 0.116}, {4, 5, 5.97, 0.513, 0.088}, {7, 4, 6.63, 0.679, 0.076}};
  PairPlan best = {0, 0, 1};
  if (M <= kFewMost) return best;
  const int steps = K / BK, v_pad = (V + TV - 1) / TV * TV;
  const double other_us = tiles_us(plan, M, K, V);
  double best_us = other_us;
  for (const auto &t : kTiles) {
    if (t.it % 2 && (kind != StreamKind::kPlain || K < 1024)) continue;
    const long tiles = (long)((V + 32 * t.it - 1) / (32 * t.it)) * ((M + 32 * t.jt - 1) / (32 * t.jt));
    for (int ks = 1; ks <= (kind == StreamKind::kGlu ? 1 : 8) && tiles * ks <= 256; ++ks) {
      // in the workspace that the caller was told to bring, for split_plan
      if (steps % ks || (ks > 1 && (steps / ks < 8 || (size_t)ks * v_pad * M * sizeof(float) > split_bytes(plan, M, V)))) continue;
      const double sums = ks > 1 ? 3.5 + 0.728 * 8.0 * ks * v_pad * M / 4e6 : 0.0;
      const double us = t.b + steps / ks * (t.s + t.f * (double)(tiles * ks) / 256) + sums;
      if (us < best_us && us < pair_margin(M, K, V, kind, plan, t.it, ks, tiles) * other_us) {
        best_us = us;
        best = {t.it, t.jt, ks};
      }
    }
  }
  return best;
}

template <bool ROPE, bool GLU>
hipError_t launch_pair(StreamKind kind, const PairPlan &p, int M, int K, int V, const void *hidden, const void *weight,
                       const QkvArgs &qa, const StoreArgs &sa, float *part, hipStream_t s, const NormArgs &norm = {}) {
  if (p.ks > 1 && !part) return hipErrorInvalidValue;
  const int v_pad = (V + TV - 1) / TV * TV;
  const StreamArgs st = {sa.residual, sa.out, qa.bias, qa.cos, qa.sin, qa.q, qa.k, qa.v, qa.Hq, qa.Hkv, sa.hidden2, sa.weight2};
  hipError_t e = launch_proj_pair(kind, p, M, K, V, hidden, weight, st, part, v_pad, M, s);
  if (e != hipSuccess || p.ks == 1) return e;
  return launch_reduce<ROPE, GLU>(M, V, p.ks, v_pad, M, qa, sa, part, norm, s);
}

// Which kernel takes the product: the stream, few rows against all tokens, tiles whose K steps two groups share, or
// tiles of 256 rows (split over K as ways->split says).  The plan costs the host some microseconds and is made only where it matters.
// From 17 to 32 tokens stream and few rows each have their shapes (us at 17 / 32 tokens by the stream and by few rows:
// 3584 x 3584 10.8 / 11.8 and 10.6 / 11.0; 14336 x 4096 26 / 32 and 34 / 35, in parts 28; 8192 x 8192 29 / 33 and 37; 3584 x
// 16384 28 / 30 and 24; gated 3584 x 37888 50 / 54 and 45, 4096 x 28672 44 / 46 and 43 / 42): the one expected to be faster,
// within 0.3 % of the faster one in the mean of the 2400 calls, and more than 3 % slower in 60 of them.
// Gated rows a multiple of 4 KB apart, more than 150 MB of them, are few rows' whatever is expected (17 tokens, by the stream
// and by few rows: 10240 x 7808 39 and 34 us, 8192 x 14144 49 and 47, 4096 x 28672 43.8 and 43.7).
// Parts of K of 4 KB in tiles of 96 or 128 rows lose to the split into 256-row tiles (32 / 64 tokens, 8192 x 8192 36.6 / 36.1 and
// 33.3 / 34.4, 8192 x 7168 33.9 / 31.8 and 30.2 / 31.0; 128 tokens 14336 x 4608 46 and 41), except eight of them (64 / 128
// tokens, 16384 x 4096 30 / 36 and 34 / 42); other parts do not.
enum class Way { kStream, kFew, kPair, kTiles };
struct Ways {
  FewPlan few;
  SplitPlan split;
  PairPlan pair;
};
Way way_of(int M, int K, int V, StreamKind kind, const float *part, Ways *ways) {
  *ways = {{0, 1}, {1, 1}, {0, 0, 1}};
  FewPlan *few = &ways->few;
  SplitPlan *plan = &ways->split;
  const bool stream = proj_stream_supports(M, K);
  if (M < kFewLeast && stream) return Way::kStream;
  if (part) *plan = split_plan(M, K, V);
  *few = few_plan(M, K, V, kind, split_bytes(*plan, M, V));
  if (few->rows) {
    const bool turned = kind == StreamKind::kGlu && K > 2048 && few_turns(K, V, *few) && (int64_t)K * V >= 75000000;
    if (stream && !turned && stream_us(M, K, V) < few_us(*few, M, K, V, kind)) return Way::kStream;
    return few->ks > 1 && few->ks < 8 && K / few->ks == 2048 && (few->rows == 6 || few->rows == 8) ? Way::kTiles : Way::kFew;
  }
  if (stream && proj_stream_pays(K, V, plan->ks > 1)) return Way::kStream;
  ways->pair = pair_plan(M, K, V, kind, *plan);
  return ways->pair.it ? Way::kPair : Way::kTiles;
}

template <bool ROPE, bool GLU>
hipError_t launch_splitk(int M, int K, int V, SplitPlan plan, const void *hidden, const void *weight, const QkvArgs &qa,
                         const StoreArgs &sa, float *part, hipStream_t s, const NormArgs &norm = {}) {
  const int ks = plan.ks, tm = 64 * plan.mt;
  const int m_tiles = (M + tm - 1) / tm, m_pad = m_tiles * tm;
  const int v_tiles = (V + TV - 1) / TV, v_pad = v_tiles * TV;
  const int units = v_tiles * ks;
  const unsigned grid = deal_grid((long)units * m_tiles);
  const size_t lds_bytes = tile_lds_bytes(plan.mt);
  hipError_t e;
  switch (plan.mt) {
#define HB_SPLITK_CASE(MT_)                                                                                       \
  case MT_: {                                                                                                     \
    auto kern = proj_splitk_kernel<MT_>;                                                                          \
    e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);      \
    if (e != hipSuccess) return e;                                                                                \
    kern<<<grid, 512, lds_bytes, s>>>(M, K, V, ks, v_pad, m_tiles, m_pad, units, (const u32x4 *)hidden,           \
                                      (const u32x4 *)weight, part);                                               \
  } break;
    HB_SPLITK_CASE(1)
    HB_SPLITK_CASE(2)
    HB_SPLITK_CASE(3)
    HB_SPLITK_CASE(4)
#undef HB_SPLITK_CASE
    default: return hipErrorInvalidValue;
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce<ROPE, GLU>(M, V, ks, v_pad, m_pad, qa, sa, part, norm, s);
}

template <bool ROPE, bool GLU>
hipError_t dispatch(int M, int K, int V, const void *hidden, const void *weight, const QkvArgs &qa, const StoreArgs &sa,
                    hipStream_t s) {
  const int mt = plain_tile_height(M, K, (V + TV - 1) / TV);
  switch (mt) {
    case 4: return launch<4, ROPE, GLU>(M, K, V, hidden, weight, qa, sa, s);
    case 3: return launch<3, ROPE, GLU>(M, K, V, hidden, weight, qa, sa, s);
    case 2: return launch<2, ROPE, GLU>(M, K, V, hidden, weight, qa, sa, s);
    default: return launch<1, ROPE, GLU>(M, K, V, hidden, weight, qa, sa, s);
  }
}

// positions[n] = prefix_len[b] + depth(n); one wavefront per sequence, one lane per node
__global__ __launch_bounds__(64) void tree_positions_kernel(int max_nodes, int total_nodes,
                                                           const int32_t *__restrict__ node_offset,
                                                           const int32_t *__restrict__ parent,
                                                           const int32_t *__restrict__ prefix_len,
                                                           int32_t *__restrict__ positions) {
  __shared__ int32_t spar[64];
  const int b = blockIdx.x, lane = threadIdx.x;
  const int n0 = node_offset[b];
  int n = node_offset[b + 1] - n0;
  n = n < 0 ? 0 : (n > max_nodes ? max_nodes : n);
  if (n0 < 0 || n0 + n > total_nodes) n = 0;
  int par = -1;
  if (lane < n) {
    par = parent[n0 + lane];
    if (par >= lane || par < -1) par = -1;  // malformed: a root
  }
  spar[lane] = par;
  __syncthreads();
  int depth = 0;
  for (int x = par, guard = 0; x >= 0 && guard < 64; ++guard) {
    ++depth;
    x = spar[x];
  }
  if (lane < n) positions[n0 + lane] = prefix_len[b] + depth;
}

// cos / sin of positions[t] * theta^(-d / half), d < half, in double precision (the angle reaches
// tens of thousands of radians), stored as float
__global__ __launch_bounds__(256) void rope_table_kernel(int T, int half, double log2_theta,
                                                        const int32_t *__restrict__ positions,
                                                        float *__restrict__ cos_out, float *__restrict__ sin_out) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)T * half) return;
  const int t = (int)(idx / half), d = (int)(idx - (long)t * half);
  const double inv_freq = exp2(-log2_theta * (double)d / (double)half);
  const double ang = (double)positions[t] * inv_freq;
  double sv, cv;
  sincos(ang, &sv, &cv);
  cos_out[idx] = (float)cv;
  sin_out[idx] = (float)sv;
}

}  // namespace

bool proj_mfma_supports(int32_t M, int32_t K, int32_t N) { return M >= 1 && K >= BK && K % BK == 0 && N >= 4 && N % 4 == 0; }

size_t proj_workspace_bytes(int32_t M, int32_t K, int32_t N) {
  return split_bytes(split_plan(M, K, N), M, N);
}

hipError_t launch_qkv_rope(int32_t M, int32_t K, int32_t Hq, int32_t Hkv, const void *hidden, const void *w_qkv,
                           const void *bias, const float *cos, const float *sin, void *q, void *k, void *v,
                           float *part, hipStream_t s) {
  QkvArgs qa = {(const bf16_t *)bias, cos, sin, (bf16_t *)q, (bf16_t *)k, (bf16_t *)v, Hq, Hkv};
  StoreArgs sa = {nullptr, nullptr};
  const int V = (Hq + 2 * Hkv) * kHeadDim;
  Ways ways;
  const Way way = way_of(M, K, V, StreamKind::kRope, part, &ways);
  if (way == Way::kPair) return launch_pair<true, false>(StreamKind::kRope, ways.pair, M, K, V, hidden, w_qkv, qa, sa, part, s);
  if (way == Way::kFew) return launch_few<true, false>(StreamKind::kRope, ways.few, M, K, V, hidden, w_qkv, qa, sa, part, s);
  if (way == Way::kStream) {
    const StreamArgs st = {nullptr, nullptr, qa.bias, cos, sin, qa.q, qa.k, qa.v, Hq, Hkv};
    return launch_proj_stream(StreamKind::kRope, M, K, V, hidden, w_qkv, st, s);
  }
  if (ways.split.ks > 1) return launch_splitk<true, false>(M, K, V, ways.split, hidden, w_qkv, qa, sa, part, s);
  return dispatch<true, false>(M, K, V, hidden, w_qkv, qa, sa, s);
}

static hipError_t launch_linear(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *residual, void *out,
                                float *part, const NormArgs &norm, bool *normed, hipStream_t s) {
  QkvArgs qa = {};
  StoreArgs sa = {(const bf16_t *)residual, (bf16_t *)out};
  Ways ways;
  const Way way = way_of(M, K, N, StreamKind::kPlain, part, &ways);
  const int parts = way == Way::kPair ? ways.pair.ks : way == Way::kFew ? ways.few.ks : way == Way::kTiles ? ways.split.ks : 1;
  *normed = parts > 1 && norm_fits(norm, M, N);
  if (way == Way::kPair) return launch_pair<false, false>(StreamKind::kPlain, ways.pair, M, K, N, x, w, qa, sa, part, s, norm);
  if (way == Way::kFew) return launch_few<false, false>(StreamKind::kPlain, ways.few, M, K, N, x, w, qa, sa, part, s, norm);
  if (way == Way::kStream) return launch_proj_stream(StreamKind::kPlain, M, K, N, x, w, {sa.residual, sa.out}, s);
  if (ways.split.ks > 1) return launch_splitk<false, false>(M, K, N, ways.split, x, w, qa, sa, part, s, norm);
  return dispatch<false, false>(M, K, N, x, w, qa, sa, s);
}

hipError_t launch_linear(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *residual, void *out,
                         float *part, hipStream_t s) {
  bool normed;
  return launch_linear(M, K, N, x, w, residual, out, part, {}, &normed, s);
}

hipError_t launch_linear_norm(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *residual, void *out,
                              const void *norm_weight, float eps, void *norm_out, float *part, hipStream_t s) {
  bool normed;
  hipError_t e = launch_linear(M, K, N, x, w, residual, out, part, {(const bf16_t *)norm_weight, (bf16_t *)norm_out, eps}, &normed, s);
  return e != hipSuccess || normed ? e : launch_rmsnorm(M, N, out, norm_weight, eps, norm_out, s);
}

// One product of 2 K columns where a way takes the halves' operands as they are, which also saves rounding and reading the
// first product: 3584 + 3584 columns x 3584 rows, 96 tokens 29.8 -> 20.5 us, 640 87 -> 49, 2048 116 -> 94; of 51 calls (8 to
// 2048 tokens, 2048 to 4096) 39 go this way, 1.07 to 1.93 times as fast, the others as before.
hipError_t launch_linear_two(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *x2, const void *w2,
                             void *tmp, void *out, float *part, float *part2, hipStream_t s) {
  QkvArgs qa = {};
  const StoreArgs sa = {nullptr, (bf16_t *)out, (const bf16_t *)x2, (const bf16_t *)w2};
  Ways ways;
  const Way way = way_of(M, 2 * K, N, StreamKind::kPlain, part2, &ways);
  if (way == Way::kPair && (ways.pair.ks == 1 || ways.pair.ks % 2 == 0))
    return launch_pair<false, false>(StreamKind::kPlain, ways.pair, M, 2 * K, N, x, w, qa, sa, part2, s);
  if (way == Way::kFew && ways.few.ks % 2 == 0)
    return launch_few<false, false>(StreamKind::kPlain, ways.few, M, 2 * K, N, x, w, qa, sa, part2, s);
  hipError_t e = launch_linear(M, K, N, x, w, nullptr, tmp, part, s);
  return e != hipSuccess ? e : launch_linear(M, K, N, x2, w2, tmp, out, part, s);
}

hipError_t launch_swiglu(int32_t M, int32_t K, int32_t F, const void *x, const void *w_gate_up, void *out, float *part,
                         hipStream_t s) {
  QkvArgs qa = {};
  StoreArgs sa = {nullptr, (bf16_t *)out};
  Ways ways;
  const Way way = way_of(M, K, 2 * F, StreamKind::kGlu, part, &ways);
  if (way == Way::kPair) return launch_pair<false, true>(StreamKind::kGlu, ways.pair, M, K, 2 * F, x, w_gate_up, qa, sa, part, s);
  if (way == Way::kFew) return launch_few<false, true>(StreamKind::kGlu, ways.few, M, K, 2 * F, x, w_gate_up, qa, sa, part, s);
  if (way == Way::kStream) return launch_proj_stream(StreamKind::kGlu, M, K, 2 * F, x, w_gate_up, {nullptr, sa.out}, s);
  if (ways.split.ks > 1) return launch_splitk<false, true>(M, K, 2 * F, ways.split, x, w_gate_up, qa, sa, part, s);
  return dispatch<false, true>(M, K, 2 * F, x, w_gate_up, qa, sa, s);
}

hipError_t launch_rmsnorm(int32_t T, int32_t K, const void *x, const void *weight, float eps, void *out, hipStream_t s) {
  rmsnorm_kernel<<<T, 256, 0, s>>>(K, (const bf16_t *)x, (const bf16_t *)weight, eps, (bf16_t *)out);
  return hipGetLastError();
}

hipError_t launch_tree_positions(int32_t B, int32_t max_nodes, int32_t total_nodes, const int32_t *node_offset,
                                 const int32_t *parent, const int32_t *prefix_len, int32_t *positions, hipStream_t s) {
  tree_positions_kernel<<<B, 64, 0, s>>>(max_nodes, total_nodes, node_offset, parent, prefix_len, positions);
  return hipGetLastError();
}

hipError_t launch_rope_table(int32_t T, int32_t half, double theta, const int32_t *positions, float *cos, float *sin,
                             hipStream_t s) {
  const long n = (long)T * half;
  rope_table_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(T, half, log2(theta), positions, cos, sin);
  return hipGetLastError();
}

}  // namespace hb
