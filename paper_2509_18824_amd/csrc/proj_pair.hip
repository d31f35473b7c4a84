// Projections of more than a few tokens by tiles of which the chip holds about one round: C^T = W H^T, a
// workgroup per tile of 32 IT weight rows x 32 JT tokens.
//
// The tile loop of mfma_gemm_tile.inc lets the two wavefronts of a SIMD alternate between operands and matrix
// instructions, each on its own part of one K step.  Its phases cost about 280 clocks beside the matrix work (the
// barrier, the latency of the LDS reads), so its rate falls with the size of a wavefront's part: 64 x 64 for a tile
// of 256 x 128, 64 x 32 for 256 x 64, which is what is left when 3584 weight rows and 960 tokens are to occupy
// 256 CUs.  Here the wavefronts share K instead: wavefronts 0-3 take the even K steps and 4-7 the odd ones, each group all
// of the tile, so a tile of 128 x 128 has parts of 64 x 64 and of 224 x 128 parts of 112 x 64.  A phase is one K step for one
// group's operands and the step before it for the other's matrix instructions.  In the end the two groups' sums
// meet in LDS, as [token][weight row], from where results leave in whole lines.
#include "mfma_gemm_tile.h"

namespace hb {

namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kHeadDim = 128;

// One K step of both operands in LDS: TV weight rows, then TM tokens, 128 bytes each.
constexpr int stage_bytes(int it, int jt) { return 32 * (it + jt) * CH * 16; }
constexpr int stages(int it, int jt) { return 163840 / stage_bytes(it, jt) < 5 ? 163840 / stage_bytes(it, jt) : 5; }
constexpr int sums_bytes(int it, int jt) { return (32 * it + 4) * 32 * jt * 4; }
constexpr int lds_bytes(int it, int jt) {
  return stages(it, jt) * stage_bytes(it, jt) > sums_bytes(it, jt) ? stages(it, jt) * stage_bytes(it, jt) : sums_bytes(it, jt);
}

enum { kPlainKind, kRopeKind, kGluKind, kPartKind };

__device__ inline float bf16_of(uint32_t word, int e) { return __uint_as_float(e & 1 ? word & 0xffff0000u : word << 16); }

// KIND: plain projection (+ residual), rotary embedding, gated, or the partial sums of one of `ks` parts of K.
template <int KIND, int IT, int JT>
__global__ __launch_bounds__(512) void proj_pair_kernel(int M, int Kfull, int V, int ks, int m_tiles, int units,
                                                        const u32x4 *__restrict__ hidden_full,
                                                        const u32x4 *__restrict__ weight_full, StreamArgs sa,
                                                        float *__restrict__ part, int v_pad, int m_pad) {
  constexpr int TVP = 32 * IT, TM = 32 * JT, STAGE = (TVP + TM) * CH, R = stages(IT, JT), N = IT + JT;
  extern __shared__ u32x4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, quad = wave & 3, wv = quad >> 1, wm = quad & 1;
  // every XCD gets one run of units, neighbours share weight rows
  const int per = (units + kXcds - 1) / kXcds, slot = (int)blockIdx.x / kXcds;
  const int unit = (int)blockIdx.x % kXcds * per + slot;
  if (slot >= per || unit >= units) return;
  const int m_tile = unit % m_tiles, v_unit = unit / m_tiles;
  const int v_tile = KIND == kPartKind ? v_unit / ks : v_unit, kpart = KIND == kPartKind ? v_unit % ks : 0;
  const int K = KIND == kPartKind ? Kfull / ks : Kfull;
  const int m0 = m_tile * TM, v0 = v_tile * TVP;
  // two: each half of K from its own operands.  An even number of parts reads one or the other; a whole tile changes over
  // at step `half`, by the distance of the operands.
  const bool two = (KIND == kPlainKind || KIND == kPartKind) && sa.hidden2;
  const int kp = (two ? Kfull / 2 : Kfull) / 8, kfrom = two && 2 * kpart >= ks && KIND == kPartKind ? kpart - ks / 2 : kpart;
  const u32x4 *hidden = (kfrom != kpart ? (const u32x4 *)sa.hidden2 : hidden_full) + (size_t)kfrom * (K / 8);
  const u32x4 *weight = (kfrom != kpart ? (const u32x4 *)sa.weight2 : weight_full) + (size_t)kfrom * (K / 8);
  const bool change = KIND == kPlainKind && two;
  const int half = change ? K / 2 / BK : 0;
  const long to_hidden2 = change ? ((long)(uintptr_t)sa.hidden2 - (long)(uintptr_t)hidden) / 16 - (long)half * CH : 0;
  const long to_weight2 = change ? ((long)(uintptr_t)sa.weight2 - (long)(uintptr_t)weight) / 16 - (long)half * CH : 0;

  // Weight row of tile row t.  Rotary and gated tiles alternate between 16 rows of the first kind (d, gate) and the
  // 16 of the second (d + 64, up) that belong to them.
  auto row_of = [&](int t) {
    if (KIND == kRopeKind) {
      const int p = (v0 + t) >> 5;
      return (p >> 2) * kHeadDim + (p & 3) * 16 + ((t >> 4) & 1) * 64 + (t & 15);
    }
    if (KIND == kGluKind) return ((t >> 4) & 1) * (V >> 1) + ((v0 + t) >> 5) * 16 + (t & 15);
    return v0 + t;
  };
  // Global -> LDS directly, eight rows an instruction, the swizzle applied on the source side; rows past the end
  // are clamped and dropped below.  A group's wavefront takes every fourth eight rows of the step.
  const int grow = lane >> 3;
  const u32x4 *src[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int r8 = (quad + 4 * i) * 8 + grow;
    if (i < IT) {
      const int r = row_of(r8);
      src[i] = weight + (size_t)(r < V ? r : V - 1) * kp + ((lane & 7) ^ grow);
    } else {
      const int r = m0 + r8 - TVP;
      src[i] = hidden + (size_t)(r < M ? r : M - 1) * kp + ((lane & 7) ^ grow);
    }
  }
  typedef __attribute__((address_space(1))) const void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;
  const int k_steps = K / BK, last = k_steps - 1;
  // past the end the last step is fetched again into a free stage (no branch in the loop); nothing reads it
  auto issue = [&](int step, int stage) {
    const int k = step < last ? step : last;
    const long w_off = k * CH + (change && k >= half ? to_weight2 : 0), h_off = k * CH + (change && k >= half ? to_hidden2 : 0);
#pragma unroll
    for (int i = 0; i < N; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + (i < IT ? w_off : h_off)), (lptr_t)(lds + stage * STAGE + (quad + 4 * i) * 64), 16, 0, 0);
  };
  // All loads of this wavefront but those of its newest steps have landed (with R stages, (R - 2) / 2 of its steps).
#define HB_PAIR_LANDED() asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * ((R - 2) / 2)) : "memory")
#define HB_PAIR_PHASE() asm volatile("s_barrier" ::: "memory")

  f32x4 acc[IT][JT];
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int j = 0; j < JT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int frag_row = lane & 15, frag_k = lane >> 4;

  // Pipeline.  In phase p the group p % 2 reads step p from LDS and requests step p + R - 1 into the stage that
  // was read a phase earlier; the other group does the matrix instructions of step p - 1.  Step s is so requested by the
  // group of (s + R + 1) % 2, which sees that it has landed at the end of phase s - 1: with an odd R at the end of its own
  // matrix instructions, with an even R behind its requests.
#pragma unroll
  for (int s = 0; s < R - 1; ++s)
    if (((s + R + 1) & 1) == grp) issue(s, s);
  HB_PAIR_LANDED();
  HB_PAIR_PHASE();
  if (grp) HB_PAIR_PHASE();
  int stage = grp, free = grp ? 0 : R - 1;
#pragma unroll 1
  for (int t = grp; t < k_steps; t += 2) {
    const u32x4 *cw = lds + stage * STAGE, *ch = cw + TVP * CH;
    bf16x8 a[2][IT], b[2][JT];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int c = s * 4 + frag_k;  // this lane's 8-k piece
#pragma unroll
      for (int i = 0; i < IT; ++i) a[s][i] = __builtin_bit_cast(bf16x8, cw[swz((wv * IT + i) * 16 + frag_row, c)]);
#pragma unroll
      for (int j = 0; j < JT; ++j) b[s][j] = __builtin_bit_cast(bf16x8, ch[swz((wm * JT + j) * 16 + frag_row, c)]);
    }
    issue(t + R - 1, free);
#pragma unroll
    for (int s = 0; s < 2; ++s) {  // the LDS reads are waited for here
#pragma unroll
      for (int i = 0; i < IT; ++i) asm volatile("" : "+v"(a[s][i]));
#pragma unroll
      for (int j = 0; j < JT; ++j) asm volatile("" : "+v"(b[s][j]));
    }
    if (R % 2 == 0) HB_PAIR_LANDED();
    HB_PAIR_PHASE();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int jj = 0; jj < JT; ++jj) {
          const int j = (i & 1) ? JT - 1 - jj : jj;  // one operand stays for the next instruction
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s][i], b[s][j], acc[i][j], 0, 0, 0);
        }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (R % 2 == 1) HB_PAIR_LANDED();
    HB_PAIR_PHASE();
    stage = stage + 2 >= R ? stage + 2 - R : stage + 2;
    free = free + 2 >= R ? free + 2 - R : free + 2;
  }
  if ((k_steps & 1) == grp) HB_PAIR_PHASE();  // both groups pass k_steps + 1 phases
#undef HB_PAIR_LANDED
#undef HB_PAIR_PHASE
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // all loads landed, all operand reads done: LDS is free

  // The groups' sums as [token][weight row]: each group hands over half of the token tiles and adds to the other half.
  constexpr int XS = TVP + 4, J0 = (JT + 1) / 2;
  float *xs = (float *)lds;
  float *mine = xs + (size_t)(wm * 16 * JT + frag_row) * XS + wv * 16 * IT + 4 * frag_k;
#define HB_PAIR_AT(i_, j_) (*(f32x4 *)(mine + (j_) * 16 * XS + (i_) * 16))
#pragma unroll
  for (int j = 0; j < JT; ++j)
    if ((j < J0) == (grp == 1)) {
#pragma unroll
      for (int i = 0; i < IT; ++i) HB_PAIR_AT(i, j) = acc[i][j];
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < JT; ++j)
    if ((j < J0) == (grp == 0)) {
#pragma unroll
      for (int i = 0; i < IT; ++i) HB_PAIR_AT(i, j) += acc[i][j];
    }
  __syncthreads();
#undef HB_PAIR_AT

  // Results: neighbouring lanes take neighbouring features of a token, four each.
  constexpr int PIECES = KIND == kPlainKind || KIND == kPartKind ? TVP / 4 : TVP / 8;
#pragma unroll 4
  for (int idx = tid; idx < TM * PIECES; idx += 512) {
    const int tok = idx / PIECES, pc = idx % PIECES, m = m0 + tok;
    if (m >= M) break;
    if (KIND == kPlainKind || KIND == kPartKind) {
      const int n = v0 + pc * 4;
      if (n >= V) continue;  // V % 4 == 0
      f32x4 x = *(const f32x4 *)(xs + (size_t)tok * XS + pc * 4);
      if (KIND == kPartKind) {
        *(f32x4 *)(part + ((size_t)kpart * m_pad + m) * v_pad + n) = x;
      } else {
        if (sa.residual) {
          const u32x2 r = *(const u32x2 *)(sa.residual + (size_t)m * V + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] += bf16_of(r[e >> 1], e);
        }
        *(u32x2 *)(sa.out + (size_t)m * V + n) = (u32x2){pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
      }
    } else {
      const int p = (v0 >> 5) + (pc >> 2), dd = (pc & 3) * 4;  // block of 16 pairs, first of this lane's four
      f32x4 x1 = *(const f32x4 *)(xs + (size_t)tok * XS + (pc >> 2) * 32 + dd);
      f32x4 x2 = *(const f32x4 *)(xs + (size_t)tok * XS + (pc >> 2) * 32 + 16 + dd);
      if (KIND == kGluKind) {
        const int F = V >> 1, f = p * 16 + dd;
        if (f >= F) continue;  // F % 4 == 0
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = x1[e] / (1.f + __expf(-x1[e])) * x2[e];
        *(u32x2 *)(sa.out + (size_t)m * F + f) = (u32x2){pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
      } else {
        const int head = p >> 2, d = (p & 3) * 16 + dd;
        if (head >= sa.Hq + 2 * sa.Hkv) continue;
        bf16_t *dst = head < sa.Hq ? sa.q + ((size_t)m * sa.Hq + head) * kHeadDim
                      : head < sa.Hq + sa.Hkv ? sa.k + ((size_t)m * sa.Hkv + (head - sa.Hq)) * kHeadDim
                                              : sa.v + ((size_t)m * sa.Hkv + (head - sa.Hq - sa.Hkv)) * kHeadDim;
        if (sa.bias) {
          const u32x2 b1 = *(const u32x2 *)(sa.bias + head * kHeadDim + d);
          const u32x2 b2 = *(const u32x2 *)(sa.bias + head * kHeadDim + d + 64);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x1[e] += bf16_of(b1[e >> 1], e);
            x2[e] += bf16_of(b2[e >> 1], e);
          }
        }
        if (head < sa.Hq + sa.Hkv) {
          const f32x4 cs = *(const f32x4 *)(sa.cos + (size_t)m * 64 + d);
          const f32x4 sn = *(const f32x4 *)(sa.sin + (size_t)m * 64 + d);
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
    }
  }
}

template <int KIND, int IT, int JT>
hipError_t launch(const PairPlan &p, int M, int K, int V, const void *hidden, const void *weight, const StreamArgs &sa, float *part,
                  int v_pad, int m_pad, hipStream_t s) {
  const int m_tiles = (M + 32 * JT - 1) / (32 * JT), v_tiles = (V + 32 * IT - 1) / (32 * IT);
  const long units = (long)m_tiles * v_tiles * p.ks;
  constexpr int bytes = lds_bytes(IT, JT);
  auto kern = proj_pair_kernel<KIND, IT, JT>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  kern<<<(unsigned)((units + kXcds - 1) / kXcds * kXcds), 512, bytes, s>>>(M, K, V, p.ks, m_tiles, (int)units, (const u32x4 *)hidden,
                                                                          (const u32x4 *)weight, sa, part, v_pad, m_pad);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_proj_pair(StreamKind kind, const PairPlan &p, int32_t M, int32_t K, int32_t V, const void *hidden,
                            const void *weight, const StreamArgs &sa, float *part, int32_t v_pad, int32_t m_pad, hipStream_t s) {
#define HB_PAIR_CASE(KIND_, IT_, JT_) \
  if (p.it == IT_ && p.jt == JT_) return launch<KIND_, IT_, JT_>(p, M, K, V, hidden, weight, sa, part, v_pad, m_pad, s);
#define HB_PAIR_EVEN(KIND_) HB_PAIR_CASE(KIND_, 4, 4) HB_PAIR_CASE(KIND_, 4, 5)
  if (p.ks > 1) {
    if (!part) return hipErrorInvalidValue;
    HB_PAIR_EVEN(kPartKind)  // the parts of a rotary or gated product meet in proj_reduce_kernel: rows in memory order
    HB_PAIR_CASE(kPartKind, 7, 4)
  } else if (kind == StreamKind::kPlain) {
    HB_PAIR_EVEN(kPlainKind)
    HB_PAIR_CASE(kPlainKind, 7, 4)
  } else if (kind == StreamKind::kRope) {
    HB_PAIR_EVEN(kRopeKind)
  } else {
    HB_PAIR_EVEN(kGluKind)
  }
#undef HB_PAIR_EVEN
#undef HB_PAIR_CASE
  return hipErrorInvalidValue;
}

}  // namespace hb
