// The projections for 17 to 128 tokens: all tokens in one tile, few weight rows.
//
// With so many tokens the weights are still most of what a projection reads, but a workgroup per 256 weight
// rows leaves most CUs idle, and the split over K that occupied them pays for it with a second launch and
// 5 to 15 MB of partial sums.  Here a tile is 16 R weight rows, R chosen so that the tiles occupy the chip
// once, against all tokens; K is split only where it is long (proj_reduce_kernel sums the parts).
//
// Eight wavefronts.  Up to 128 tokens each takes 16 of them and all rows; up to 64 tokens four groups of 16,
// twice, each half of every K step, and the halves' sums meet in LDS.  Weights and tokens go from memory to LDS
// directly (eight rows of 128 bytes a load, swizzled on the source side) into a ring as deep as LDS allows, all
// stages but one in flight; one barrier per stage of KSP K steps of 64.  A tile's 16-row groups come in
// pairs for the rotary embedding (rows d and d + 64 of a head) and for the gated projection (gate and up rows
// of the same features), so that both members are one lane's own accumulators.
//
// What bounds it: memory where the weights are many, else the CU's path from L2 (64 bytes a clock for 16 R +
// 128 rows a K step) and the time until the first tile is there.  Rows a multiple of 4 KB apart also met on few memory
// channels until the workgroups walked K from steps of their own (few_turns; us before and now: gated 64 tokens 4096 x 32768
// 62 and 44, 128 tokens 64 and 55, 24 tokens 4096 x 16384 37 and 25; 64 tokens 16384 x 2048 22 and 19.6).
#include "hb_internal.h"

namespace hb {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

constexpr int kWaves = 8;
constexpr int kHeadDim = 128;
// Weights beyond the last-level cache's 256 MB, gated: loaded with the non-temporal hint (3584 x 37888, 128 tokens
// 61.5 -> 57.9 us; split over K the hint costs up to 10 %)
constexpr int64_t kUncached = (int64_t)1 << 27;
enum Kind { kPlain, kRope, kGlu, kPart };

template <int R, int TOK, int KSP>
struct Shape {
  static constexpr int kGroups = 2 * R + TOK / 8;          // 8-row groups of a K step: weights, then tokens
  static constexpr int kLoads = kGroups * KSP;             // 1 KiB each, of a stage
  static constexpr int kMost = (kLoads + kWaves - 1) / kWaves;
  static constexpr int kRest = kLoads % kWaves;            // wavefronts that issue kMost; the others one less
  static constexpr int kStages = 160 / kLoads < 8 ? 160 / kLoads : 8;
  static_assert(kStages >= 3 && kStages * kLoads >= (TOK == 64 ? 4 * R : 0), "ring, and room for the halves' sums");
  static constexpr size_t kLdsBytes = (size_t)kStages * kLoads * 1024;
};

// TURN: workgroups begin at stages of their own
template <Kind KIND, int R, int TOK, int KSP, bool TURN>
__device__ __forceinline__ void few_tile(int M, int K, int V, int ks, bool uncached, int v_pad, int m_pad, const u32x4 *__restrict__ hidden,
                                         const u32x4 *__restrict__ weight, const StreamArgs &sa, float *__restrict__ part) {
  using Sh = Shape<R, TOK, KSP>;
  constexpr int SUB = TOK == 128 ? 2 : 1;  // 32-k sub-steps of a K step that a wavefront takes
  extern __shared__ u32x4 lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j16 = lane & 15, kq = lane >> 4;
  const int tile = (int)blockIdx.x / ks, kpart = (int)blockIdx.x % ks;
  const int stages = K / 64 / ks / KSP;
  const bool two = KIND == kPart && sa.hidden2;  // each half of K from its own operands (`ks` is even)
  const int kp = (two ? K / 2 : K) / 8, kfrom = two && 2 * kpart >= ks ? kpart - ks / 2 : kpart;
  if (kfrom != kpart) {
    hidden = (const u32x4 *)sa.hidden2;
    weight = (const u32x4 *)sa.weight2;
  }
  const int F = V >> 1;

  // lane -> row lane / 8 of a group's eight, piece swizzled; rows past the end are clamped and dropped at the end
  const u32x4 *src[Sh::kMost];
#pragma unroll
  for (int i = 0; i < Sh::kMost; ++i) {
    const int n = wave + kWaves * i, kk = n / Sh::kGroups, g = n % Sh::kGroups;
    const int r8 = lane >> 3;
    const u32x4 *base;
    if (g < 2 * R) {
      const int sub = g >> 1, rr = (g & 1) * 8 + r8;
      int row;
      if (KIND == kGlu) {
        const int f = tile * 8 * R + (sub >> 1) * 16 + rr;
        row = (sub & 1) * F + (f < F ? f : F - 1);
      } else if (KIND == kRope) {
        const int pair = tile * (R / 2) + (sub >> 1);
        row = (pair >> 2) * kHeadDim + (pair & 3) * 16 + (sub & 1) * 64 + rr;
      } else {
        row = tile * 16 * R + sub * 16 + rr;
      }
      base = weight + (size_t)(row < V ? row : V - 1) * kp;
    } else {
      const int m = (g - 2 * R) * 8 + r8;
      base = hidden + (size_t)(m < M ? m : M - 1) * kp;
    }
    src[i] = base + (size_t)kfrom * (K / 8 / ks) + kk * 8 + ((lane & 7) ^ r8);
  }
  const bool full = Sh::kRest == 0 || wave < Sh::kRest;
  const int turn = TURN ? (int)((blockIdx.x >> 3) % (unsigned)stages) : 0;
  auto issue = [&](int st, int slot) {
    st = st < stages ? st : stages - 1;  // past the end the last stage again: the waits count loads
    if (TURN) st = st + turn < stages ? st + turn : st + turn - stages;
#pragma unroll
    for (int i = 0; i < Sh::kMost; ++i) {
      if (i == Sh::kMost - 1 && !full) break;
      const auto from = (gptr_t)(src[i] + (size_t)st * (8 * KSP));
      const auto to = (lptr_t)(lds + (slot * Sh::kLoads + wave + kWaves * i) * 64);
      if (KIND == kGlu && uncached && (wave + kWaves * i) % Sh::kGroups < 2 * R)
        __builtin_amdgcn_global_load_lds(from, to, 16, 0, 2);
      else
        __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
    }
  };

  f32x4 acc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int group = TOK == 128 ? wave : wave & 3, half = TOK == 128 ? 0 : wave >> 2;
#pragma unroll
  for (int i = 0; i < Sh::kStages - 1; ++i) issue(i, i);
  int cur = 0, free_slot = Sh::kStages - 1;
#pragma unroll 1
  for (int t = 0; t < stages; ++t) {
    // this wavefront's loads of stage t have landed, its reads of stage t - 1 are done; behind the barrier everybody's
    if (full) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((Sh::kStages - 2) * Sh::kMost) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((Sh::kStages - 2) * (Sh::kMost - 1)) : "memory");
    asm volatile("s_barrier" ::: "memory");
    // reads first: the address unit takes the loads behind them while LDS delivers
    const u32x4 *st = lds + cur * Sh::kLoads * 64;
    bf16x8 a[KSP][SUB][R], b[KSP][SUB];
#pragma unroll
    for (int kk = 0; kk < KSP; ++kk)
#pragma unroll
      for (int s = 0; s < SUB; ++s) {
        const int c = (TOK == 128 ? s : half) * 4 + kq;
        const u32x4 *at = st + kk * Sh::kGroups * 64 + j16 * 8 + (c ^ (j16 & 7));
#pragma unroll
        for (int i = 0; i < R; ++i) a[kk][s][i] = __builtin_bit_cast(bf16x8, at[i * 128]);
        b[kk][s] = __builtin_bit_cast(bf16x8, at[(R + group) * 128]);
      }
    issue(t + Sh::kStages - 1, free_slot);
#pragma unroll
    for (int kk = 0; kk < KSP; ++kk)
#pragma unroll
      for (int s = 0; s < SUB; ++s) {
#pragma unroll
        for (int i = 0; i < R; ++i) asm volatile("" : "+v"(a[kk][s][i]));
        asm volatile("" : "+v"(b[kk][s]));
      }
#pragma unroll
    for (int kk = 0; kk < KSP; ++kk)
#pragma unroll
      for (int s = 0; s < SUB; ++s)
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][s][i], b[kk][s], acc[i], 0, 0, 0);
    cur = cur + 1 == Sh::kStages ? 0 : cur + 1;
    free_slot = free_slot + 1 == Sh::kStages ? 0 : free_slot + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (TOK == 64) {
    __syncthreads();  // every load has landed, every read is done: the ring is free
    f32x4 *sum = reinterpret_cast<f32x4 *>(lds);
    if (half) {
#pragma unroll
      for (int i = 0; i < R; ++i) sum[(i * 4 + group) * 64 + lane] = acc[i];
    }
    __syncthreads();
    if (half) return;
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i] += sum[(i * 4 + group) * 64 + lane];
  }

  // accumulator e of lane (j16, kq) in group i: row 4 kq + e of the group, token m
  const int m = group * 16 + j16;
  if (KIND == kPart) {
    float *dst = part + ((size_t)kpart * m_pad + m) * v_pad + tile * 16 * R + 4 * kq;
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (tile * 16 * R + i * 16 < v_pad) *(f32x4 *)(dst + i * 16) = acc[i];
    return;
  }
  if (m >= M) return;
  if (KIND == kPlain) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int n = tile * 16 * R + i * 16 + 4 * kq;  // n .. n + 3, V % 4 == 0
      if (n >= V) continue;
      f32x4 x = acc[i];
      if (sa.residual) {
        const u32x2 r = *(const u32x2 *)(sa.residual + (size_t)m * V + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] += __uint_as_float((e & 1) ? (r[e >> 1] & 0xffff0000u) : (r[e >> 1] << 16));
      }
      *(u32x2 *)(sa.out + (size_t)m * V + n) = (u32x2){pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
    }
  } else {
#pragma unroll
    for (int p = 0; p < R / 2; ++p) {
      f32x4 x1 = acc[2 * p], x2 = acc[2 * p + 1];
      if (KIND == kGlu) {
        const int f = tile * 8 * R + p * 16 + 4 * kq;  // f .. f + 3, F % 4 == 0
        if (f >= F) continue;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = x1[e] / (1.f + __expf(-x1[e])) * x2[e];
        *(u32x2 *)(sa.out + (size_t)m * F + f) = (u32x2){pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
      } else {
        const int pair = tile * (R / 2) + p, head = pair >> 2, d = (pair & 3) * 16 + 4 * kq;
        if (head >= sa.Hq + 2 * sa.Hkv) continue;
        if (sa.bias) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x1[e] += bf16_to_f32(sa.bias[head * kHeadDim + d + e]);
            x2[e] += bf16_to_f32(sa.bias[head * kHeadDim + 64 + d + e]);
          }
        }
        bf16_t *dst = head < sa.Hq ? sa.q + ((size_t)m * sa.Hq + head) * kHeadDim
                      : head < sa.Hq + sa.Hkv ? sa.k + ((size_t)m * sa.Hkv + (head - sa.Hq)) * kHeadDim
                                              : sa.v + ((size_t)m * sa.Hkv + (head - sa.Hq - sa.Hkv)) * kHeadDim;
        if (head < sa.Hq + sa.Hkv) {
          const f32x4 cs = *(const f32x4 *)(sa.cos + (size_t)m * 64 + d);
          const f32x4 sn = *(const f32x4 *)(sa.sin + (size_t)m * 64 + d);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float c1 = x1[e] * cs[e] - x2[e] * sn[e];
            const float c2 = x2[e] * cs[e] + x1[e] * sn[e];
            x1[e] = c1;
            x2[e] = c2;
          }
        }
        *(u32x2 *)(dst + d) = (u32x2){pack_bf16(x1[0], x1[1]), pack_bf16(x1[2], x1[3])};
        *(u32x2 *)(dst + d + 64) = (u32x2){pack_bf16(x2[0], x2[1]), pack_bf16(x2[2], x2[3])};
      }
    }
  }
}

template <Kind KIND, int R, int TOK, int KSP>
__global__ __launch_bounds__(512) void proj_few_kernel(int M, int K, int V, int ks, bool uncached, int v_pad, int m_pad,
                                                       const u32x4 *__restrict__ hidden, const u32x4 *__restrict__ weight,
                                                       StreamArgs sa, float *__restrict__ part) {
  few_tile<KIND, R, TOK, KSP, false>(M, K, V, ks, uncached, v_pad, m_pad, hidden, weight, sa, part);
}
// A kernel of its own for those that turn: asked for in the one, it cost short calls 1 to 2 %.
struct Turned {};
template <Kind KIND, int R, int TOK, int KSP>
__global__ __launch_bounds__(512) void proj_few_kernel(int M, int K, int V, int ks, bool uncached, int v_pad, int m_pad,
                                                       const u32x4 *__restrict__ hidden, const u32x4 *__restrict__ weight,
                                                       StreamArgs sa, float *__restrict__ part, Turned) {
  few_tile<KIND, R, TOK, KSP, true>(M, K, V, ks, uncached, v_pad, m_pad, hidden, weight, sa, part);
}

template <Kind KIND, int R, int TOK, int KSP>
hipError_t launch(int M, int K, int V, int ks, int v_pad, int m_pad, const void *hidden, const void *weight, const StreamArgs &sa,
                  float *part, hipStream_t s) {
  using Sh = Shape<R, TOK, KSP>;
  const int tiles = KIND == kGlu ? (V / 2 + 8 * R - 1) / (8 * R) : (V + 16 * R - 1) / (16 * R);
  const bool uncached = (int64_t)K * V >= kUncached;
  auto run = [&](auto kern, auto... turned) {
    const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Sh::kLdsBytes);
    if (e != hipSuccess) return e;
    kern<<<tiles * ks, 512, Sh::kLdsBytes, s>>>(M, K, V, ks, uncached, v_pad, m_pad, (const u32x4 *)hidden, (const u32x4 *)weight, sa, part, turned...);
    return hipGetLastError();
  };
  using Whole = void (*)(int, int, int, int, bool, int, int, const u32x4 *, const u32x4 *, StreamArgs, float *);
  using Turning = void (*)(int, int, int, int, bool, int, int, const u32x4 *, const u32x4 *, StreamArgs, float *, Turned);
  return few_turns(K, V, {R, ks}) ? run((Turning)proj_few_kernel<KIND, R, TOK, KSP>, Turned{}) : run((Whole)proj_few_kernel<KIND, R, TOK, KSP>);
}

template <Kind KIND, int TOK>
hipError_t dispatch(const FewPlan &p, int M, int K, int V, int v_pad, int m_pad, const void *hidden, const void *weight,
                    const StreamArgs &sa, float *part, hipStream_t s) {
#define HB_FEW(R_, KSP_) return launch<KIND, R_, TOK, KSP_>(M, K, V, p.ks, v_pad, m_pad, hidden, weight, sa, part, s)
  const bool two = K / 64 / p.ks % 2 == 0;  // K steps that go two to a stage
  switch (p.rows) {
    case 1:
      if constexpr (KIND == kPlain) {
        if (two) HB_FEW(1, 2);
        HB_FEW(1, 1);
      }
      return hipErrorInvalidValue;
    case 2:
      if (two) HB_FEW(2, 2);
      HB_FEW(2, 1);
    case 4:
      if (two) HB_FEW(4, 2);
      HB_FEW(4, 1);
    case 6: HB_FEW(6, 1);
    case 8: HB_FEW(8, 1);
    case 10: HB_FEW(10, 1);
    default: return hipErrorInvalidValue;
  }
#undef HB_FEW
}

}  // namespace

hipError_t launch_proj_few(StreamKind kind, const FewPlan &p, int32_t M, int32_t K, int32_t V, const void *hidden,
                           const void *weight, const StreamArgs &sa, float *part, int32_t v_pad, int32_t m_pad, hipStream_t s) {
#define HB_KIND(K_) (M <= 64 ? dispatch<K_, 64>(p, M, K, V, v_pad, m_pad, hidden, weight, sa, part, s) \
                             : dispatch<K_, 128>(p, M, K, V, v_pad, m_pad, hidden, weight, sa, part, s))
  if (p.ks > 1) return HB_KIND(kPart);
  switch (kind) {
    case StreamKind::kRope: return HB_KIND(kRope);
    case StreamKind::kGlu: return HB_KIND(kGlu);
    default: return HB_KIND(kPlain);
  }
#undef HB_KIND
}

}  // namespace hb
