// The projections around the attention for up to 16 tokens, and up to 32 where this is the faster way: streams of
// the weight matrix.
//
// With so few tokens a projection is its weights read once from HBM and next to no arithmetic.  What
// counts is that every CU has enough bytes in flight all the time and that nothing else is launched:
// a workgroup takes tiles of 16 weight rows over the whole of K, so that there are no partial results
// in memory and no second kernel, and the tiles are small enough to occupy all CUs (4608 rows: 288).
//
// The eight wavefronts of a workgroup deal out the K steps of 64; each has a ring of LDS stages of
// its own, filled from memory directly (eight rows of 128 bytes per load: fragment-order loads would
// take four times as long in the address unit) and emptied into matrix instructions, with no barrier:
// a wavefront waits for its own loads only.  The ring runs on across the workgroup's tiles.  At the
// end of a tile the wavefronts' sums meet in LDS, in the order of the wavefronts.
//
// HREG: with K at most 4096 a wavefront meets the same steps in every tile (at most eight) and keeps
// the tokens' fragments in registers; the ring then holds weights only and two workgroups fit a CU.
// Otherwise the tokens travel through the ring beside the weights.
//
// A tile is eight rows and their eight partners: for the rotary embedding the rows 64 further on in
// the head, for the gated projection the up rows of the same features, else the next eight.
//
// What bounds it: the weight stream where there is enough of it (gated, 272 MB: 5.9 TB/s), the time
// until the first tile arrives and the sums at the end where there is not (3584 x 3584: 8.9 us).
#include "hb_internal.h"

namespace hb {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lptr_t;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kHeadDim = 128;
constexpr int kRegSteps = 8;                   // K steps of a wavefront whose tokens stay in registers
constexpr int kBufferFlags = 0x00027000;       // untyped 32-bit elements
constexpr int kNonTemporal = 2;                // every weight is read once: 8 tokens, gated projection 51 -> 46 us

__device__ inline int swz(int r, int c) { return r * 8 + (c ^ ((r & 7) ^ ((r >> 3) & 1))); }

template <StreamKind KIND, int HG, bool HREG>
struct Shape {
  static constexpr int TT = (HG + 1) / 2;                            // 16-token tiles
  static constexpr int kStagePieces = 128 + (HREG ? 0 : 64 * HG);    // 16 weight rows (+ the tokens) of 128 bytes
  static constexpr int kStages = HREG ? 4 : (HG == 1 ? 5 : HG == 2 ? 4 : 3);
  static constexpr int kLoads = kStagePieces / 64;                   // per step
  static constexpr int kRedFloats = kWaves * 16 * 16 * TT;
  static constexpr int kReds = TT == 1 ? 2 : 1;                      // buffers for the wavefronts' sums
  static constexpr size_t kLdsBytes = (size_t)kWaves * kStages * kStagePieces * 16 + kReds * kRedFloats * 4;
  static_assert(kLdsBytes <= (HREG ? 80 : 160) * 1024, "two workgroups per CU, or one");
};

// HG: groups of eight tokens (M <= 8 HG)
template <StreamKind KIND, int HG, bool HREG>
__global__ __launch_bounds__(kThreads) void proj_stream_kernel(int M, int K, int N, int tiles,
                                                               const u32x4 *__restrict__ hidden,
                                                               const u32x4 *__restrict__ weight, StreamArgs sa) {
  using Sh = Shape<KIND, HG, HREG>;
  constexpr int TT = Sh::TT;
  extern __shared__ u32x4 lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j16 = lane & 15, kq = lane >> 4;
  u32x4 *ring = lds + wave * Sh::kStages * Sh::kStagePieces;
  float *red = reinterpret_cast<float *>(lds + kWaves * Sh::kStages * Sh::kStagePieces);

  const int row_bytes = K * 2;
  const int steps = K / 64;
  const int mine = (steps - wave + kWaves - 1) / kWaves;  // steps wave, wave + 8, ...
  const int my_tiles = (tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  // lane -> row lane / 8 of eight, piece swizzled on the source side; the partners are rows 8 .. 15
  const int r8 = lane >> 3;
  const int src0 = r8 * row_bytes + ((lane & 7) ^ r8) * 16, src1 = r8 * row_bytes + ((lane & 7) ^ r8 ^ 1) * 16;
  const auto h_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)hidden, 0, M * row_bytes, kBufferFlags);

  // position of the next load in the stream of (tile, step)
  int load_tile = blockIdx.x, load_step = 0, load_slot = 0;
  auto issue = [&]() {
    // the tile's rows and partners; rows past the end are out of range and arrive as zeros
    const int t = min(load_tile, tiles - 1);
    long row, partner;
    int rows, partners;
    if (KIND == StreamKind::kRope) {
      row = (long)(t / 8) * kHeadDim + t % 8 * 8;
      partner = row + 64;
      rows = partners = 8;
    } else if (KIND == StreamKind::kGlu) {
      row = (long)t * 8;
      partner = row + (N >> 1);
      rows = partners = min(8, (N >> 1) - t * 8);
    } else {
      row = (long)t * 16;
      partner = row + 8;
      rows = min(8, N - t * 16);
      partners = max(0, min(8, N - t * 16 - 8));
    }
    const int k = (wave + load_step * kWaves) * 128;
    u32x4 *dst = ring + load_slot * Sh::kStagePieces;
    const auto a = __builtin_amdgcn_make_buffer_rsrc((void *)(weight + row * (row_bytes / 16)), 0, rows * row_bytes, kBufferFlags);
    const auto b = __builtin_amdgcn_make_buffer_rsrc((void *)(weight + (partners ? partner : row) * (row_bytes / 16)), 0,
                                                     partners * row_bytes, kBufferFlags);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(a, (lptr_t)dst, 16, src0, k, 0, kNonTemporal);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (lptr_t)(dst + 64), 16, src1, k, 0, kNonTemporal);
    if (!HREG) {
#pragma unroll
      for (int i = 0; i < HG; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(h_rsrc, (lptr_t)(dst + 128 + i * 64), 16,
                                                 ((i & 1) ? src1 : src0) + i * 8 * row_bytes, k, 0, 0);
    }
    // past the last tile its last steps are loaded again: the waits count loads
    load_slot = load_slot + 1 == Sh::kStages ? 0 : load_slot + 1;
    if (++load_step == mine) {
      load_step = 0;
      load_tile += gridDim.x;
    }
  };
  if (mine > 0) {
#pragma unroll
    for (int i = 0; i < Sh::kStages; ++i) issue();
  }
  bf16x8 hreg[HREG ? kRegSteps : 1][2][TT];
  if (HREG) {
#pragma unroll
    for (int s = 0; s < kRegSteps; ++s)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
          if (s < mine)
            hreg[s][ks][tt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                h_rsrc, (tt * 16 + (lane >> 2)) * row_bytes + (lane & 3) * 16, (wave + s * kWaves) * 128 + ks * 64, 0));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < kRegSteps; ++s)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          // loaded with four neighbouring lanes in one row (four rows take the address unit four times
          // as long); lane (j16, kq) takes its piece from lane 4 j16 + kq
          u32x4 x = __builtin_bit_cast(u32x4, hreg[s][ks][tt]);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_ds_bpermute((4 * j16 + kq) * 4, x[e]);
          hreg[s][ks][tt] = __builtin_bit_cast(bf16x8, x);
          asm volatile("" : "+v"(hreg[s][ks][tt]));
        }
  }

  int slot = 0;
#pragma unroll 1
  for (int n = 0; n < my_tiles; ++n) {
    f32x4 acc[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc[tt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto step = [&](int s) {
      // this stage has landed; the newer loads stay in flight
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((Sh::kStages - 1) * Sh::kLoads) : "memory");
      const u32x4 *st = ring + slot * Sh::kStagePieces;
      bf16x8 w[2], h[2][TT];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        w[ks] = __builtin_bit_cast(bf16x8, st[swz(j16, 4 * ks + kq)]);
        if (!HREG) {
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) h[ks][tt] = __builtin_bit_cast(bf16x8, st[128 + tt * 128 + swz(HG == 1 ? j16 & 7 : j16, 4 * ks + kq)]);
        }
      }
      // the stage has been read and can be filled again
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        asm volatile("" : "+v"(w[ks]));
        if (!HREG) {
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) asm volatile("" : "+v"(h[ks][tt]));
        }
      }
      issue();
      slot = slot + 1 == Sh::kStages ? 0 : slot + 1;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
          acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks], HREG ? hreg[HREG ? s : 0][ks][tt] : h[ks][tt], acc[tt], 0, 0, 0);
    };
    if (HREG) {
#pragma unroll
      for (int s = 0; s < kRegSteps; ++s)
        if (s < mine) step(s);
    } else {
#pragma unroll 1
      for (int s = 0; s < mine; ++s) step(0);
    }

    // lane (j16, kq) holds rows 4 kq .. 4 kq + 3 of token j16; with two buffers one barrier per tile is enough
    float *r = red + (Sh::kReds == 2 ? n & 1 : 0) * Sh::kRedFloats;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) *reinterpret_cast<f32x4 *>(r + ((wave * TT + tt) * 16 + j16) * 16 + 4 * kq) = acc[tt];
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    auto sum = [&](int m, int row) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) x += r[((w * TT + (m >> 4)) * 16 + (m & 15)) * 16 + row];
      return x;
    };
    const int tile = blockIdx.x + n * gridDim.x;
    if (KIND == StreamKind::kPlain) {
      const int m = tid >> 4, row = tid & 15, col = tile * 16 + row;
      if (m < M && m < 16 * TT && col < N) {
        float x = sum(m, row);
        if (sa.residual) x += bf16_to_f32(sa.residual[(size_t)m * N + col]);
        sa.out[(size_t)m * N + col] = f32_to_bf16(x);
      }
    } else {
      const int m = tid >> 3, i = tid & 7;
      if (m < M && m < 16 * TT) {
        float x1 = sum(m, i), x2 = sum(m, 8 + i);
        if (KIND == StreamKind::kGlu) {
          const int F = N >> 1, f = tile * 8 + i;
          if (f < F) sa.out[(size_t)m * F + f] = f32_to_bf16(x1 / (1.f + __expf(-x1)) * x2);
        } else {
          const int head = tile >> 3, d = (tile & 7) * 8 + i;
          if (sa.bias) {
            x1 += bf16_to_f32(sa.bias[head * kHeadDim + d]);
            x2 += bf16_to_f32(sa.bias[head * kHeadDim + d + 64]);
          }
          bf16_t *dst = head < sa.Hq ? sa.q + ((size_t)m * sa.Hq + head) * kHeadDim
                        : head < sa.Hq + sa.Hkv ? sa.k + ((size_t)m * sa.Hkv + (head - sa.Hq)) * kHeadDim
                                                : sa.v + ((size_t)m * sa.Hkv + (head - sa.Hq - sa.Hkv)) * kHeadDim;
          if (head < sa.Hq + sa.Hkv) {
            const float cs = sa.cos[(size_t)m * 64 + d], sn = sa.sin[(size_t)m * 64 + d];
            const float a = x1 * cs - x2 * sn, b = x2 * cs + x1 * sn;
            x1 = a;
            x2 = b;
          }
          dst[d] = f32_to_bf16(x1);
          dst[d + 64] = f32_to_bf16(x2);
        }
      }
    }
    if (Sh::kReds == 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may land in LDS that belongs to somebody else
}

template <StreamKind KIND, int HG, bool HREG>
hipError_t launch(int M, int K, int N, const void *hidden, const void *weight, const StreamArgs &sa, hipStream_t s) {
  using Sh = Shape<KIND, HG, HREG>;
  const int tiles = KIND == StreamKind::kGlu ? (N / 2 + 7) / 8 : (N + 15) / 16;
  const int most = HREG ? 512 : 256;  // workgroups resident at once
  auto kern = proj_stream_kernel<KIND, HG, HREG>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Sh::kLdsBytes);
  if (e != hipSuccess) return e;
  kern<<<tiles < most ? tiles : most, kThreads, Sh::kLdsBytes, s>>>(M, K, N, tiles, (const u32x4 *)hidden, (const u32x4 *)weight, sa);
  return hipGetLastError();
}

template <StreamKind KIND>
hipError_t dispatch(int M, int K, int N, const void *hidden, const void *weight, const StreamArgs &sa, hipStream_t s) {
  const bool reg = K / 64 <= kWaves * kRegSteps;
  if (M <= 16 && reg) return launch<KIND, 2, true>(M, K, N, hidden, weight, sa, s);
  if (M <= 8) return launch<KIND, 1, false>(M, K, N, hidden, weight, sa, s);
  if (M <= 16) return launch<KIND, 2, false>(M, K, N, hidden, weight, sa, s);
  return reg ? launch<KIND, 4, true>(M, K, N, hidden, weight, sa, s) : launch<KIND, 4, false>(M, K, N, hidden, weight, sa, s);
}

}  // namespace

// Measured on weights too many to stay in the last-level cache, against the tile kernels (split over
// K, two launches; gated: one workgroup per tile), microseconds at 8 / 16 / 32 tokens, K x rows:
//   3584 x 3584   8.9 / 9.3 / 12.1    16.3 / 16.2 / 16.2
//   3584 x 4608   13.1 / 14.9 / 21    17.4 / 16.8 / 16.6
//   18944 x 3584  28 / 33 / 42        45 / 45 / 45
//   18944 x 1024  21 / 26 / 34        25 / 25 / 25
//   3584 x 37888  46 / 49 / 56 (gated)   60 / 60 / 62
//   512 x 16384   9 / 10 / 15         12 / 12 / 12
//   8192 x 2048   12.4 / 13.8 / 17.2  19.5 / 19.3 / 19.3
// Up to 16 tokens everywhere; from 17 to 32 proj_mfma.hip compares it with proj_few.hip.
bool proj_stream_supports(int32_t M, int32_t K) {
  return M <= 32 && K % 64 == 0 && K / 64 >= kWaves && (int64_t)K * 64 < ((int64_t)1 << 31);
}
// 17 to 32 tokens where proj_few.hip has no division of the rows (more than 40960 of them, many short gated ones): what
// comes from memory in any case, from about 120 MB on (2048 x 24576, 32 tokens: 28 both; 3584 x 18432: 32 to 34 against
// 37 to 39), and, where K is not split, all but the shortest (2048 x 16384 gated: 22 against 31; 1024 x 32768: 25
// against 22).
bool proj_stream_pays(int32_t K, int32_t N, bool split) { return (int64_t)K * N >= 60 * 1000 * 1000 || (!split && K >= 2048); }

hipError_t launch_proj_stream(StreamKind kind, int32_t M, int32_t K, int32_t N, const void *hidden, const void *weight,
                              const StreamArgs &sa, hipStream_t s) {
  switch (kind) {
    case StreamKind::kRope: return dispatch<StreamKind::kRope>(M, K, N, hidden, weight, sa, s);
    case StreamKind::kGlu: return dispatch<StreamKind::kGlu>(M, K, N, hidden, weight, sa, s);
    default: return dispatch<StreamKind::kPlain>(M, K, N, hidden, weight, sa, s);
  }
}

}  // namespace hb
