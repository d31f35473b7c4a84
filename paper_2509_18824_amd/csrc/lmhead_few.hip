// LM head with fused argmax for up to 128 hidden rows, and for up to 256 where a workgroup then has one tile: a stream of
// the weight matrix (lmhead_mfma.hip, of which this is the arithmetic, has the rest).
//
// Every workgroup, one per CU, has a run of consecutive vocabulary rows for itself and takes it in tiles of up to 320 rows
// of equal height against one hidden tile.  The loads run on across its tiles, a lane keeps its best over all of them, and
// the wavefronts' bests meet in LDS once at the end: one atomic per hidden row and workgroup.
//
// What bounds it: memory, and the CU's path from L2 beside it.  A K step of 64 fetches 128 bytes of every weight row of
// the tile and of every hidden row, and with hidden rows that are always the same line 128 rows x 3584 x 152064 took 190 us
// where they took 211, 60 rows 171 and 186 (without matrix instructions 203 and 185): hence the tallest tile that LDS holds
// (128 rows: tiles of 304 against 208, 183 and 199 us), and all 256 CUs at work instead of the 200 that shared 594 tiles
// of 256 rows evenly.  us, tiles of 256 rows one by one and this: 152064 x 3584, 8 rows 172 -> 165, 60 186 -> 168,
// 128 210 -> 183; x 4096, 8 rows 230 -> 193, 128 247 -> 212; 100000 x 2048, 8 rows 95 -> 94; 32000 x 3584, 64 rows 58 -> 45; 64000 x 3584, 128
// rows, where both have the same tiles, 83 -> 84.
//
// All runs begin with K's first step.  Steps of their own would spread rows a multiple of 4 KB apart, which meet on few memory
// channels where everybody reads the same columns (100000 x 2048, 8 rows 94 and 68 us, 128 rows 101 and 79; 152064 x 4096 193 and
// 190, 212 and 201), but equal rows of different runs would no longer have equal logits, and the larger rounding would win
// instead of the lower id.
//
// Two wavefronts of a SIMD alternate between operands and matrix instructions as in mfma_gemm_tile.inc.
#include "mfma_gemm_tile.h"

namespace hb {

namespace {

constexpr int kBufferFlags = 0x00027000;  // untyped 32-bit elements
constexpr int kWaves = 8;
constexpr int kMostTall = 5;              // 64 vocabulary rows each, of a tile

// MT: 32-row hidden tiles of a wavefront, WT: its 16-row vocabulary tiles (4 x 2 wavefronts)
template <int MT, int WT>
struct Few {
  static constexpr int kRows = 64 * WT, kTok = 64 * MT;    // of a tile: vocabulary rows, hidden rows
  static constexpr int kW = kRows / 8 / kWaves, kH = kTok / 8 / kWaves;  // loads of a wavefront per K step
  static constexpr int kWStage = kRows * CH, kHStage = kTok * CH;        // 16-byte pieces
  // LDS stages of the weights and of the hidden rows: four where they fit (hidden rows one step ahead, in two stages, made
  // every step of a short tile wait: 128 rows x 3584 x 32000 58.0 us, with four 52.4; five or six the same or slower).  The tallest tile with 128 hidden rows has three and two.
  static constexpr int kFit = 160 / (8 * (WT + MT));
  static constexpr int kRing = kFit < 3 ? 3 : kFit < 4 ? kFit : 4, kHRing = kFit < 3 ? 2 : kRing;
  static constexpr bool kSame = kHRing == kRing;             // both tiles of a step are fetched together
  static constexpr size_t kLds = (size_t)(kRing * kWStage + kHRing * kHStage) * 16;
  static_assert(kLds <= 160 * 1024, "more LDS than a CU has");
};

// 16 bytes a lane from `offset` of `from`, plus `k_offset` inside its row, to LDS, lane after lane; from `bytes` on zeros
template <int HINT>
__device__ __forceinline__ void rows_to_lds(const u32x4 *from, int bytes, u32x4 *to, int offset, int k_offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)from, 0, bytes, kBufferFlags),
                                           (__attribute__((address_space(3))) void *)to, 16, offset, k_offset, 0, HINT);
}

// the largest key of the lanes l, l ^ 16, l ^ 32 and l ^ 48
__device__ __forceinline__ unsigned long long max_of_lane_groups(unsigned long long key) {
  typedef unsigned int swap2 __attribute__((ext_vector_type(2)));
  auto larger = [](swap2 hi, swap2 lo) {
    const unsigned long long a = ((unsigned long long)hi[0] << 32) | lo[0], b = ((unsigned long long)hi[1] << 32) | lo[1];
    return a > b ? a : b;
  };
  key = larger(__builtin_amdgcn_permlane16_swap((uint32_t)(key >> 32), (uint32_t)(key >> 32), false, false),
               __builtin_amdgcn_permlane16_swap((uint32_t)key, (uint32_t)key, false, false));
  return larger(__builtin_amdgcn_permlane32_swap((uint32_t)(key >> 32), (uint32_t)(key >> 32), false, false),
                __builtin_amdgcn_permlane32_swap((uint32_t)key, (uint32_t)key, false, false));
}

// ALONE: one hidden tile, nobody shares a workgroup's weights, which then carry the non-temporal hint.  Else the hidden
// tiles of a run are neighbours on one XCD.
template <int MT, int WT, bool ALONE>
__global__ __launch_bounds__(512) void lmhead_few_kernel(int M, int K, int V, int m_tiles, int own, int height,
                                                         const u32x4 *__restrict__ hidden, const u32x4 *__restrict__ weight,
                                                         unsigned long long *__restrict__ keys) {
  using F = Few<MT, WT>;
  constexpr int JT = 2 * MT;
  extern __shared__ u32x4 lds[];
  u32x4 *lw = lds, *lh = lds + F::kRing * F::kWStage;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave >> 1, wm = wave & 1;
  const int j16 = lane & 15, kq = lane >> 4;
  const int row_bytes = K * 2, k_steps = K / BK;
  const int slot = (int)blockIdx.x / kXcds;
  const int first = (slot / m_tiles * kXcds + (int)blockIdx.x % kXcds) * own, end = min(V, first + own);
  const int m0 = slot % m_tiles * F::kTok;
  if (first >= end) return;
  hidden += (size_t)m0 * (row_bytes / 16);
  const int m_rows = min(M - m0, F::kTok);

  // A load is eight rows of 128 bytes, pieces swizzled on the source side (lane -> row lane / 8); rows past the tile's or
  // past the hidden rows arrive as zeros.
  const int mine = (lane >> 3) * row_bytes + ((lane & 7) ^ (lane >> 3)) * 16;
  int w_off[F::kW], h_off[F::kH];
#pragma unroll
  for (int i = 0; i < F::kW; ++i) w_off[i] = (wave + kWaves * i) * 8 * row_bytes + mine;
#pragma unroll
  for (int i = 0; i < F::kH; ++i) h_off[i] = (wave + kWaves * i) * 8 * row_bytes + mine;
  int w_at = first, w_k = 0, h_k = 0;  // what is fetched next; past the last step that step again: the waits count loads
  auto issue_w = [&](int slot) {
    const u32x4 *from = weight + (size_t)w_at * (row_bytes / 16);
    const int bytes = __builtin_amdgcn_readfirstlane(min(height, end - w_at)) * row_bytes;
#pragma unroll
    for (int i = 0; i < F::kW; ++i) rows_to_lds<ALONE ? 2 : 0>(from, bytes, lw + slot * F::kWStage + (wave + kWaves * i) * 64, w_off[i], w_k * (BK * 2));
    if (++w_k == k_steps) {
      if (w_at + height < end) {
        w_at += height;
        w_k = 0;
      } else {
        --w_k;
      }
    }
  };
  auto issue_h = [&](int slot) {
#pragma unroll
    for (int i = 0; i < F::kH; ++i) rows_to_lds<0>(hidden, m_rows * row_bytes, lh + slot * F::kHStage + (wave + kWaves * i) * 64, h_off[i], h_k * (BK * 2));
    h_k = h_k + 1 == k_steps ? 0 : h_k + 1;
  };

  float best[JT];
  int best_v[JT];
#pragma unroll
  for (int j = 0; j < JT; ++j) {
    best[j] = -__builtin_huge_valf();
    best_v[j] = -1;
  }
  // Phases as in mfma_gemm_tile.inc, steps counted through all tiles: loads as far ahead as there are stages, less one.
  const bool late = wave >= kWaves / 2;
  int cur = 0, w_free = 0, h_slot = 0;
#pragma unroll
  for (int t = 0; t < F::kRing - 1; ++t) {
    if (t < F::kHRing - 1) issue_h(t);
    issue_w(t);
    ++w_free;
  }
  auto landed = [&] { asm volatile("s_waitcnt vmcnt(%0)" ::"n"((F::kRing - 2) * (F::kSame ? F::kW + F::kH : F::kW)) : "memory"); };
  auto phase = [&] { asm volatile("s_barrier" ::: "memory"); };
  landed();
  phase();
  if (late) {
    if (!F::kSame) issue_h(1);
    phase();
  }
#pragma unroll 1
  for (int v0 = first; v0 < end; v0 += height) {
    f32x4 acc[WT][JT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j = 0; j < JT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int kt = 0; kt < k_steps; ++kt) {
      const u32x4 *cw = lw + cur * F::kWStage, *chh = lh + (F::kSame ? cur : h_slot) * F::kHStage;
      bf16x8 a[2][WT], b[2][JT];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int c = s * 4 + kq;
#pragma unroll
        for (int i = 0; i < WT; ++i) a[s][i] = __builtin_bit_cast(bf16x8, cw[swz((wv * WT + i) * 16 + j16, c)]);
#pragma unroll
        for (int j = 0; j < JT; ++j) b[s][j] = __builtin_bit_cast(bf16x8, chh[swz((wm * JT + j) * 16 + j16, c)]);
      }
      if (F::kSame) issue_h(w_free);
      else if (!late) issue_h(h_slot ^ 1);
      issue_w(w_free);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int i = 0; i < WT; ++i) asm volatile("" : "+v"(a[s][i]));
#pragma unroll
        for (int j = 0; j < JT; ++j) asm volatile("" : "+v"(b[s][j]));
      }
      if (late) landed();
      phase();
      if (!F::kSame && late) issue_h(h_slot);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int jj = 0; jj < JT; ++jj) {
            const int j = (i & 1) ? JT - 1 - jj : jj;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s][i], b[s][j], acc[i][j], 0, 0, 0);
          }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (!late) landed();
      phase();
      cur = cur + 1 == F::kRing ? 0 : cur + 1;
      w_free = w_free + 1 == F::kRing ? 0 : w_free + 1;
      h_slot ^= 1;
    }
    // Scanning (tile, i, e) in order visits v in increasing order, so a strict '>' keeps the lowest v among equal values;
    // NaN compares false and never wins.
    const int v = v0 + wv * 16 * WT + 4 * kq, left = min(end, v0 + height) - v;
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      int at = -1;
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool take = i * 16 + e < left && acc[i][j][e] > best[j];
          best[j] = take ? acc[i][j][e] : best[j];
          at = take ? i * 16 + e : at;
        }
      best_v[j] = at < 0 ? best_v[j] : v + at;
    }
  }
  if (!late) phase();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // all loads have landed, all operands are read: LDS is free
  unsigned long long(*row_key)[F::kTok] = reinterpret_cast<unsigned long long(*)[F::kTok]>(lds);
#pragma unroll
  for (int j = 0; j < JT; ++j) {
    // a lane that saw nothing above -inf offers no candidate (key 0 loses to every real key)
    const unsigned long long key = max_of_lane_groups(best_v[j] >= 0 ? argmax_key(best[j], (uint32_t)best_v[j]) : 0ull);
    if (kq == 0) row_key[wv][(wm * JT + j) * 16 + j16] = key;
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m >= m_rows) return;
  unsigned long long key = row_key[0][m];
#pragma unroll
  for (int w = 1; w < 4; ++w) key = row_key[w][m] > key ? row_key[w][m] : key;
  // skip the atomic when the row already holds something at least as good
  if (key > __atomic_load_n(&keys[m0 + m], __ATOMIC_RELAXED)) atomicMax(&keys[m0 + m], key);
}

template <int MT, int WT>
hipError_t launch(int M, int K, int V, int m_tiles, int own, int height, const void *hidden, const void *weight, unsigned long long *keys, hipStream_t s) {
  using F = Few<MT, WT>;
  auto kern = m_tiles == 1 ? lmhead_few_kernel<MT, WT, true> : lmhead_few_kernel<MT, WT, false>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)F::kLds);
  if (e != hipSuccess) return e;
  const int groups = (V + own - 1) / own;
  kern<<<(groups + kXcds - 1) / kXcds * kXcds * m_tiles, 512, F::kLds, s>>>(M, K, V, m_tiles, own, height, (const u32x4 *)hidden, (const u32x4 *)weight, keys);
  return hipGetLastError();
}

}  // namespace

// How M hidden rows are tiled: 64 or 128 rows a tile; none where the tiles of lmhead_mfma.hip stay.  us by those, and by 64 and 128
// a tile here:
// - Up to 16384 vocabulary rows a workgroup reads mostly hidden rows, and two tiles of 64 over longer runs read the fewest: 64
//   rows x 4096 x 4096 53, 31 and 37, 128 rows 49, 30 and 37; x 12288 56, 33 and 37, 52, 37 and 39; 2048 x 16384 34, 25 and 28, 32, 26
//   and 28.  Long K beyond 12288 of them is taken by 128 for any number of rows (4096 x 16384, 64 rows 58, 36.5 and 39.4, 128 rows
//   58, 44 and 41.9): by 64 a tile 128 rows would take 1.15 times as long as 64, more than the 1.12 that few vocabulary rows are
//   held to.  Below K = 1024 a launch of 256 workgroups is most of it (64 rows x 4096: K 64 8.1 and 11.2, 512 13.2 and 14.9).
// - Up to 64 rows: from K = 640 on (64 rows, 32000: K 512 17.3 and 17.9, 768 21.5 and 20.2; 64000 26.8 and 27.8, which is the most
//   that is lost), where 256-row tiles are more than one round of CUs from 128 on (100000: K 64 17.8 and 19.0, 128 20.7 and 20.4, 512
//   30.5 and 28.7), and always where they are more than two (152000, K 64 21.6 and 20.1).
// - Up to 128 rows, by 128 a tile: one round of 256-row tiles from K = 1536 on (K 1024: 32000 23.6 and 25.4; 1536 32.0 and 31.3),
//   beyond it from 512 on (82000: K 256 25.4 and 25.8, 512 33.4 and 31.6), beyond two also for shorter K (152000, K 128 28.8 and 26.4).
// - Up to 256 rows: two hidden tiles of 128 where a run is one tile, from above K = 2048 on, where they are even (256 rows,
//   24576 x 4096 85 and 66, 32000 x 3584 81 and 72, x 1024 27.7 and 29.5; several tiles, 50000 x 3584, 94 and 118).
// Offsets inside a tile and the lengths of its buffers are 32 bits: 320 rows have to end below 2 GB.  Longer rows are the other
// kernel's, which has 64-bit addresses.
static int few_height(int M, int K, int V) {
  constexpr int kRound = 256 * TV;  // vocabulary rows of one round of the other kernel's tiles
  if (M > 256 || (int64_t)K * 2 * 64 * kMostTall >= (int64_t)1 << 31) return 0;
  if (V <= 16384) return M > 128 || K < 1024 ? 0 : V <= 12288 || K <= 2048 ? 64 : 128;
  if (M <= 64) return K >= (V > kRound ? 128 : 640) || V > 2 * kRound ? 64 : 0;
  if (M <= 128) return K >= (V > kRound ? 512 : 1536) || (V > 2 * kRound && K >= 128) ? 128 : 0;
  const int groups = 32 / ((M + 127) / 128) * kXcds, run = (V + groups - 1) / groups;
  return K > 2048 && run > 160 && run <= 64 * kMostTall ? 128 : 0;
}
bool lmhead_few_takes(int32_t M, int32_t K, int32_t V) { return few_height(M, K, V) != 0; }

hipError_t launch_lmhead_few(int32_t M, int32_t K, int32_t V, const void *hidden, const void *weight,
                             unsigned long long *keys, hipStream_t s) {
  const int rows = few_height(M, K, V);
  if (!rows) return hipErrorInvalidValue;
  const int m_tiles = (M + rows - 1) / rows, groups = 32 / m_tiles * kXcds;
  // Runs of several tiles in whole 16 rows (128 rows x 3584 x 152064, 608 a run 183 us, 594 185), of one tile as they come
  // (64000: 250 a run 77.0, 256 77.5).
  int own = (V + groups - 1) / groups;
  if (own > 64 * kMostTall) own = (own + 15) / 16 * 16;
  const int n = (own + 64 * kMostTall - 1) / (64 * kMostTall), height = ((own + n - 1) / n + 7) / 8 * 8;  // whole loads
#define HB_FEW(MT_, WT_) \
  case WT_: return launch<MT_, WT_>(M, K, V, m_tiles, own, height, hidden, weight, keys, s)
#define HB_FEW_ALL(MT_)       \
  switch ((height + 63) / 64) { \
    HB_FEW(MT_, 1);           \
    HB_FEW(MT_, 2);           \
    HB_FEW(MT_, 3);           \
    HB_FEW(MT_, 4);           \
    HB_FEW(MT_, 5);           \
    default: return hipErrorInvalidValue; \
  }
  if (rows == 64) HB_FEW_ALL(1);
  HB_FEW_ALL(2);
#undef HB_FEW_ALL
#undef HB_FEW
}

}  // namespace hb
