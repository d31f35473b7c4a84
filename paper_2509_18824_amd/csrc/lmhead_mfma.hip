// LM head with fused argmax on the bf16 matrix cores of gfx950.
//
// Computes C^T[v, m] = sum_k W[v, k] * H[m, k] tile by tile and never stores it: the weight
// rows are the MFMA "A" operand and the hidden rows the "B" operand, so that one lane's
// accumulators of a 16x16 tile all belong to ONE hidden row m and four different vocabulary
// entries v.  The row-wise argmax is then an in-register scan, two exchanges between the four
// lane groups, and one 64-bit atomic max per (row, workgroup).
//
// Workgroup: 512 threads = 8 wavefronts (two per SIMD) in a 4 (v) x 2 (m) arrangement; workgroup
// tile TV = 256 vocabulary rows x TM = 64 * MT hidden rows, K step 64.  Both operands are
// K-contiguous in memory ([V, K] and [M, K] row-major), which is exactly what the MFMA operand
// layout wants (8 consecutive k per lane), so tiles go global -> LDS directly as 16-byte pieces
// (global_load_lds), XOR-swizzled so that the 16-byte operand reads of 8 consecutive rows hit
// all banks.  Weight tiles sit in a ring of three LDS stages and are fetched two K steps ahead,
// hidden tiles in two stages one step ahead (64 rows: in three, two steps ahead); the two wavefronts of a
// SIMD alternate between reading operands and matrix instructions (see mfma_gemm_tile.inc).
//
// What bounds the kernel at many rows is power (see there): 960 x 3584 x 152064 on normal values 876 ->
// 826 us, 1024 rows 940 -> 839, 768 rows 752 -> 667 against 32x32x16 with one barrier per K step.
// Workgroups go in lockstep so that shared tiles are fetched from HBM once.
//
// Up to 128 rows (but for short K), and some calls of up to 256, go to lmhead_few.hip.  A row's sum over K
// has the same order there, in every tile and for any number of hidden rows: equal rows have equal logits, so that the lowest
// id of several wins, and a token's logits do not depend on the tokens beside it.
//
// Grid: persistent workgroups, one per CU, in groups that walk the vocabulary tiles in lockstep
// (one hidden tile per member) on one XCD.
#include "mfma_gemm_tile.h"

namespace hb {

namespace {

// MT: 32-row hidden tiles per wavefront (the workgroup covers TM = 64 * MT hidden rows).
// WNT: weight loads carry the non-temporal hint.  With one hidden tile nobody shares a weight
// tile, and streaming it through L2 without displacing the hidden rows is worth 5 % (64 rows x 512 to
// 960 x 4096 to 16384 1 to 5 %); with several
// hidden tiles the hint evicts weight lines before all sharers have read them.
template <int MT, bool WNT>
__global__ __launch_bounds__(512) void lmhead_mfma_kernel(int M, int K, int V, int m_tiles, int v_tiles, int groups, int spare, int spare_tiles,
                                                          const u32x4 *__restrict__ hidden,
                                                          const u32x4 *__restrict__ weight,
                                                          unsigned long long *__restrict__ keys) {
  constexpr int TM = 64 * MT;
  constexpr int NT = 512;                  // threads
  constexpr int WV = 4;                    // wavefront rows along the vocabulary
  extern __shared__ u32x4 lds[];           // [3][TV*CH] weight, then [kHiddenStages][TM*CH] hidden
  u32x4 *lw = lds;
  u32x4 *lh = lds + 3 * TV * CH;
  // per-row candidates of the epilogue; reuses the weight stages once the K loop is over
  unsigned long long (*row_key)[TM] = reinterpret_cast<unsigned long long (*)[TM]>(lds);
  static_assert(WV * TM * 8 <= 3 * TV * CH * 16, "row_key fits in the weight stages");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wv = wave >> 1;  // which 64 vocabulary rows of the tile
  const int wm = wave & 1;   // which 32*MT hidden rows of the tile

  // Persistent workgroups in lockstep groups.  Workgroup ids go round-robin to the XCDs
  // (id % 8); on each XCD the grid places `groups` groups of m_tiles workgroups, one workgroup
  // per CU.  The workgroups of a group take the same sequence of vocabulary tiles, one hidden
  // tile each; having identical work they advance together, so the weight tile they share is
  // fetched from HBM once and found in the XCD's L2 by the others, and the groups of an XCD read
  // the same K range of the hidden rows at about the same time.
  // When the groups do not fill the XCD's CUs, the `spare` remaining workgroups of each XCD take
  // the XCD's first `spare_tiles` vocabulary tiles off the groups' hands, as units of one
  // (vocabulary tile, hidden tile) pair dealt round-robin, so that the groups need one round
  // fewer; consecutive units share the weight tile, which the spare workgroups therefore read at
  // about the same time.
  const int id = blockIdx.x;
  const int xcd = id % kXcds;
  const int slot = id / kXcds;
  const int in_group = groups * m_tiles;
  const bool is_spare = slot >= in_group;
  const int kp = K / 8;  // 16-byte pieces per matrix row (K % 8 == 0)
#pragma unroll 1
  for (int it = 0;; ++it) {
  int nth, m_tile;  // the XCD's nth vocabulary tile against hidden tile m_tile
  if (!is_spare) {
    nth = spare_tiles + slot / m_tiles + it * groups;
    m_tile = slot % m_tiles;
  } else {
    const int unit = slot - in_group + it * spare;
    if (unit >= spare_tiles * m_tiles) break;
    nth = unit / m_tiles;
    m_tile = unit - nth * m_tiles;
  }
  const int v_tile = nth * kXcds + xcd;
  if (v_tile >= v_tiles) break;
  const int m0 = m_tile * TM;
  const int v0 = v_tile * TV;

#define HB_GEMM_W_ROW(t_) (v0 + (t_))
#include "mfma_gemm_tile.inc"
#undef HB_GEMM_W_ROW

  // Epilogue.  Accumulator e of lane l in tile (i, j) is C^T[v, m] with
  //   v = v0 + wv*64 + i*16 + 4*(l/16) + e,   m = m0 + wm*32*MT + j*16 + l%16.
  // Scanning (i, e) in order visits v in increasing order, so a strict '>' keeps the lowest v
  // among equal values; NaN compares false and never wins.
#pragma unroll
  for (int j = 0; j < JT; ++j) {
    float best = -__builtin_huge_valf();
    int best_v = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int v = v0 + wv * 64 + i * 16 + 4 * frag_k + e;
        float x = acc[i][j][e];
        bool take = (v < V) && (x > best);
        best = take ? x : best;
        best_v = take ? v : best_v;
      }
    // a lane that saw nothing above -inf offers no candidate (key 0 loses to every real key)
    unsigned long long key = best_v >= 0 ? argmax_key(best, (uint32_t)best_v) : 0ull;
    unsigned long long other = __shfl_xor(key, 16, 64);
    key = other > key ? other : key;
    other = __shfl_xor(key, 32, 64);
    key = other > key ? other : key;
    if (lane < 16) row_key[wv][wm * 32 * MT + j * 16 + lane] = key;
  }
  __syncthreads();
  for (int r = tid; r < TM; r += NT) {
    int m = m0 + r;
    if (m >= M) continue;
    unsigned long long key = row_key[0][r];
#pragma unroll
    for (int w = 1; w < WV; ++w) key = row_key[w][r] > key ? row_key[w][r] : key;
    // skip the atomic when the row already holds something at least as good
    if (key > __atomic_load_n(&keys[m], __ATOMIC_RELAXED)) atomicMax(&keys[m], key);
  }
  __syncthreads();  // row_key shares LDS with the stages the next vocabulary tile fills
  }  // vocabulary tiles of this workgroup
}

// How the workgroups of an XCD share v_tiles / 8 vocabulary tiles against m_tiles hidden tiles.
struct Shares {
  int groups, spare, spare_tiles, rounds;
};
Shares share_tiles(int m_tiles, int v_tiles) {
  // groups per XCD: at most as many as its 32 CUs hold with one workgroup per CU; then the
  // fewest that still need the same number of rounds, so that every group gets the same number
  // of vocabulary tiles (594 tiles of one hidden tile: 25 groups x 3 rounds per XCD instead of 32
  // groups of which a third work a round longer)
  int max_groups = 32 / m_tiles;
  if (max_groups < 1) max_groups = 1;
  const int need = (v_tiles + kXcds - 1) / kXcds, rounds = (need + max_groups - 1) / max_groups;
  Shares sh = {(need + rounds - 1) / rounds, 0, 0, rounds};
  // CUs of an XCD that no group occupies: if handing them a few vocabulary tiles (every XCD has
  // at least v_tiles / 8) saves the groups a round, do so (960 rows = 5 hidden tiles: 6 groups
  // on 30 CUs would need 13 rounds for 75 tiles; with 3 tiles on the 2 other CUs, 15 units in 8
  // rounds, they need 12).  The fewest tiles that reach the best round count are handed over.
  if (m_tiles <= 32) {
    const int left = 32 - max_groups * m_tiles;
    for (int y = 1; left > 0 && y <= v_tiles / kXcds; ++y) {
      const int full = (need - y + max_groups - 1) / max_groups;
      const int mine = (y * m_tiles + left - 1) / left;
      const int cost = full > mine ? full : mine;
      if (cost < sh.rounds) sh = {max_groups, left, y, cost};
    }
  }
  return sh;
}

template <int MT, bool WNT>
hipError_t launch(int M, int K, int V, const void *hidden, const void *weight, unsigned long long *keys,
                  hipStream_t s) {
  constexpr int TM = 64 * MT;
  const int m_tiles = (M + TM - 1) / TM, v_tiles = (V + TV - 1) / TV;
  const Shares sh = share_tiles(m_tiles, v_tiles);
  size_t lds_bytes = tile_lds_bytes(MT);
  auto kern = lmhead_mfma_kernel<MT, WNT>;
  hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)((sh.groups * m_tiles + sh.spare) * kXcds));
  kern<<<grid, 512, lds_bytes, s>>>(M, K, V, m_tiles, v_tiles, sh.groups, sh.spare, sh.spare_tiles, (const u32x4 *)hidden, (const u32x4 *)weight, keys);
  return hipGetLastError();
}

}  // namespace

bool lmhead_mfma_supports(int32_t dtype, int32_t M, int32_t K, int32_t V) {
  return dtype == HB_BF16 && K % BK == 0 && M >= 1 && V >= 1;  // other K: the scalar kernel
}

hipError_t launch_lmhead_mfma(int32_t M, int32_t K, int32_t V, const void *hidden, const void *weight,
                              unsigned long long *keys, hipStream_t s) {
  if (lmhead_few_takes(M, K, V)) return launch_lmhead_few(M, K, V, hidden, weight, keys, s);
  // Hidden tile height: rounds of a vocabulary tile by what one takes (us a round of 56 K steps, 500 to 1000 rows x 3584 x
  // 152064: 40, 53, 68 and 83 for 64 to 256 hidden rows; on few CUs a tile waits for its own K steps, and a lower one is
  // ahead there too).  The fewest padded rows, which chose before, gave 257 to 320, 385 to 448, 641 to 704 and 769 to 832 rows
  // tiles of 64, many to a vocabulary tile (us, so and by rounds: 320 x 3584 x 152064 519 and 371, 400 683 and 446, 700 1050 and
  // 662, 800 1218 and 813, 880 893 and 813; 700 x 4096 x 32000 262 and 164).  Equal rounds: the fewest padded rows.
  // Rows that fit one tile stay in it once two would go round more than once: rounds beyond the first wait for the weights,
  // and one tile reads them once a CU (227 x 4096 x 69031: two of 128 193, one 166; 237 x 3584 x 96490 193 and 176; within the
  // round two are ahead, 203 x 2048 x 20148 38 and 47).
  static const int kRound[5] = {0, 40, 53, 68, 83};
  const int v_tiles = (V + TV - 1) / TV;
  int best_mt = 4;
  long best = -1;
  for (int mt = 4; mt >= 1; --mt) {
    const int m_tiles = (M + 64 * mt - 1) / (64 * mt);
    if (M <= 256 && m_tiles > 1 && v_tiles > 32 / 2 * kXcds) continue;
    const long us = (long)share_tiles(m_tiles, v_tiles).rounds * ((m_tiles + 31) / 32) * kRound[mt];
    const long cost = us * 1000000 + (long)m_tiles * 64 * mt;
    if (best < 0 || cost < best) {
      best = cost;
      best_mt = mt;
    }
  }
  switch (best_mt) {
    case 1: return M <= 64 * 1 ? launch<1, true>(M, K, V, hidden, weight, keys, s)
                            : launch<1, false>(M, K, V, hidden, weight, keys, s);
    case 2: return M <= 64 * 2 ? launch<2, true>(M, K, V, hidden, weight, keys, s)
                            : launch<2, false>(M, K, V, hidden, weight, keys, s);
    case 3: return M <= 64 * 3 ? launch<3, true>(M, K, V, hidden, weight, keys, s)
                            : launch<3, false>(M, K, V, hidden, weight, keys, s);
    default: return M <= 64 * 4 ? launch<4, true>(M, K, V, hidden, weight, keys, s)
                            : launch<4, false>(M, K, V, hidden, weight, keys, s);
  }
}

}  // namespace hb
