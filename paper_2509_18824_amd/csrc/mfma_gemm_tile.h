// What the kernels that include mfma_gemm_tile.inc share with it: the tile's sizes and its layout in LDS.
#pragma once
#include "hb_internal.h"

namespace hb {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;           // k per step
constexpr int TV = 256;          // weight rows per workgroup
constexpr int CH = BK / 8;       // 16-byte pieces per row per step (8)
constexpr int kXcds = 8;

// Hidden tile stages in LDS.  With 64 rows three: 7 rows x 3584 x 152064 through this loop 169.9 us (176.6 with two); with
// 128 two: 128 rows 204 us (209 with three).  More do not fit.  (The LM head of so few rows now has
// lmhead_few.hip's loop, but for short K.)
constexpr int kHiddenStages(int mt) { return mt == 1 ? 3 : 2; }
constexpr size_t tile_lds_bytes(int mt) { return (size_t)(3 * TV + kHiddenStages(mt) * 64 * mt) * CH * 16; }

// Offset (in 16-byte pieces) of piece `c` of row `r` in a swizzled [rows][8] tile.  Rows are
// 128 bytes; the XOR spreads one logical piece of 8 consecutive rows over distinct 16-byte bank
// groups.  The operand reads of 16x16x32 (lane l: row l % 16, piece l / 16) then run at 256 bytes
// a clock; with row bit 3 in the XOR as well, as 32x32x16 wants it, at 128.
__device__ inline int swz(int r, int c) { return r * CH + (c ^ (r & 7)); }

}  // namespace

}  // namespace hb
