// Internal declarations shared by the translation units of libhb (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "hb.h"

namespace hb {

// thread-local error text behind hb_last_error()
int32_t fail(int32_t code, const char *fmt, ...);
int32_t fail_hip(hipError_t e, const char *what);

#define HB_HIP_TRY(expr)                                  \
  do {                                                    \
    hipError_t e__ = (expr);                              \
    if (e__ != hipSuccess) return ::hb::fail_hip(e__, #expr); \
  } while (0)

// ---- storage helpers --------------------------------------------------------------------
typedef uint16_t bf16_t;  // upper half of an IEEE float32

__host__ __device__ inline float bf16_to_f32(bf16_t x) {
  union { uint32_t u; float f; } c;
  c.u = (uint32_t)x << 16;
  return c.f;
}

// round to nearest even; NaN stays NaN (quiet)
__host__ __device__ inline bf16_t f32_to_bf16(float f) {
  union { uint32_t u; float f; } c;
  c.f = f;
  uint32_t u = c.u;
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x0040u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// two in one register, the first in the lower half
__device__ inline uint32_t pack_bf16(float a, float b) { return (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16); }

template <typename T> __device__ inline float load_f32(const T *p);
template <> __device__ inline float load_f32<float>(const float *p) { return *p; }
template <> __device__ inline float load_f32<bf16_t>(const bf16_t *p) { return bf16_to_f32(*p); }
template <typename T> __device__ inline void store_f32(T *p, float v);
template <> __device__ inline void store_f32<float>(float *p, float v) { *p = v; }
template <> __device__ inline void store_f32<bf16_t>(bf16_t *p, float v) { *p = f32_to_bf16(v); }

// ---- split-K plan -----------------------------------------------------------------------
// A sequence's prefix is cut into `splits` chunks of `chunk_tokens` tokens (a multiple of the
// page size and of the kernels' key tile).  Chunk 0 also takes the tree keys.  Partials of
// row R = node * Hq + head and chunk c live at  part_o[(R * splits + c) * D .. +D)  (fp32,
// un-normalised) and part_ml[(R * splits + c) * 2 .. +2) = (running max, running sum).
struct AttnPlan {
  int32_t splits;
  int32_t chunk_tokens;
  int32_t row_groups;  // MFMA kernel: workgroups that split the query rows of one (sequence, kv head, chunk)
  int32_t min_per;     // ... 64-key tiles that a worker takes at least
  int32_t workers;     // MFMA kernel: > 0 = work-proportional schedule with this many workers per kv head
  bool mfma;
  size_t ml_offset;  // byte offset of part_ml in the workspace
  size_t bytes;      // workspace size (0 when splits == 1)
};
int32_t make_attn_plan(const hb_attn_desc *d, AttnPlan *plan);  // validates shape fields

// 64-bit words that a kernel sets to zero on the way (0 words: none), for the launch after it.  Every thread calls it,
// with its place in the grid; a grid may have up to 2^32 - 1 threads in a dimension, so they are counted in 64 bits.
struct ClearArgs {
  unsigned long long *at;
  int32_t words;
};
__host__ __device__ inline void clear_words(const ClearArgs &c, uint32_t group, uint32_t groups, uint32_t thread, uint32_t threads) {
  for (int64_t i = (int64_t)group * threads + thread; i < c.words; i += (int64_t)groups * threads) c.at[i] = 0ull;
}

// ---- kernel launchers (each enqueues on `s`, returns a hipError_t from the launch) -------
hipError_t launch_attn_scalar(const hb_attn_desc &d, const AttnPlan &plan, const void *q,
                              const void *k_tree, const void *v_tree, const void *k_pool,
                              const void *v_pool, const int32_t *block_table,
                              const int32_t *prefix_len, const int32_t *node_offset,
                              const int32_t *parent, void *out, float *lse, float *part_o,
                              float *part_ml, ClearArgs clear, hipStream_t s);
hipError_t launch_attn_mfma(const hb_attn_desc &d, const AttnPlan &plan, const void *q,
                            const void *k_tree, const void *v_tree, const void *k_pool,
                            const void *v_pool, const int32_t *block_table,
                            const int32_t *prefix_len, const int32_t *node_offset,
                            const int32_t *parent, void *out, float *lse, float *part_o,
                            float *part_ml, ClearArgs clear, hipStream_t s);
bool attn_mfma_supports(const hb_attn_desc &d);
int32_t attn_mfma_row_groups(const hb_attn_desc &d);
int32_t attn_mfma_waves(const hb_attn_desc &d);  // wavefronts per workgroup (4 or 8)
hipError_t launch_attn_merge(const hb_attn_desc &d, const AttnPlan &plan, const float *part_o,
                             const float *part_ml, void *out, float *lse, hipStream_t s);

hipError_t launch_lmhead_scalar(int32_t dtype, int32_t M, int32_t K, int32_t V, const void *hidden,
                                const void *weight, unsigned long long *keys, hipStream_t s);
bool lmhead_few_takes(int32_t M, int32_t K, int32_t V);
hipError_t launch_lmhead_few(int32_t M, int32_t K, int32_t V, const void *hidden, const void *weight, unsigned long long *keys,
                             hipStream_t s);
hipError_t launch_lmhead_mfma(int32_t M, int32_t K, int32_t V, const void *hidden,
                              const void *weight, unsigned long long *keys, hipStream_t s);
bool lmhead_mfma_supports(int32_t dtype, int32_t M, int32_t K, int32_t V);
hipError_t launch_lmhead_init(unsigned long long *keys, int32_t M, hipStream_t s);
hipError_t launch_lmhead_finish(const unsigned long long *keys, int32_t M, int32_t V,
                                int32_t *out_ids, float *out_max, hipStream_t s);

// Few tokens (proj_stream.hip): N counts weight rows (for the gated projection gate and up rows together)
enum class StreamKind { kPlain, kRope, kGlu };
struct StreamArgs {
  const bf16_t *residual;  // plain: [M, N] or null
  bf16_t *out;             // plain [M, N], gated [M, N / 2]
  const bf16_t *bias;      // rotary: [N] or null
  const float *cos, *sin;  // [M, 64]
  bf16_t *q, *k, *v;       // [M, Hq, 128], [M, Hkv, 128], [M, Hkv, 128]
  int Hq, Hkv;
  // plain: the columns of K's second half, [M, K / 2] and [N, K / 2] beside a first half of the same shape, or null (both
  // operands in one piece)
  const bf16_t *hidden2, *weight2;
};
bool proj_stream_supports(int32_t M, int32_t K);
bool proj_stream_pays(int32_t K, int32_t N, bool split);  // against tiles of 256 rows (split: over K)
hipError_t launch_proj_stream(StreamKind kind, int32_t M, int32_t K, int32_t N, const void *hidden, const void *weight,
                              const StreamArgs &sa, hipStream_t s);

// 17 to 128 tokens (proj_few.hip): 16 `rows` weight rows a tile, K in `ks` parts (more than one: partial sums
// [part][token of m_pad][weight row of v_pad] to `part` instead of results); rows = 0: not taken
struct FewPlan {
  int32_t rows, ks;
};
// Rows and parts of K a multiple of 4 KB apart meet on few memory channels while everybody reads the same columns: there
// the workgroups begin at K steps of their own.  Few weights lose 1 to 2 % by it, since the tokens' columns are shared less
// (24 tokens, 6144 x 1216 9.52 and 9.68 us), from some 30 MB on they gain (2048 x 8576 12.9 -> 12.3); low tiles of rows an odd
// multiple of 4 KB apart do not (128 tokens, rotary 14336 x 3072 in seven parts 26.5 and 28.5).
inline bool few_turns(int32_t K, int32_t N, const FewPlan &p) {
  return K / p.ks % 2048 == 0 && (p.ks == 1 || K % 4096 == 0 || p.rows >= 8) && (int64_t)K * N >= 15000000;
}
hipError_t launch_proj_few(StreamKind kind, const FewPlan &p, int32_t M, int32_t K, int32_t N, const void *hidden,
                           const void *weight, const StreamArgs &sa, float *part, int32_t v_pad, int32_t m_pad, hipStream_t s);

// Tiles of 32 it weight rows x 32 jt tokens whose K steps two groups of wavefronts share (proj_pair.hip), K in `ks`
// parts (more than one: partial sums as above); it = 0: not taken
struct PairPlan {
  int32_t it, jt, ks;
};
hipError_t launch_proj_pair(StreamKind kind, const PairPlan &p, int32_t M, int32_t K, int32_t N, const void *hidden,
                            const void *weight, const StreamArgs &sa, float *part, int32_t v_pad, int32_t m_pad, hipStream_t s);

bool proj_mfma_supports(int32_t M, int32_t K, int32_t N);
// part: fp32 scratch of proj_workspace_bytes(M, K, N) bytes, for the ways that split K, or null (then K stays whole)
size_t proj_workspace_bytes(int32_t M, int32_t K, int32_t N);
hipError_t launch_qkv_rope(int32_t M, int32_t K, int32_t Hq, int32_t Hkv, const void *hidden, const void *w_qkv,
                           const void *bias, const float *cos, const float *sin, void *q, void *k, void *v,
                           float *part, hipStream_t s);
hipError_t launch_linear(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *residual,
                         void *out, float *part, hipStream_t s);
// ... and the rows of out, normalised by root mean square, to norm_out
hipError_t launch_linear_norm(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *residual,
                              void *out, const void *norm_weight, float eps, void *norm_out, float *part, hipStream_t s);
// out = x w^T + x2 w2^T (tmp [M, N] is used where that takes two products); part2: scratch for (M, 2 K, N), part for (M, K, N)
hipError_t launch_linear_two(int32_t M, int32_t K, int32_t N, const void *x, const void *w, const void *x2, const void *w2,
                             void *tmp, void *out, float *part, float *part2, hipStream_t s);
hipError_t launch_swiglu(int32_t M, int32_t K, int32_t F, const void *x, const void *w_gate_up, void *out, float *part,
                         hipStream_t s);
hipError_t launch_rmsnorm(int32_t T, int32_t K, const void *x, const void *weight, float eps, void *out, hipStream_t s);
hipError_t launch_tree_positions(int32_t B, int32_t max_nodes, int32_t total_nodes, const int32_t *node_offset,
                                 const int32_t *parent, const int32_t *prefix_len, int32_t *positions, hipStream_t s);
hipError_t launch_rope_table(int32_t T, int32_t half, double theta, const int32_t *positions, float *cos, float *sin,
                             hipStream_t s);

hipError_t launch_tree_accept(int32_t B, int32_t max_nodes, const int32_t *node_offset,
                              const int32_t *parent, const int32_t *draft_ids,
                              const int32_t *target_ids, const int32_t *prev_target, int32_t max_path,
                              int32_t *accept_len, int32_t *accept_path, int32_t *out_tokens,
                              int32_t *bonus_id, hipStream_t s);
hipError_t launch_tree_accept_sample(int32_t B, int32_t max_nodes, int32_t V, const int32_t *node_offset,
                                     const int32_t *parent, const int32_t *draft_ids, const float *p_target,
                                     const float *q_draft, const uint32_t *u_accept, const uint32_t *u_bonus,
                                     int32_t max_path, int32_t *accept_len, int32_t *accept_path,
                                     int32_t *out_tokens, int32_t *bonus_id, uint32_t *work, int32_t polls, hipStream_t s);
size_t topk_workspace_bytes(int32_t M, int32_t V, int32_t k);
hipError_t launch_topk_logprob(int32_t dtype, int32_t M, int32_t V, int32_t k, const void *logits, int32_t *out_ids,
                               float *out_logp, void *work, hipStream_t s);
hipError_t launch_tree_grow(int32_t B, int32_t K, int32_t level, int32_t C, const int32_t *child_ids,
                            const float *child_logp, float *cand_score, int32_t *cand_token, int32_t *cand_parent,
                            int32_t *frontier, int32_t *frontier_slot, hipStream_t s);
hipError_t launch_tree_finalize(int32_t B, int32_t C, int32_t n, const float *cand_score, const int32_t *cand_token,
                                const int32_t *cand_parent, const int32_t *root_token, int32_t *node_offset,
                                int32_t *parent, int32_t *draft_ids, int32_t *depth, unsigned long long *anc,
                                int32_t *node_cand, float *node_score, hipStream_t s);
int32_t meta_rows_pad(int32_t H, int32_t Q);
hipError_t launch_meta_fold(int32_t Q, int32_t D, int32_t H, const void *f_q, const void *w_q, const void *w_k,
                            void *a_fold, float *qproj, hipStream_t s);
hipError_t launch_meta_attn(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, const void *feats, const void *v_proj,
                            const void *a_fold, const int32_t *residual_layers, void *pre, void *res_out,
                            float *part, hipStream_t s);
bool meta_project_supports(int32_t D, int32_t H);
bool meta_project_pays(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q);
size_t meta_project_workspace_bytes(int32_t S, int32_t D, int32_t H, int32_t Q);
size_t meta_project_least_bytes(int32_t S, int32_t D, int32_t H, int32_t Q);  // less is refused
hipError_t launch_meta_attn_project(int32_t S, int32_t L, int32_t D, int32_t H, int32_t Q, const void *feats,
                                    const void *a_fold, const void *w_v, const int32_t *residual_layers, void *pre,
                                    void *res_out, float *part, size_t part_bytes, hipStream_t s);
size_t meta_attn_workspace_bytes(int32_t S, int32_t D, int32_t H, int32_t Q);
hipError_t launch_kv_compact(const hb_attn_desc &d, const void *k_tree, const void *v_tree,
                             void *k_pool, void *v_pool, const int32_t *block_table,
                             const int32_t *prefix_len, const int32_t *node_offset,
                             const int32_t *accept_len, const int32_t *accept_path,
                             int32_t max_path, int32_t *out_slots, int32_t *new_len, hipStream_t s);

hipError_t launch_kv_compact_layers(const hb_attn_desc &d, int32_t n_layers, const void *const *k_tree,
                                    const void *const *v_tree, void *const *k_pool, void *const *v_pool,
                                    const int32_t *block_table, const int32_t *prefix_len,
                                    const int32_t *node_offset, const int32_t *accept_len,
                                    const int32_t *accept_path, int32_t max_path, int32_t *out_slots,
                                    int32_t *new_len, hipStream_t s);

// LM head's keys -> ids, greedy acceptance and the append to `layers` layers (0: no append); the K/V tensors are
// given themselves, or tables of their device addresses, one per layer
struct TailArgs {
  const unsigned long long *keys;
  int32_t M, V, max_path, layers, row_bytes, path_slots;  // the last two are the launcher's
  bool tables;
  const int32_t *node_offset, *parent, *draft_ids, *block_table, *prefix_len;
  const void *k_tree, *v_tree;
  void *k_pool, *v_pool;
  int32_t *target_ids, *accept_len, *accept_path, *out_tokens, *bonus_id, *out_slots, *new_len;
};
hipError_t launch_verify_tail(const hb_attn_desc &d, TailArgs t, hipStream_t s);

// ---- argmax key: (order-preserving float bits << 32) | (0xffffffff - index) ---------------
// max over keys = largest value, lowest index among equal values.  NaN is mapped to -inf.
__device__ inline unsigned long long argmax_key(float v, uint32_t idx) {
  if (!(v == v)) v = -__builtin_huge_valf();
  uint32_t u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (unsigned long long)(0xffffffffu - idx);
}
__device__ inline float argmax_key_value(unsigned long long key) {
  uint32_t u = (uint32_t)(key >> 32);
  u = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
  return __uint_as_float(u);
}
__device__ inline uint32_t argmax_key_index(unsigned long long key) {
  return 0xffffffffu - (uint32_t)(key & 0xffffffffull);
}
// the id a key stands for; a row that saw nothing above -inf (key 0) names token 0
__device__ inline int32_t argmax_key_id(unsigned long long key, int32_t V) {
  const uint32_t idx = key ? argmax_key_index(key) : 0u;
  return idx < (uint32_t)V ? (int32_t)idx : 0;
}

}  // namespace hb
