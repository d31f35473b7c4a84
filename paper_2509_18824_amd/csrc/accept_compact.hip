// Greedy longest-accepted-path selection and KV compaction.
//
// Acceptance: one wavefront per sequence, one lane per tree node (at most 64 nodes).  Each lane
// walks to the root once to collect its ancestor set as a 64-bit mask; a wave ballot of the
// per-node match flags then tells every lane at once whether its whole path matches.
// Compaction: one workgroup per (path slot, sequence) copies that node's K and V rows into the
// page slot that follows the prefix, in 16-byte pieces.
#include "hb_internal.h"

namespace hb {

namespace {

// Acceptance of one tree by one wavefront, lane = node (live: it exists).  par: parent node or anything below 0;
// tgt: the target's token after the node; match_root: the root counts as accepted.  Every lane gets the same result
// but anc, its ancestors and itself.
struct Accepted {
  int len;                  // nodes on the accepted path; 0: not even the root
  int target;               // the target's token after the last of them
  unsigned long long path;  // the nodes on it, a bit each
};
__device__ __forceinline__ Accepted accept_wave(int lane, bool live, int par, int did, int tgt, bool match_root, int max_path) {
  if (!live || par >= lane || par < -1 || lane == 0) par = -1;  // malformed: treat as a root-like node
  // ancestor set (self included) and whether this node's own id matches its parent's target
  unsigned long long anc = live ? (1ull << lane) : 0ull;
  for (int x = par; __any(x >= 0);) {  // parents precede their children: at most 63 steps
    const int up = __shfl(par, x < 0 ? 0 : x, 64);
    if (x >= 0) {
      anc |= 1ull << x;
      x = up;
    }
  }
  const bool rooted = live && (anc & 1ull);  // a path that does not reach node 0 is never accepted
  const int par_target = __shfl(tgt, par < 0 ? 0 : par, 64);
  const bool match = live && (lane == 0 ? match_root : did == par_target);
  const unsigned long long match_mask = __ballot(match);
  const int depth = __popcll(anc) - 1;
  const bool accepted = rooted && ((anc & ~match_mask) == 0ull) && depth < max_path;
  // deepest accepted node, lowest id among equals: maximise depth * 64 + (63 - lane)
  int key = accepted ? depth * 64 + (63 - lane) : -1;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) key = max(key, __shfl_xor(key, off, 64));
  if (key < 0) return {0, -1, 0ull};
  const int best = 63 - (key & 63);
  return {(key >> 6) + 1, __shfl(tgt, best, 64), (unsigned long long)__shfl((long long)anc, best, 64)};
}

// What a sequence's wavefront writes; bonus_if_none: no node accepted (no nodes at all, or a rejected root), so that
// nothing is emitted and the pending token stays what it was.
__device__ __forceinline__ void store_accepted(const Accepted &a, int lane, int did, int bonus_if_none, int b, int max_path,
                                               int32_t *__restrict__ accept_len, int32_t *__restrict__ accept_path,
                                               int32_t *__restrict__ out_tokens, int32_t *__restrict__ bonus_id) {
  int32_t *path = accept_path + (size_t)b * max_path, *tokens = out_tokens + (size_t)b * max_path;
  if ((a.path >> lane) & 1ull) {
    const int rank = __popcll(a.path & ((1ull << lane) - 1ull));
    path[rank] = lane;
    if (rank >= 1) tokens[rank - 1] = did;
  }
  for (int j = a.len + lane; j < max_path; j += 64) path[j] = tokens[j] = -1;
  if (lane == 0) {
    if (a.len) tokens[a.len - 1] = a.target;
    accept_len[b] = a.len;
    bonus_id[b] = a.len ? a.target : bonus_if_none;
  }
}

__global__ __launch_bounds__(64) void tree_accept_kernel(
    int max_nodes, const int32_t *__restrict__ node_offset, const int32_t *__restrict__ parent,
    const int32_t *__restrict__ draft_ids, const int32_t *__restrict__ target_ids,
    const int32_t *__restrict__ prev_target, int max_path, int32_t *__restrict__ accept_len, int32_t *__restrict__ accept_path, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ bonus_id) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int n0 = node_offset[b];
  int n = node_offset[b + 1] - n0;
  n = n < 0 ? 0 : (n > max_nodes ? max_nodes : n);
  const bool live = lane < n;
  int par = -1, did = 0, tgt = 0;
  if (live) {
    par = parent[n0 + lane];
    did = draft_ids[n0 + lane];
    tgt = target_ids[n0 + lane];
  }
  // the root is the pending committed token (always a match) unless the caller names the token
  // the target chose last step: then the root is a guess like any other node
  const int prev = prev_target ? prev_target[b] : -1;
  const Accepted a = accept_wave(lane, live, par, did, tgt, !prev_target || did == prev, max_path);
  store_accepted(a, lane, did, prev, b, max_path, accept_len, accept_path, out_tokens, bonus_id);
}

// path slot j of sequence b, of one layer: the path has len nodes, node the j-th (looked at if j < len);
// out_slots / new_len are written when given
__device__ __forceinline__ void compact_one(
    const hb_attn_desc &d, int row_bytes, int j, int b, int len, int node, const uint4 *__restrict__ k_tree,
    const uint4 *__restrict__ v_tree, uint4 *__restrict__ k_pool, uint4 *__restrict__ v_pool,
    const int32_t *__restrict__ block_table, const int32_t *__restrict__ prefix_len,
    const int32_t *__restrict__ node_offset, int max_path, int32_t *__restrict__ out_slots, int32_t *__restrict__ new_len) {
  len = len < 0 ? 0 : (len > max_path ? max_path : len);
  int L = prefix_len[b];
  L = L < 0 ? 0 : L;
  if (j == 0 && threadIdx.x == 0 && new_len) new_len[b] = L + len;
  const long long p = (long long)L + j;
  const bool in_table = p < (long long)d.max_blocks_per_seq * d.page_size;
  if (j >= len || !in_table) {
    if (threadIdx.x == 0 && out_slots) out_slots[(size_t)b * max_path + j] = -1;
    return;
  }
  const int n0 = node_offset[b];
  int n = node_offset[b + 1] - n0;
  node = node < 0 ? 0 : (node >= n ? n - 1 : node);
  int src = n0 + node;
  src = src < 0 ? 0 : (src >= d.total_nodes ? d.total_nodes - 1 : src);
  int blk = block_table[(size_t)b * d.max_blocks_per_seq + (int)(p / d.page_size)];
  blk = blk < 0 ? 0 : (blk >= d.num_blocks ? d.num_blocks - 1 : blk);
  const int off = (int)(p % d.page_size);
  if (threadIdx.x == 0 && out_slots) out_slots[(size_t)b * max_path + j] = blk * d.page_size + off;
  const int vec_per_row = row_bytes / 16;  // 16-byte pieces of one head's row
  for (int t = threadIdx.x; t < d.num_kv_heads * vec_per_row; t += blockDim.x) {
    int h = t / vec_per_row, w = t - h * vec_per_row;
    size_t s_idx = ((size_t)src * d.num_kv_heads + h) * vec_per_row + w;
    size_t d_idx = (((size_t)blk * d.num_kv_heads + h) * d.page_size + off) * vec_per_row + w;
    k_pool[d_idx] = k_tree[s_idx];
    v_pool[d_idx] = v_tree[s_idx];
  }
}

__global__ __launch_bounds__(256) void kv_compact_kernel(
    hb_attn_desc d, int row_bytes, const uint4 *__restrict__ k_tree, const uint4 *__restrict__ v_tree,
    uint4 *__restrict__ k_pool, uint4 *__restrict__ v_pool, const int32_t *__restrict__ block_table,
    const int32_t *__restrict__ prefix_len, const int32_t *__restrict__ node_offset,
    const int32_t *__restrict__ accept_len, const int32_t *__restrict__ accept_path, int max_path,
    int32_t *__restrict__ out_slots, int32_t *__restrict__ new_len) {
  const int j = blockIdx.x, b = blockIdx.y;
  compact_one(d, row_bytes, j, b, accept_len[b], accept_path[(size_t)b * max_path + j], k_tree, v_tree, k_pool, v_pool,
              block_table, prefix_len, node_offset, max_path, out_slots, new_len);
}

// all layers in one launch: blockIdx.z = layer, its tensors from tables of device pointers
__global__ __launch_bounds__(256) void kv_compact_layers_kernel(
    hb_attn_desc d, int row_bytes, const uint4 *const *__restrict__ k_tree, const uint4 *const *__restrict__ v_tree,
    uint4 *const *__restrict__ k_pool, uint4 *const *__restrict__ v_pool, const int32_t *__restrict__ block_table,
    const int32_t *__restrict__ prefix_len, const int32_t *__restrict__ node_offset,
    const int32_t *__restrict__ accept_len, const int32_t *__restrict__ accept_path, int max_path,
    int32_t *__restrict__ out_slots, int32_t *__restrict__ new_len) {
  const int j = blockIdx.x, b = blockIdx.y, l = blockIdx.z;
  compact_one(d, row_bytes, j, b, accept_len[b], accept_path[(size_t)b * max_path + j], k_tree[l], v_tree[l], k_pool[l],
              v_pool[l], block_table, prefix_len, node_offset, max_path, l == 0 ? out_slots : nullptr, l == 0 ? new_len : nullptr);
}

// What follows the LM head, in one launch: the ids of all rows from their keys, acceptance, the append of the
// accepted nodes.  Each of these is a chain of two or three memory round trips; as launches of their own (and one
// more to clear the keys, which the attention kernel now does) they took 1.5 us each of the GPU's time in a full
// stream and the host's of two calls: step of one 60-node tree 214.9 -> 210.3 us, 16 chains of 8 nodes 239.8 -> 234.8,
// four nodes of a unit-sized float32 model 31.1 -> 20.3.  A workgroup per (path slot that a tree's nodes can fill,
// sequence, layer); its first wavefront works the sequence's acceptance out
// by itself (a key, a parent and a drafted token per lane), which is cheaper than to wait for anybody.  The first workgroup
// of a sequence writes the results; the ids are dealt to all workgroups.
// MANY: more of them than the grid has workgroups (a kernel of its own: the loop costs the other one 0.4 to 0.8 us).
template <bool MANY>
__global__ __launch_bounds__(256) void verify_tail_kernel(hb_attn_desc d, TailArgs t) {
  __shared__ int s_len, s_node;
  const int tid = threadIdx.x, l = blockIdx.y;
  const long first = ((long)l * gridDim.x + blockIdx.x) * 256 + tid, threads = (long)gridDim.x * gridDim.y * 256;
  for (long i = first; i < t.M; i += threads) {
    const int id = argmax_key_id(t.keys[i], t.V);
    t.target_ids[i] = id;
  }
  unsigned item = blockIdx.x;
  do {
    const int b = (int)item / t.path_slots, j = (int)item % t.path_slots;
    if (b >= d.batch) return;  // an empty batch, or done
    if (tid < 64) {
      const int n0 = t.node_offset[b];
      int n = t.node_offset[b + 1] - n0;
      n = n < 0 ? 0 : (n > d.max_nodes_per_tree ? d.max_nodes_per_tree : n);
      const bool live = tid < n && n0 >= 0 && n0 + tid < t.M;
      int par = -1, did = 0, tgt = 0;
      if (live) {
        par = t.parent[n0 + tid];
        did = t.draft_ids[n0 + tid];
        tgt = argmax_key_id(t.keys[n0 + tid], t.V);
      }
      const Accepted a = accept_wave(tid, live, par, did, tgt, true, t.max_path);
      if (j == 0 && l == 0) store_accepted(a, tid, did, -1, b, t.max_path, t.accept_len, t.accept_path, t.out_tokens, t.bonus_id);
      if (tid == 0) s_len = a.len;
      if (((a.path >> tid) & 1ull) && __popcll(a.path & ((1ull << tid) - 1ull)) == j) s_node = tid;
    }
    if (t.layers) {
      __syncthreads();
      const bool tables = t.tables;
      compact_one(d, t.row_bytes, j, b, s_len, j < s_len ? s_node : 0, (const uint4 *)(tables ? ((const void *const *)t.k_tree)[l] : t.k_tree),
                  (const uint4 *)(tables ? ((const void *const *)t.v_tree)[l] : t.v_tree),
                  (uint4 *)(tables ? ((void *const *)t.k_pool)[l] : t.k_pool), (uint4 *)(tables ? ((void *const *)t.v_pool)[l] : t.v_pool),
                  t.block_table, t.prefix_len, t.node_offset, t.max_path, l == 0 ? t.out_slots : nullptr, l == 0 ? t.new_len : nullptr);
      // slots that no path of a tree reaches
      if (t.path_slots < t.max_path && j == 0 && l == 0 && t.out_slots)
        for (int past = t.path_slots + tid; past < t.max_path; past += 256) t.out_slots[(size_t)b * t.max_path + past] = -1;
      if (MANY) __syncthreads();  // s_len and s_node are read
    }
    item += gridDim.x;
  } while (MANY);
}

}  // namespace

hipError_t launch_tree_accept(int32_t B, int32_t max_nodes, const int32_t *node_offset,
                              const int32_t *parent, const int32_t *draft_ids,
                              const int32_t *target_ids, const int32_t *prev_target, int32_t max_path,
                              int32_t *accept_len, int32_t *accept_path, int32_t *out_tokens,
                              int32_t *bonus_id, hipStream_t s) {
  tree_accept_kernel<<<B, 64, 0, s>>>(max_nodes, node_offset, parent, draft_ids, target_ids, prev_target, max_path,
                                      accept_len, accept_path, out_tokens, bonus_id);
  return hipGetLastError();
}

hipError_t launch_kv_compact(const hb_attn_desc &d, const void *k_tree, const void *v_tree,
                             void *k_pool, void *v_pool, const int32_t *block_table,
                             const int32_t *prefix_len, const int32_t *node_offset,
                             const int32_t *accept_len, const int32_t *accept_path,
                             int32_t max_path, int32_t *out_slots, int32_t *new_len, hipStream_t s) {
  int row_bytes = d.head_dim * (d.dtype == HB_F32 ? 4 : 2);  // head_dim % 8 == 0, so % 16 == 0
  dim3 grid((unsigned)max_path, (unsigned)d.batch);
  kv_compact_kernel<<<grid, 256, 0, s>>>(d, row_bytes, (const uint4 *)k_tree, (const uint4 *)v_tree,
                                         (uint4 *)k_pool, (uint4 *)v_pool, block_table, prefix_len,
                                         node_offset, accept_len, accept_path, max_path, out_slots, new_len);
  return hipGetLastError();
}

hipError_t launch_kv_compact_layers(const hb_attn_desc &d, int32_t n_layers, const void *const *k_tree,
                                    const void *const *v_tree, void *const *k_pool, void *const *v_pool,
                                    const int32_t *block_table, const int32_t *prefix_len,
                                    const int32_t *node_offset, const int32_t *accept_len,
                                    const int32_t *accept_path, int32_t max_path, int32_t *out_slots,
                                    int32_t *new_len, hipStream_t s) {
  int row_bytes = d.head_dim * (d.dtype == HB_F32 ? 4 : 2);
  dim3 grid((unsigned)max_path, (unsigned)d.batch, (unsigned)n_layers);
  kv_compact_layers_kernel<<<grid, 256, 0, s>>>(d, row_bytes, (const uint4 *const *)k_tree, (const uint4 *const *)v_tree,
                                                (uint4 *const *)k_pool, (uint4 *const *)v_pool, block_table,
                                                prefix_len, node_offset, accept_len, accept_path, max_path,
                                                out_slots, new_len);
  return hipGetLastError();
}

hipError_t launch_verify_tail(const hb_attn_desc &d, TailArgs t, hipStream_t s) {
  t.row_bytes = d.head_dim * (d.dtype == HB_F32 ? 4 : 2);
  // acceptance alone needs one workgroup a sequence; a tree has no more nodes than a wavefront has lanes
  t.path_slots = !t.layers ? 1 : t.max_path < 64 ? t.max_path : 64;
  constexpr long kMost = 1l << 22;  // workgroups of 256 threads: far from the 2^32 - 1 threads that a grid may have
  const long items = (long)d.batch * t.path_slots;
  if (items > INT32_MAX - kMost) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(items < 1 ? 1 : items < kMost ? items : kMost), (unsigned)(t.layers > 0 ? t.layers : 1));
  if (items > kMost) verify_tail_kernel<true><<<grid, 256, 0, s>>>(d, t);
  else verify_tail_kernel<false><<<grid, 256, 0, s>>>(d, t);
  return hipGetLastError();
}

}  // namespace hb
