// LM head with fused argmax, scalar fp32 kernels (any dtype, any sizes), plus the two tiny
// kernels every LM-head path shares: key initialisation and the final unpack.
//
// lmhead_rows_kernel serves few rows (see there).  Otherwise each workgroup computes a 64 x 64 tile of logits (rows of `hidden` x rows of `weight`) in
// registers, reduces each row of the tile to one (value, index) key and folds it into the
// row's global key with a 64-bit atomic max.  max over keys is order independent, so the
// result does not depend on scheduling.
#include "hb_internal.h"

namespace hb {

namespace {

constexpr int TM = 64, TN = 64, TK = 16;

template <typename T>
__global__ __launch_bounds__(256) void lmhead_scalar_kernel(int M, int K, int V, const T *__restrict__ hidden,
                                                            const T *__restrict__ weight,
                                                            unsigned long long *__restrict__ keys) {
  __shared__ float sh[TK][TM + 1];
  __shared__ float sw[TK][TN + 1];
  __shared__ unsigned long long srow[TM];
  const int tid = threadIdx.x;
  const int tx = tid & 15;   // column group: columns tx*4 .. tx*4+3
  const int ty = tid >> 4;   // row group: rows ty*4 .. ty*4+3
  const int m0 = blockIdx.y * TM;
  const int v0 = blockIdx.x * TN;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  if (tid < TM) srow[tid] = 0ull;

  for (int k0 = 0; k0 < K; k0 += TK) {
    // 64 rows x 16 k for each operand: 1024 elements, 4 per thread
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int e = tid + 256 * r;
      int rr = e >> 4, kk = e & 15;
      int m = m0 + rr, v = v0 + rr, k = k0 + kk;
      sh[kk][rr] = (m < M && k < K) ? load_f32(hidden + (size_t)m * K + k) : 0.f;
      sw[kk][rr] = (v < V && k < K) ? load_f32(weight + (size_t)v * K + k) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < TK; ++kk) {
      float a[4], bcol[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sh[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bcol[j] = sw[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], bcol[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int v = v0 + tx * 4 + j;
      if (v < V) {
        unsigned long long key = argmax_key(acc[i][j], (uint32_t)v);
        best = key > best ? key : best;
      }
    }
    if (best) atomicMax(&srow[ty * 4 + i], best);
  }
  __syncthreads();
  if (tid < TM && m0 + tid < M && srow[tid]) atomicMax(&keys[m0 + tid], srow[tid]);
}

// Few rows: the product is bound by latency and by the weight rows, and a 64 x 64 tile would leave
// most of its rows empty and give work to V / 64 workgroups only, each a chain of K / 16 round
// trips.  Here a wavefront takes kRowsV weight rows against kRowsM hidden rows with its lanes spread
// over K (16-byte loads, all of a step's twelve in flight), and the 32 sums are folded over the
// lanes by halving: each step sends half of the values and keeps the other.
constexpr int kRowsV = 4, kRowsM = 8;
constexpr int kRowsWaves = 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Piece;  // 16 bytes of a row
template <> struct Piece<float> {
  static constexpr int n = 4;
  f32x4 v;
  __device__ float at(int e) const { return v[e]; }
};
template <> struct Piece<bf16_t> {
  static constexpr int n = 8;
  u32x4 v;
  __device__ float at(int e) const { return __uint_as_float((e & 1) ? (v[e >> 1] & 0xffff0000u) : (v[e >> 1] << 16)); }
};

template <int N>
__device__ inline void fold_lanes(float (&x)[kRowsV * kRowsM], int lane) {
  // lanes that differ in bit 2 N of their number exchange halves of x[0 .. 2 N)
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool up = lane & (2 * N);
    const float keep = up ? x[i + N] : x[i], send = up ? x[i] : x[i + N];
    x[i] = keep + __shfl_xor(send, 2 * N, 64);
  }
}

template <typename T>
__global__ __launch_bounds__(64 * kRowsWaves) void lmhead_rows_kernel(int M, int K, int V, int m_groups, const T *__restrict__ hidden,
                                                                      const T *__restrict__ weight,
                                                                      unsigned long long *__restrict__ keys) {
  __shared__ unsigned long long best[kRowsWaves][kRowsM];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the groups of hidden rows are neighbours, so that memory gives a weight row once and the last-level cache
  // the others (one group after the other, 32 rows x 3592 x 152064 float32: 1900 us, beside each
  // other 1435)
  const int group = blockIdx.x / m_groups;
  const int v0 = (group * kRowsWaves + wave) * kRowsV, m0 = ((int)blockIdx.x - group * m_groups) * kRowsM;
  const T *w[kRowsV], *h[kRowsM];  // rows past the end read the last one and are dropped below
#pragma unroll
  for (int i = 0; i < kRowsV; ++i) w[i] = weight + (size_t)min(v0 + i, V - 1) * K;
#pragma unroll
  for (int j = 0; j < kRowsM; ++j) h[j] = hidden + (size_t)min(m0 + j, M - 1) * K;
  float acc[kRowsV * kRowsM];
#pragma unroll
  for (int i = 0; i < kRowsV * kRowsM; ++i) acc[i] = 0.f;
  for (int k = lane * Piece<T>::n; k < K; k += 64 * Piece<T>::n) {
    Piece<T> a[kRowsV], b[kRowsM];
#pragma unroll
    for (int i = 0; i < kRowsV; ++i) a[i] = *reinterpret_cast<const Piece<T> *>(w[i] + k);
#pragma unroll
    for (int j = 0; j < kRowsM; ++j) b[j] = *reinterpret_cast<const Piece<T> *>(h[j] + k);
#pragma unroll
    for (int i = 0; i < kRowsV; ++i)
#pragma unroll
      for (int j = 0; j < kRowsM; ++j)
#pragma unroll
        for (int e = 0; e < Piece<T>::n; ++e) acc[i * kRowsM + j] = fmaf(a[i].at(e), b[j].at(e), acc[i * kRowsM + j]);
  }
  fold_lanes<16>(acc, lane);
  fold_lanes<8>(acc, lane);
  fold_lanes<4>(acc, lane);
  fold_lanes<2>(acc, lane);
  fold_lanes<1>(acc, lane);
  const float x = acc[0] + __shfl_xor(acc[0], 1, 64);  // product of weight row lane / 16 and hidden row (lane / 2) % 8
  const int v = v0 + (lane >> 4);
  unsigned long long key = v < V ? argmax_key(x, (uint32_t)v) : 0ull;
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const unsigned long long other = __shfl_xor(key, off, 64);
    key = other > key ? other : key;
  }
  if (lane < 2 * kRowsM && !(lane & 1)) best[wave][lane >> 1] = key;
  __syncthreads();
  if (threadIdx.x < kRowsM && m0 + (int)threadIdx.x < M) {
    key = best[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < kRowsWaves; ++i) key = best[i][threadIdx.x] > key ? best[i][threadIdx.x] : key;
    unsigned long long *dst = &keys[m0 + threadIdx.x];
    if (key > __atomic_load_n(dst, __ATOMIC_RELAXED)) atomicMax(dst, key);
  }
}

__global__ void lmhead_init_kernel(unsigned long long *keys, int M) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < M) keys[i] = 0ull;
}

__global__ void lmhead_finish_kernel(const unsigned long long *keys, int M, int V, int32_t *out_ids,
                                     float *out_max) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  unsigned long long key = keys[i];
  out_ids[i] = argmax_key_id(key, V);
  if (out_max) out_max[i] = key ? argmax_key_value(key) : -__builtin_huge_valf();
}

}  // namespace

// Up to 32 rows the wavefronts' re-reading of the weight rows, once per eight hidden rows, costs less
// than the tile kernel's empty rows and round trips (float32, call with both small kernels):
// K x V = 256 x 1000, 1..256 rows 17.5 us against 32.6..36; 1024 x 32000: 8 rows 44 us against 157, 32 rows 93
// against 159, 64 rows 224 against 177 (one group of rows after the other); 1032 x 128000, 32 rows 406 against 396.
// Rows must consist of whole 16-byte pieces.
static bool rows_kernel_takes(int32_t dtype, int32_t M, int32_t K) {
  return M <= 32 && K % (dtype == HB_F32 ? Piece<float>::n : Piece<bf16_t>::n) == 0;
}

hipError_t launch_lmhead_scalar(int32_t dtype, int32_t M, int32_t K, int32_t V, const void *hidden,
                                const void *weight, unsigned long long *keys, hipStream_t s) {
  if (rows_kernel_takes(dtype, M, K)) {
    constexpr int kPerGroup = kRowsWaves * kRowsV;
    const int m_groups = (M + kRowsM - 1) / kRowsM;
    const unsigned grid = (unsigned)((V + kPerGroup - 1) / kPerGroup) * (unsigned)m_groups;
    if (dtype == HB_F32)
      lmhead_rows_kernel<float><<<grid, 64 * kRowsWaves, 0, s>>>(M, K, V, m_groups, (const float *)hidden, (const float *)weight, keys);
    else
      lmhead_rows_kernel<bf16_t><<<grid, 64 * kRowsWaves, 0, s>>>(M, K, V, m_groups, (const bf16_t *)hidden, (const bf16_t *)weight, keys);
    return hipGetLastError();
  }
  dim3 grid((unsigned)((V + TN - 1) / TN), (unsigned)((M + TM - 1) / TM));
  if (dtype == HB_F32)
    lmhead_scalar_kernel<float><<<grid, 256, 0, s>>>(M, K, V, (const float *)hidden, (const float *)weight, keys);
  else
    lmhead_scalar_kernel<bf16_t><<<grid, 256, 0, s>>>(M, K, V, (const bf16_t *)hidden, (const bf16_t *)weight, keys);
  return hipGetLastError();
}

hipError_t launch_lmhead_init(unsigned long long *keys, int32_t M, hipStream_t s) {
  lmhead_init_kernel<<<(M + 255) / 256, 256, 0, s>>>(keys, M);
  return hipGetLastError();
}

hipError_t launch_lmhead_finish(const unsigned long long *keys, int32_t M, int32_t V, int32_t *out_ids,
                                float *out_max, hipStream_t s) {
  lmhead_finish_kernel<<<(M + 255) / 256, 256, 0, s>>>(keys, M, V, out_ids, out_max);
  return hipGetLastError();
}

}  // namespace hb
