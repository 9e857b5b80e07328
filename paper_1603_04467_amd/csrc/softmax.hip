// Classifier cost head: SoftMax (the paper's section 2, Table 1) of the output
// layer's logits, the cross-entropy against integer class labels
// L = sum_n (log sum_j exp(z_nj) - z_n,y_n), and its gradient with respect to
// the logits, G = softmax(z) - onehot(y).
//
// Two kernels, by the row's length:
//  - up to kWaveCols columns: one wavefront per row (4 rows per 256-thread
//    block), the lanes striding over the row for the maximum, the sum of
//    exp(z - max) and the gradient, with butterfly shuffles for the two row
//    reductions;
//  - longer rows: one block per row that reads it once, in 16-byte chunks, and
//    keeps it in registers through the three passes.
// The loss is a float64 partial per block (of its rows' terms in row order),
// and one final block sums the partials in index order, so it is bitwise
// reproducible.

#include "common.h"
#include "kernels.h"

namespace tfd {

namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = kThreads / kWave;

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void softmax_xent_kernel(const T* __restrict__ z,
                                                                const int32_t* __restrict__ labels,
                                                                T* __restrict__ grad, double* __restrict__ partial,
                                                                int64_t rows, int64_t cols) {
  __shared__ double terms[kRowsPerBlock];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + w;
  double term = 0.0;
  if (row < rows) {
    const T* zr = z + row * cols;
    T* gr = grad + row * cols;
    float m = -INFINITY;
    for (int64_t c = lane; c < cols; c += kWave) m = fmaxf(m, load_f32(zr + c));
    m = wave_max(m);
    float s = 0.0f;
    for (int64_t c = lane; c < cols; c += kWave) s += expf(load_f32(zr + c) - m);
    s = wave_sum(s);
    const float inv = 1.0f / s;
    const int32_t y = labels[row];
    for (int64_t c = lane; c < cols; c += kWave) {
      float p = expf(load_f32(zr + c) - m) * inv;
      if (c == y) p -= 1.0f;
      store_from_f32(gr + c, p);
    }
    if (lane == 0) {
      term = (y >= 0 && y < cols) ? (double)logf(s) + (double)m - (double)load_f32(zr + y)
                                  : __builtin_nan("");
    }
  }
  if (lane == 0) terms[w] = term;
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < kRowsPerBlock; ++i) acc += terms[i];
    partial[blockIdx.x] = acc;
  }
}

// Rows of kWaveCols columns or fewer stay with a wavefront per row: a block
// per row would leave most of its threads idle.
constexpr int64_t kWaveCols = 512;

template <typename T> __device__ __forceinline__ void unpack16(const u32x4& v, float* x);
template <> __device__ __forceinline__ void unpack16<float>(const u32x4& v, float* x) {
  const f32x4 f = __builtin_bit_cast(f32x4, v);
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = f[e];
}
template <> __device__ __forceinline__ void unpack16<bf16>(const u32x4& v, float* x) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[2 * e] = bf16_bits_to_f32(v[e] & 0xFFFFu);
    x[2 * e + 1] = bf16_bits_to_f32(v[e] >> 16);
  }
}
template <typename T> __device__ __forceinline__ u32x4 pack16(const float* x);
template <> __device__ __forceinline__ u32x4 pack16<float>(const float* x) {
  return __builtin_bit_cast(u32x4, f32x4{x[0], x[1], x[2], x[3]});
}
template <> __device__ __forceinline__ u32x4 pack16<bf16>(const float* x) {
  u32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (uint32_t)bf16_bits(x[2 * e]) | ((uint32_t)bf16_bits(x[2 * e + 1]) << 16);
  return v;
}

// Sum or maximum over the block's NT threads, the same on every thread: the
// waves' butterflies, then the wave results in wave order. Two buffers in
// turn need no barrier between calls.
template <int NT, bool MAX>
__device__ __forceinline__ float block_reduce(float v, float* sh) {
  v = MAX ? wave_max(v) : wave_sum(v);
  if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = v;
  __syncthreads();
  float t = sh[0];
#pragma unroll
  for (int i = 1; i < NT / kWave; ++i) t = MAX ? fmaxf(t, sh[i]) : t + sh[i];
  return t;
}

// One row per block of NT threads (kPerBlock rows in turn where the workspace
// has no partial for each), up to NT * NC whole 16-byte chunks. Bound by HBM
// (the row in, the gradient out) once the row is read once: 2048 x 32768 bf16
// took 487 us with a wavefront per row (2-byte loads, the row read three times,
// two exponentials per element), 65-73 us here (3.7-4.1 TB/s). A row that does
// not start on a 16-byte boundary has up to V - 1 elements before its first
// whole chunk and after its last, one per thread; logits and gradient rows
// share their alignment (checked by the launcher).
template <typename T, int NT, int NC, int kPerBlock>
__global__ __launch_bounds__(NT) void softmax_xent_row_kernel(const T* __restrict__ z,
                                                              const int32_t* __restrict__ labels,
                                                              T* __restrict__ grad, double* __restrict__ partial,
                                                              int64_t rows, int64_t cols) {
  constexpr int V = elem_traits<T>::vec;
  __shared__ float sh[2][NT / kWave];
  const int tid = threadIdx.x;
  double term = 0.0;
  // (the rows' turns need no barrier between them: a wave is at most one
  // reduction ahead, in the other buffer)
#pragma unroll 1
  for (int r = 0; r < kPerBlock; ++r) {
    const int64_t row = (int64_t)blockIdx.x * kPerBlock + r;
    if (kPerBlock > 1 && row >= rows) break;
    const T* zr = z + row * cols;
    T* gr = grad + row * cols;
    const int n = (int)cols;
    const int head = min(n, (int)((16 - (reinterpret_cast<uintptr_t>(zr) & 15)) & 15) / (int)sizeof(T));
    const int body = (n - head) / V;  // whole chunks
    const int tail0 = head + body * V;
    // the element outside the whole chunks that this thread holds, if any
    const int edge = tid < head ? tid : (tid - head < n - tail0 ? tail0 + tid - head : -1);

    // Chunks past the row hold -infinity: they leave the maximum as it is and
    // add exp(-inf) = 0 to the sum.
    float x[NC][V];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = tid + i * NT;
      if (c < body) {
        unpack16<T>(*reinterpret_cast<const u32x4*>(zr + head + (int64_t)c * V), x[i]);
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e) x[i][e] = -INFINITY;
      }
    }
    const float ze = edge >= 0 ? load_f32(zr + edge) : -INFINITY;
    const int32_t y = labels[row];
    float m = ze;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int e = 0; e < V; ++e) m = fmaxf(m, x[i][e]);
    m = block_reduce<NT, true>(m, sh[0]);
    const float ee = expf(ze - m);
    float s = ee;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        x[i][e] = expf(x[i][e] - m);
        s += x[i][e];
      }
    }
    s = block_reduce<NT, false>(s, sh[1]);
    const float inv = 1.0f / s;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = tid + i * NT;
      if (c < body) {
        const int at = head + c * V;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          x[i][e] *= inv;
          if (at + e == y) x[i][e] -= 1.0f;
        }
        *reinterpret_cast<u32x4*>(gr + head + (int64_t)c * V) = pack16<T>(x[i]);
      }
    }
    if (edge >= 0) {
      float p = ee * inv;
      if (edge == y) p -= 1.0f;
      store_from_f32(gr + edge, p);
    }
    if (tid == 0)
      term += (y >= 0 && y < n) ? (double)logf(s) + (double)m - (double)load_f32(zr + y) : __builtin_nan("");
  }
  if (tid == 0) partial[blockIdx.x] = term;
}

template <typename T, int NT, int NC>
hipError_t launch_row(const T* z, const int32_t* labels, T* grad, double* partial, int64_t rows, int64_t cols,
                      int per_block, hipStream_t s) {
  if (per_block == 1)
    hipLaunchKernelGGL((softmax_xent_row_kernel<T, NT, NC, 1>), dim3((unsigned)rows), NT, 0, s, z, labels, grad,
                       partial, rows, cols);
  else
    hipLaunchKernelGGL((softmax_xent_row_kernel<T, NT, NC, kRowsPerBlock>),
                       dim3((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock)), NT, 0, s, z, labels, grad,
                       partial, rows, cols);
  return hipGetLastError();
}

// The fewest threads whose registers hold a row (8 chunks each at most).
template <typename T>
int row_threads(int64_t cols) { return cols / elem_traits<T>::vec <= 2048 ? 256 : 1024; }

// Whether rows go one to a block: longer than a wavefront's share, short
// enough for a block's registers (8 chunks per thread of 1024 threads), no more
// than a grid of 2^32 threads holds, and logits and gradient with the same
// alignment so that both move in whole chunks.
template <typename T>
bool row_per_block(const T* z, const T* grad, int64_t rows, int64_t cols) {
  constexpr int V = elem_traits<T>::vec;
  return cols > kWaveCols && cols / V + 1 <= 8 * 1024 && rows * row_threads<T>(cols) < (1LL << 32) &&
         ((reinterpret_cast<uintptr_t>(z) ^ reinterpret_cast<uintptr_t>(grad)) & 15) == 0 &&
         (reinterpret_cast<uintptr_t>(z) & (sizeof(T) - 1)) == 0;
}

template <typename T>
hipError_t launch_rows(const T* z, const int32_t* labels, T* grad, double* partial, int64_t rows, int64_t cols,
                       int per_block, hipStream_t s) {
  const int64_t chunks = cols / elem_traits<T>::vec;  // at most this many whole ones in a row
  if (row_threads<T>(cols) == 1024)
    return chunks <= 4096 ? launch_row<T, 1024, 4>(z, labels, grad, partial, rows, cols, per_block, s)
                          : launch_row<T, 1024, 8>(z, labels, grad, partial, rows, cols, per_block, s);
  if (chunks <= 256) return launch_row<T, 256, 1>(z, labels, grad, partial, rows, cols, per_block, s);
  if (chunks <= 512) return launch_row<T, 256, 2>(z, labels, grad, partial, rows, cols, per_block, s);
  if (chunks <= 1024) return launch_row<T, 256, 4>(z, labels, grad, partial, rows, cols, per_block, s);
  return launch_row<T, 256, 8>(z, labels, grad, partial, rows, cols, per_block, s);
}

__global__ __launch_bounds__(kThreads) void sum_partials_kernel(const double* partial, int64_t n, double* out) {
  __shared__ double sh[kThreads];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kThreads) acc += partial[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
#pragma unroll
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

}  // namespace

// One partial per block of four rows.
size_t softmax_xent_ws_bytes(int64_t rows) {
  return (size_t)(rows > 0 ? (rows + kRowsPerBlock - 1) / kRowsPerBlock : 1) * sizeof(double);
}

template <typename T>
static hipError_t launch_t(const T* logits, const int32_t* labels, T* grad, double* partial, int64_t rows,
                           int64_t cols, int per_block, int64_t* blocks, hipStream_t s) {
  if (row_per_block(logits, grad, rows, cols)) {
    *blocks = (rows + per_block - 1) / per_block;
    return launch_rows(logits, labels, grad, partial, rows, cols, per_block, s);
  }
  *blocks = (rows + kRowsPerBlock - 1) / kRowsPerBlock;
  hipLaunchKernelGGL((softmax_xent_kernel<T>), dim3((unsigned)*blocks), kThreads, 0, s, logits, labels, grad, partial,
                     rows, cols);
  return hipGetLastError();
}

hipError_t launch_softmax_xent(const void* logits, const int32_t* labels, void* grad, double* loss, int64_t rows,
                               int64_t cols, bool bf16_t, void* ws, size_t ws_bytes, hipStream_t s) {
  double* partial = static_cast<double*>(ws);
  const int per_block = ws_bytes >= (size_t)rows * sizeof(double) ? 1 : kRowsPerBlock;
  int64_t blocks = 0;
  if (rows > 0) {
    const hipError_t e =
        bf16_t ? launch_t((const bf16*)logits, labels, (bf16*)grad, partial, rows, cols, per_block, &blocks, s)
               : launch_t((const float*)logits, labels, (float*)grad, partial, rows, cols, per_block, &blocks, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(sum_partials_kernel, 1, kThreads, 0, s, (const double*)partial, blocks, loss);
  return hipGetLastError();
}

}  // namespace tfd
