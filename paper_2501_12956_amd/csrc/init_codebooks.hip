// T^0: initial per-row codebooks (input of Algorithm 1), built from per-row
// quantiles of W.  One workgroup per row holds the row in registers and finds the
// at most 32 order statistics that the C quantiles interpolate between by radix
// selection (row_select.h).  Bound by LDS atomics and the levels' barriers.
// Against a bitonic sort of the row in LDS: 2048 x 2048 110 -> 31 us, 4096 x 4096
// 500 -> 94 us, 8192 x 28672 9.3 -> 1.5 ms (4 bits).
// Also: fp16 -> fp32 conversion of W for the fp32 solve.
#include "ganq_internal.h"
#include "row_select.h"

namespace ganq {
namespace {

// Entry s of the codebook lies between the order statistics lo and hi of a row of n.
__device__ inline double quantile_ranks(int s, int C, int mode, int n, int& lo, int& hi) {
  if (mode == GANQ_INIT_MINMAX_GRID) {
    lo = 0;
    hi = n - 1;
    return (C > 1) ? (double)s / (double)(C - 1) : 0.0;
  }
  double q;
  if (mode == GANQ_INIT_QUANTILE_MID)
    q = ((double)s + 0.5) / (double)C;
  else
    q = (C > 1) ? (double)s / (double)(C - 1) : 0.5;
  const double h = q * (double)(n - 1);
  lo = (int)floor(h);
  if (lo > n - 1) lo = n - 1;
  hi = (lo + 1 < n) ? lo + 1 : n - 1;
  return h - (double)lo;
}

template <typename TW, int TPB, int EPT>
__global__ __launch_bounds__(TPB) void init_codebooks_kernel(const TW* __restrict__ W, int n, int64_t ldw, int C,
                                                             int mode, float* __restrict__ T) {
  __shared__ SelectShared<32> sh;
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x;
  uint32_t key[EPT], slot[(EPT + 3) / 4];
  load_row_keys<TW, TPB, EPT>(W + row * ldw, n, tid, key, slot);
  double frac = 0.0;
  if (tid < C) {                   // ranks s and C + s of the selection
    int lo, hi;
    frac = quantile_ranks(tid, C, mode, n, lo, hi);
    sh.rank[tid] = (uint32_t)lo;
    sh.rank[C + tid] = (uint32_t)hi;
  }
  __syncthreads();
  select_ranks<TW, TPB, EPT, 32>(sh, key, slot, 2 * C, tid);
  if (tid < C) {
    const double a = key_value(sh.key[tid], (TW)0), b = key_value(sh.key[C + tid], (TW)0);
    T[row * C + tid] = (float)(a + frac * (b - a));
  }
}

// Rows of at most 64 elements: a wavefront per row and an element per lane, which finds its place in the
// sorted row by comparing itself with all the others.
template <typename TW>
__global__ __launch_bounds__(256) void init_codebooks_short_kernel(const TW* __restrict__ W, int64_t m, int n,
                                                                   int64_t ldw, int C, int mode,
                                                                   float* __restrict__ T) {
  __shared__ uint32_t keys[4][64], sorted[4][64];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wv;
  const bool in = row < m && lane < n;
  const uint32_t key = in ? order_key(W[row * ldw + lane]) : 0u;
  keys[wv][lane] = key;
  __syncthreads();
  int rank = 0;
  for (int j = 0; j < n; ++j) {
    const uint32_t k = keys[wv][j];
    rank += (k < key || (k == key && j < lane)) ? 1 : 0;
  }
  if (in) sorted[wv][rank] = key;
  __syncthreads();
  if (row < m && lane < C) {
    int lo, hi;
    const double frac = quantile_ranks(lane, C, mode, n, lo, hi);
    const double a = key_value(sorted[wv][lo], (TW)0), b = key_value(sorted[wv][hi], (TW)0);
    T[row * C + lane] = (float)(a + frac * (b - a));
  }
}

__global__ __launch_bounds__(256) void convert_f16_f32_kernel(const _Float16* __restrict__ src,
                                                              int64_t cols, int64_t ld_src,
                                                              float* __restrict__ dst,
                                                              int64_t ld_dst) {
  const int64_t r = blockIdx.y;
  for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < cols; c += (int64_t)gridDim.x * 256)
    dst[r * ld_dst + c] = (float)src[r * ld_src + c];
}

template <typename TW>
void launch_init(hipStream_t s, const TW* W, int64_t m, int64_t n, int64_t ldw, int C, int mode, float* T) {
  const dim3 grid((unsigned)m);
  // A selection costs the same for any row up to 2048 (65535 rows of fp32, 4 bits: 771 us, 359 us when rows
  // of 16 and 659 us when rows of 64 were sorted); comparing all pairs takes 17 and 37 us.
  if (n <= 64)
    hipLaunchKernelGGL(init_codebooks_short_kernel<TW>, dim3((unsigned)ceil_div(m, 4)), dim3(256), 0, s, W, m, (int)n,
                       ldw, C, mode, T);
  else if (n <= 2048)
    hipLaunchKernelGGL((init_codebooks_kernel<TW, 256, 8>), grid, dim3(256), 0, s, W, (int)n, ldw, C, mode, T);
  else if (n <= 4096)
    hipLaunchKernelGGL((init_codebooks_kernel<TW, 256, 16>), grid, dim3(256), 0, s, W, (int)n, ldw, C, mode, T);
  else if (n <= 16384)
    hipLaunchKernelGGL((init_codebooks_kernel<TW, 1024, 16>), grid, dim3(1024), 0, s, W, (int)n, ldw, C, mode, T);
  else
    hipLaunchKernelGGL((init_codebooks_kernel<TW, 1024, 32>), grid, dim3(1024), 0, s, W, (int)n, ldw, C, mode, T);
}

}  // namespace

// Requires n <= 32768 and nbits <= 4.
hipError_t launch_init_codebooks(hipStream_t s, const void* W, int w_is_f16, int64_t m, int64_t n,
                                 int64_t ldw, int nbits, int mode, float* T) {
  if (w_is_f16)
    launch_init(s, (const _Float16*)W, m, n, ldw, 1 << nbits, mode, T);
  else
    launch_init(s, (const float*)W, m, n, ldw, 1 << nbits, mode, T);
  return hipGetLastError();
}

hipError_t launch_convert_f16_f32(hipStream_t s, const _Float16* src, int64_t rows, int64_t cols,
                                  int64_t ld_src, float* dst, int64_t ld_dst) {
  dim3 grid((unsigned)((cols + 1023) / 1024 > 0 ? (cols + 1023) / 1024 : 1), (unsigned)rows);
  hipLaunchKernelGGL(convert_f16_f32_kernel, grid, dim3(256), 0, s, src, cols, ld_src, dst, ld_dst);
  return hipGetLastError();
}

}  // namespace ganq
