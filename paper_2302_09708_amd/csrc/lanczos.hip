// Vector kernels of the Lanczos estimate of lam_Nd, the largest eigenvalue of H that
// Alg. 1 takes as the top of the filter interval (the paper leaves its computation
// open; the library's reading is a k-step Lanczos run from a caller-given vector).
//
// One Lanczos step on the device:  w = H v_j (hx_apply with no Chebyshev terms), then
//   lanczos_dot:   w -= beta_{j-1} v_{j-1};  partial sums of v_j . w
//   lanczos_norm:  alpha_j = their sum;  w -= alpha_j v_j;  partial sums of w . w
//   lanczos_scale: beta_j = sqrt of their sum;  v_{j+1} = w / beta_j
// The coefficients stay on the device: every block of the kernel that needs one adds the
// previous kernel's block sums itself (kLzBlocks values), so a step is three launches and
// no copy to the host.  72^3 FP64, 20 steps: 1.16 -> 0.65 ms against two extra summing
// kernels and two copies to the host per step.  A step is bound by its five launches of 4 to
// 12 us each on a 3 MB vector.
// Every reduction has a fixed grid and a fixed order (grid-stride partial per thread, LDS
// tree per block, the block sums by a tree of one block's threads), so results are bitwise
// reproducible.  Orbital vectors are stored in the handle's precision (TV), w and all sums
// in FP64.
#include "common.h"

namespace chefsi {

namespace {

__device__ __forceinline__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int off = kVecThreads / 2; off > 0; off >>= 1) {
    if (t < off) red[t] += red[t + off];
    __syncthreads();
  }
  const double s = red[0];
  __syncthreads();  // red may be written again
  return s;
}

// the sum of the kLzBlocks block sums that the previous kernel left
__device__ __forceinline__ double sum_of_blocks(const double* __restrict__ partial, double* red) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < kLzBlocks; i += kVecThreads) acc += partial[i];
  return block_sum(acc, red);
}

template <typename TV>
__global__ __launch_bounds__(kVecThreads) void lanczos_dot_kernel(double* __restrict__ w, const TV* __restrict__ v,
                                                                  const TV* __restrict__ vp,
                                                                  const double* __restrict__ beta, int64_t n,
                                                                  double* __restrict__ partial) {
  __shared__ double red[kVecThreads];
  const double b = vp != nullptr ? *beta : 0.0;
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kVecThreads) {
    double wi = w[i];
    if (vp != nullptr) {
      wi -= b * double(vp[i]);
      w[i] = wi;
    }
    acc += double(v[i]) * wi;
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

template <typename TV>
__global__ __launch_bounds__(kVecThreads) void lanczos_norm_kernel(double* __restrict__ w, const TV* __restrict__ v,
                                                                   const double* __restrict__ dots, int64_t n,
                                                                   double* __restrict__ partial,
                                                                   double* __restrict__ alpha_out) {
  __shared__ double red[kVecThreads];
  double alpha = 0.0;
  if (v != nullptr) {
    alpha = sum_of_blocks(dots, red);
    if (blockIdx.x == 0 && threadIdx.x == 0) *alpha_out = alpha;
  }
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kVecThreads) {
    double wi = w[i];
    if (v != nullptr) {
      wi -= alpha * double(v[i]);
      w[i] = wi;
    }
    acc += wi * wi;
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

template <typename TV>
__global__ __launch_bounds__(kVecThreads) void lanczos_scale_kernel(const double* __restrict__ w,
                                                                    const double* __restrict__ squares, int64_t n,
                                                                    TV* __restrict__ out,
                                                                    double* __restrict__ norm_out) {
  __shared__ double red[kVecThreads];
  const double norm = sqrt(sum_of_blocks(squares, red));
  if (blockIdx.x == 0 && threadIdx.x == 0) *norm_out = norm;
  const double inv = 1.0 / norm;
  for (int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kVecThreads)
    out[i] = TV(w[i] * inv);
}

template <typename TV>
__global__ __launch_bounds__(kVecThreads) void widen_kernel(const TV* __restrict__ x, int64_t n,
                                                            double* __restrict__ w) {
  for (int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kVecThreads)
    w[i] = double(x[i]);
}

}  // namespace

template <typename TV>
hipError_t launch_lanczos_dot(double* w, const TV* v, const TV* vp, const double* beta, int64_t n, double* partial,
                              hipStream_t s) {
  hipLaunchKernelGGL((lanczos_dot_kernel<TV>), dim3(kLzBlocks), dim3(kVecThreads), 0, s, w, v, vp, beta, n, partial);
  return hipGetLastError();
}

template <typename TV>
hipError_t launch_lanczos_norm(double* w, const TV* v, const double* dots, int64_t n, double* partial,
                               double* alpha_out, hipStream_t s) {
  hipLaunchKernelGGL((lanczos_norm_kernel<TV>), dim3(kLzBlocks), dim3(kVecThreads), 0, s, w, v, dots, n, partial,
                     alpha_out);
  return hipGetLastError();
}

template <typename TV>
hipError_t launch_lanczos_scale(const double* w, const double* squares, int64_t n, TV* out, double* norm_out,
                                hipStream_t s) {
  hipLaunchKernelGGL((lanczos_scale_kernel<TV>), dim3(kLzBlocks), dim3(kVecThreads), 0, s, w, squares, n, out,
                     norm_out);
  return hipGetLastError();
}

template <typename TV>
hipError_t launch_widen(const TV* x, int64_t n, double* w, hipStream_t s) {
  hipLaunchKernelGGL((widen_kernel<TV>), dim3(kLzBlocks), dim3(kVecThreads), 0, s, x, n, w);
  return hipGetLastError();
}

template hipError_t launch_lanczos_dot<double>(double*, const double*, const double*, const double*, int64_t, double*,
                                               hipStream_t);
template hipError_t launch_lanczos_dot<float>(double*, const float*, const float*, const double*, int64_t, double*,
                                              hipStream_t);
template hipError_t launch_lanczos_norm<double>(double*, const double*, const double*, int64_t, double*, double*,
                                                hipStream_t);
template hipError_t launch_lanczos_norm<float>(double*, const float*, const double*, int64_t, double*, double*,
                                               hipStream_t);
template hipError_t launch_lanczos_scale<double>(const double*, const double*, int64_t, double*, double*, hipStream_t);
template hipError_t launch_lanczos_scale<float>(const double*, const double*, int64_t, float*, double*, hipStream_t);
template hipError_t launch_widen<double>(const double*, int64_t, double*, hipStream_t);
template hipError_t launch_widen<float>(const float*, int64_t, double*, hipStream_t);

}  // namespace chefsi
