// Cholesky factor and triangular solves of the dense stage (Alg. 1, Diagonalization; Sec. 2.3)
// for subspaces up to kCholMax orbitals: Ms = U^T U, C = U^-T Hs U^-1, Z = U^-1 W.
//
// What bounds them is not their n^3 (600: 0.2 GFLOP) but a chain of n pivots and, in a library
// call, the kernels between its small panels.  Here a panel of 64 pivots is two launches: every
// block factors the diagonal block in registers, redundantly, carrying its own 64 columns along
// (so the solve for the panel's row of U is the same loop; 0.4 us a pivot, an LDS round and a
// division), then the trailing blocks take their update on MFMA.  The first block carries the
// identity: it leaves the panel's U_kk^-1, with which the triangular solves are products: one
// block owns 16 right-hand sides, kept in LDS, and goes through all block rows without a word
// from any other block.  n = 600: factor 1.30 -> 0.36 ms, the three solves 0.70 -> 0.22 (against
// rocSOLVER and rocBLAS); the whole subspace problem 7.24 -> 5.93 ms, 1200 16.2 -> 13.7, 40
// 0.63 -> 0.55.
#include <algorithm>

#include "common.h"

namespace chefsi {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int kNb = kCholBlock;  // 64 pivots a panel

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Panel k.  Thread (ty, tx) of 16 x 16 owns rows ty + 16 a and columns tx + 16 b (a, b < 4) of
// the symmetric diagonal block and of the block's own columns; a pivot's row goes through LDS
// (two buffers, one barrier a pivot).  Eliminated rows stay unscaled until the end: row i of U
// is row i over sqrt(d_i).  Block 0 writes U_kk to `diag` (the others may still be reading the
// block itself) and U_kk^-1 to inv; block b the columns of panel k + b.
__global__ __launch_bounds__(256) void chol_panel_kernel(double* __restrict__ A, int n, int k,
                                                         double* __restrict__ inv, double* __restrict__ diag,
                                                         int* __restrict__ info) {
  __shared__ double row[2][2 * kNb];
  __shared__ double piv[kNb];
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  const int k0 = k * kNb, m = min(kNb, n - k0);
  const int j0 = (k + blockIdx.x) * kNb, w = min(kNb, n - j0);
  const bool first = blockIdx.x == 0;
  if (k > 0 && *info != 0) return;
  double p[4][4], q[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int r = ty + 16 * a, c = tx + 16 * b, lo = min(r, c), hi = max(r, c);
      p[a][b] = hi < m ? A[k0 + lo + (int64_t)(k0 + hi) * n] : (r == c ? 1.0 : 0.0);
      q[a][b] = first ? (r == c ? 1.0 : 0.0) : (r < m && c < w ? A[k0 + r + (int64_t)(j0 + c) * n] : 0.0);
    }
#pragma unroll
  for (int ai = 0; ai < 4; ++ai)
    for (int i16 = 0; i16 < 16; ++i16) {
      const int i = 16 * ai + i16;
      if (i >= m) break;
      double* buf = row[i & 1];
      if (ty == i16) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          buf[tx + 16 * b] = p[ai][b];
          buf[kNb + tx + 16 * b] = q[ai][b];
        }
      }
      __syncthreads();
      const double d = buf[i];
      if (d <= 0.0) {  // the same value in every thread of every block
        if (first && tid == 0) *info = k0 + i + 1;
        return;
      }
      if (tid == 0) piv[i] = d;
      const double di = 1.0 / d;
      double f[4], u[4], v[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        u[b] = buf[tx + 16 * b];
        v[b] = buf[kNb + tx + 16 * b];
      }
#pragma unroll
      for (int a = ai; a < 4; ++a) f[a] = ty + 16 * a > i ? buf[ty + 16 * a] * di : 0.0;
#pragma unroll
      for (int a = ai; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          p[a][b] -= f[a] * u[b];
          q[a][b] -= f[a] * v[b];
        }
    }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int r = ty + 16 * a;
    const double s = r < m ? 1.0 / sqrt(piv[r]) : 1.0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int c = tx + 16 * b;
      if (first) {
        diag[r + kNb * c] = p[a][b] * s;
        inv[(int64_t)k * kNb * kNb + c + kNb * r] = q[a][b] * s;  // U_kk^-1 (c, r)
      } else if (r < m && c < w) {
        A[k0 + r + (int64_t)(j0 + c) * n] = q[a][b] * s;
      }
    }
  }
}

// Trailing blocks (i, j), k < i <= j, of the upper triangle: A_ij -= U_ki^T U_kj; the last block
// of the grid puts U_kk in its place.
__global__ __launch_bounds__(256) void chol_update_kernel(double* __restrict__ A, int n, int k, int nb,
                                                          const double* __restrict__ diag,
                                                          const int* __restrict__ info) {
  if (*info != 0) return;
  const int tid = threadIdx.x, k0 = k * kNb;
  if (blockIdx.x == gridDim.x - 1) {
    for (int e = tid; e < kNb * kNb; e += 256) {
      const int r = e % kNb, c = e / kNb;
      if (r <= c && k0 + c < n) A[k0 + r + (int64_t)(k0 + c) * n] = diag[e];
    }
    return;
  }
  int t = blockIdx.x, bi = k + 1, left = nb - bi;
  while (t >= left) {
    t -= left--;
    ++bi;
  }
  const int i0 = bi * kNb, j0 = (bi + t) * kNb;
  const int lane = tid & 63, wave = tid >> 6, g = lane >> 4, r = lane & 15;
  const double* pj = A + k0 + (int64_t)min(j0 + 16 * wave + r, n - 1) * n + 4 * g;
  const double* pi[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) pi[f] = A + k0 + (int64_t)min(i0 + 16 * f + r, n - 1) * n + 4 * g;
  d4 acc[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) acc[f] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < kNb / 16; ++s) {
    const d2u ja = *reinterpret_cast<const d2u*>(pj + 16 * s), jb = *reinterpret_cast<const d2u*>(pj + 16 * s + 2);
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const d2u ia = *reinterpret_cast<const d2u*>(pi[f] + 16 * s);
      const d2u ib = *reinterpret_cast<const d2u*>(pi[f] + 16 * s + 2);
      acc[f] = mfma(ja[0], ia[0], acc[f]);
      acc[f] = mfma(ja[1], ia[1], acc[f]);
      acc[f] = mfma(jb[0], ib[0], acc[f]);
      acc[f] = mfma(jb[1], ib[1], acc[f]);
    }
  }
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int v = 0; v < 4; ++v) {  // D[j][i]: lane i + 16 (j % 4), register j / 4
      const int ri = i0 + 16 * f + r, cj = j0 + 16 * wave + g + 4 * v;
      if (cj < n && ri <= cj) A[ri + (int64_t)cj * n] -= acc[f][v];
    }
}

// 16 columns of U^T Y = B (FWD) or U Y = B in LDS (column-major, pitch np + 4), one block row of
// 64 after the other: R = B_i - (what the finished rows contribute), Y_i = U_ii^-T R or U_ii^-1 R.
// Wave w owns rows 16 w .. + 15 of the block row.  BT reads B transposed; sc scales the rows of
// the result.  Every column is the block's own, so Y may be B.
template <bool FWD, bool BT>
__global__ __launch_bounds__(256) void tri_solve_kernel(const double* __restrict__ U, const double* __restrict__ inv,
                                                        int n, int nb, const double* B, double* Y,
                                                        const double* __restrict__ sc, const int* __restrict__ info) {
  extern __shared__ __align__(16) double y[];
  if (*info != 0) return;  // no factor: everything stays as it is
  const int np = nb * kNb, pitch = np + 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, r = lane & 15;
  const int c0 = blockIdx.x * 16;
  for (int e = tid; e < 16 * np; e += 256) {
    const int c = BT ? e % 16 : e / np, i = BT ? e / 16 : e % np;
    const bool in = c0 + c < n && i < n;
    y[c * pitch + i] = in ? (BT ? B[c0 + c + (int64_t)i * n] : B[i + (int64_t)(c0 + c) * n]) : 0.0;
  }
  __syncthreads();
  const double* yc = y + r * pitch + 4 * g;  // the lane's column, rows 4 g .. + 3 of a step
  for (int t = 0; t < nb; ++t) {
    const int i = FWD ? t : nb - 1 - t, i0 = i * kNb;
    const int row = min(i0 + 16 * wave + r, n - 1);  // rows past n: their products are not used
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    const int kb = FWD ? 0 : i + 1, ke = FWD ? i : nb;
    for (int k = kb; k < ke; ++k) {
      double a[4][4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int kk = k * kNb + 16 * s + 4 * g;
        if (FWD) {
          const double* p = U + kk + (int64_t)row * n;
          const d2u lo = *reinterpret_cast<const d2u*>(p), hi = *reinterpret_cast<const d2u*>(p + 2);
          a[s][0] = lo[0];
          a[s][1] = lo[1];
          a[s][2] = hi[0];
          a[s][3] = hi[1];
        } else {  // columns past n meet zero rows of y
#pragma unroll
          for (int e = 0; e < 4; ++e) a[s][e] = U[row + (int64_t)min(kk + e, n - 1) * n];
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma(a[s][e], yc[k * kNb + 16 * s + e], acc);
    }
    // D[row][col]: lane col + 16 (row % 4), register row / 4
    double* rr = y + r * pitch + i0 + 16 * wave + g;
#pragma unroll
    for (int v = 0; v < 4; ++v) rr[4 * v] -= acc[v];
    __syncthreads();
    const double* iv = inv + (int64_t)i * kNb * kNb;
    acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 16 * s + 4 * g + e, o = 16 * wave + r;
        acc = mfma(FWD ? iv[k + kNb * o] : iv[o + kNb * k], yc[i0 + 16 * s + e], acc);
      }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) rr[4 * v] = acc[v];
    __syncthreads();
  }
  for (int e = tid; e < 16 * np; e += 256) {
    const int c = e / np, i = e % np;
    if (c0 + c < n && i < n) Y[i + (int64_t)(c0 + c) * n] = sc != nullptr ? sc[i] * y[c * pitch + i] : y[c * pitch + i];
  }
}

__global__ void clear_info_kernel(int* info) { *info = 0; }

}  // namespace

size_t chol_scratch_bytes(int n) {
  return n <= kCholMax ? (size_t)((n + kNb - 1) / kNb + 1) * kNb * kNb * sizeof(double) : 0;
}

hipError_t launch_cholesky(double* A, int n, void* scratch, int* info, hipStream_t s) {
  if (n <= 0 || n > kCholMax) return hipErrorInvalidValue;
  const int nb = (n + kNb - 1) / kNb;
  double* diag = static_cast<double*>(scratch);
  double* inv = diag + kNb * kNb;
  hipLaunchKernelGGL(clear_info_kernel, dim3(1), dim3(1), 0, s, info);
  for (int k = 0; k < nb; ++k) {
    hipLaunchKernelGGL(chol_panel_kernel, dim3((unsigned)(nb - k)), dim3(256), 0, s, A, n, k, inv, diag, info);
    const int left = nb - k - 1;
    hipLaunchKernelGGL(chol_update_kernel, dim3((unsigned)(left * (left + 1) / 2 + 1)), dim3(256), 0, s, A, n, k, nb,
                       diag, info);
  }
  return hipGetLastError();
}

template <bool FWD, bool BT>
static hipError_t tri_solve(const double* U, const void* scratch, int n, const double* B, double* Y, const double* sc,
                            const int* info, hipStream_t s) {
  if (n <= 0 || n > kCholMax) return hipErrorInvalidValue;
  const int nb = (n + kNb - 1) / kNb;
  const double* inv = static_cast<const double*>(scratch) + kNb * kNb;
  const size_t lds = (size_t)16 * (nb * kNb + 4) * sizeof(double);
  hipLaunchKernelGGL((tri_solve_kernel<FWD, BT>), dim3((unsigned)((n + 15) / 16)), dim3(256), lds, s, U, inv, n, nb, B,
                     Y, sc, info);
  return hipGetLastError();
}

hipError_t launch_reduce_pencil(const double* U, const void* scratch, int n, double* H, double* tmp, const int* info,
                                hipStream_t s) {
  const hipError_t e = tri_solve<true, false>(U, scratch, n, H, tmp, nullptr, info, s);  // X = U^-T H
  if (e != hipSuccess) return e;
  return tri_solve<true, true>(U, scratch, n, tmp, H, nullptr, info, s);  // C = C^T = U^-T X^T
}

hipError_t launch_back_substitute(const double* U, const void* scratch, int n, const double* W, double* Z,
                                  const double* sc, const int* info, hipStream_t s) {
  return tri_solve<false, false>(U, scratch, n, W, Z, sc, info, s);
}

}  // namespace chefsi
