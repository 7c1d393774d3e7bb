// Both FP64 Gram products of a projection, Hs = X^T Y and Ms = X^T X (Alg. 1; Sec. 2.2), in
// one split-K kernel on v_mfma_f64_16x16x4f64 and one fixed-order sum over the splits.
//
// The columns are cut into t tiles of NF 16-wide fragments (NF <= 4, the same for every tile,
// so little is padded).  A block of four waves owns one unit over one K chunk: the diagonal
// unit of a tile forms the upper fragments of both products from one read of X and Y, an
// off-diagonal unit the NF x NF fragments of one product (t^2 units in all; results are
// symmetric, nothing below the diagonal is formed).  The waves take every fourth 16-row step
// and add their fragments through LDS, so a block writes one partial.
//
// What bounds it: a fragment's MFMA takes 64 cycles of a SIMD and a step of an off-diagonal
// 4 x 4 unit 64 of them for 16 KB of operands, so operands come straight from memory into
// registers (lane l: 32 contiguous bytes of column l % 16, whole 128-byte lines per column),
// refilled for the next step behind their last MFMA; 256 VGPRs without spills, two blocks on a
// CU.  Wide blocks wait for the matrix units (72^3, 600 orbitals: 61 TFLOP/s of the fragments
// formed, the library's large product reaches 71), below about 64 orbitals for the one read of
// X and Y, on small grids for the launches.  Both products, before (rocBLAS, split-K batches
// and a sum each) / now, us: 24^3 40 orbitals 274 / 17; 45^3 187: 526 / 148; 64^3 100: 390 /
// 227; 72^3 256: 1266 / 955; 72^3 600: 6239 / 5329.
#include "common.h"

#include <algorithm>

namespace chefsi {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));  // columns start at any multiple of 8 bytes

constexpr int kGfWaves = 4;
constexpr int kGfStep = 16;   // rows a wave takes at a time
constexpr int kGfRound = 512; // blocks at work at once: two on each of 256 CUs (NF = 4)

// (i, j), i < j, of strictly upper pair p of t tiles (row-major)
__device__ __forceinline__ void upper_pair(int p, int t, int& i, int& j) {
  int row = 0, n = t - 1;
  while (p >= n) {
    p -= n;
    ++row;
    --n;
  }
  i = row;
  j = row + 1 + p;
}

// A lane's four consecutive rows of one column.
struct GfOp {
  d2u a, b;
  __device__ __forceinline__ double operator[](int s) const { return s < 2 ? a[s] : b[s - 2]; }
};

__device__ __forceinline__ GfOp gf_load(const double* p) {
  return {*reinterpret_cast<const d2u*>(p), *reinterpret_cast<const d2u*>(p + 2)};
}

// the same past the last whole step: `left` rows remain, the others are zero
__device__ __forceinline__ GfOp gf_load_tail(const double* p, int left) {
  GfOp o;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    o.a[s] = s < left ? p[s] : 0.0;
    o.b[s] = s + 2 < left ? p[s + 2] : 0.0;
  }
  return o;
}

// Row i of a unit's fragments, one step: x_i^T y_j, and with DIAG (j >= i) x_i^T x_j.
template <int NF, bool DIAG>
__device__ __forceinline__ void gf_row(d4* acc, int i, const GfOp (&x)[NF], const GfOp (&y)[NF]) {
  constexpr int NH = NF * (NF + 1) / 2;
  const int n0 = DIAG ? i * NF - i * (i + 1) / 2 : i * NF;  // + j: fragment (i, j)
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int j = DIAG ? i : 0; j < NF; ++j)
      acc[n0 + j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][s], y[j][s], acc[n0 + j], 0, 0, 0);
    if constexpr (DIAG) {
#pragma unroll
      for (int j = i; j < NF; ++j)
        acc[NH + n0 + j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i][s], x[j][s], acc[NH + n0 + j], 0, 0, 0);
    }
  }
}

template <int NF, bool DIAG>
__device__ __forceinline__ void gf_unit(const double* __restrict__ A, const double* __restrict__ B, int64_t nd, int ns,
                                        int ti, int tj, int64_t s0, int64_t s1, double* __restrict__ out,
                                        double (&red)[kGfWaves][4][256]) {
  constexpr int NA = DIAG ? NF * (NF + 1) : NF * NF;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, r = lane & 15;
  const double* pa[NF];
  const double* pb[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {  // columns past ns repeat the last one: never stored
    pa[f] = A + (int64_t)min((ti * NF + f) * 16 + r, ns - 1) * nd + 4 * g;
    pb[f] = B + (int64_t)min((tj * NF + f) * 16 + r, ns - 1) * nd + 4 * g;
  }
  d4 acc[NA];
#pragma unroll
  for (int n = 0; n < NA; ++n) acc[n] = d4{0.0, 0.0, 0.0, 0.0};

  const int64_t whole = nd / kGfStep;  // steps with all their rows
  const int64_t e = s1 < whole ? s1 : whole;
  int64_t st = s0 + wave;
  // An operand is refilled for the wave's next step as soon as its last MFMA of this one is
  // issued: row by row where nothing below the diagonal is formed; with all NF x NF fragments
  // the second operand is needed to the end and has two sets of registers.
  GfOp x[NF], y[NF];
  auto next = [&](int64_t t) { return (t + kGfWaves < e ? t + kGfWaves : t) * kGfStep; };
  if (st < e) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      x[f] = gf_load(pa[f] + st * kGfStep);
      y[f] = gf_load(pb[f] + st * kGfStep);
    }
    if constexpr (DIAG) {
      for (; st < e; st += kGfWaves) {
        const int64_t nx = next(st);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          gf_row<NF, true>(acc, i, x, y);
          __builtin_amdgcn_sched_barrier(0);
          x[i] = gf_load(pa[i] + nx);
          y[i] = gf_load(pb[i] + nx);
        }
      }
    } else {
      GfOp z[NF];
      auto step = [&](GfOp(&cur)[NF], GfOp(&nxt)[NF]) {
        const int64_t nx = next(st);
#pragma unroll
        for (int f = 0; f < NF; ++f) nxt[f] = gf_load(pb[f] + nx);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          gf_row<NF, false>(acc, i, x, cur);
          __builtin_amdgcn_sched_barrier(0);
          x[i] = gf_load(pa[i] + nx);
        }
        st += kGfWaves;
      };
      while (st < e) {
        step(y, z);
        if (st >= e) break;
        step(z, y);
      }
    }
  }
  if (st == whole && st < s1) {  // the ragged last step
    const int left = (int)(nd - whole * kGfStep) - 4 * g;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      x[f] = gf_load_tail(pa[f] + whole * kGfStep, left);
      y[f] = gf_load_tail(pb[f] + whole * kGfStep, left);
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) gf_row<NF, DIAG>(acc, i, x, y);
  }

#pragma unroll
  for (int b = 0; b < NA; b += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (b + q < NA) *reinterpret_cast<d4*>(&red[wave][q][lane * 4]) = acc[b + q];
    __syncthreads();
    if (b + wave < NA) {
      d4 sum = *reinterpret_cast<const d4*>(&red[0][wave][lane * 4]);
#pragma unroll
      for (int w = 1; w < kGfWaves; ++w) sum += *reinterpret_cast<const d4*>(&red[w][wave][lane * 4]);
      *reinterpret_cast<d4*>(out + (int64_t)(b + wave) * 256 + lane * 4) = sum;
    }
    __syncthreads();
  }
}

template <int NF>
__global__ __launch_bounds__(64 * kGfWaves, 2) void gram_both_kernel(const double* __restrict__ X,
                                                                     const double* __restrict__ Y, int64_t nd, int ns,
                                                                     GramBothPlan p, double* __restrict__ partial) {
  __shared__ __align__(32) double red[kGfWaves][4][256];
  // consecutive ids go to the 8 XCDs in turn: an XCD takes a contiguous run of (split, unit)
  const int64_t nb = (int64_t)p.units * p.splits;
  const int64_t logical = (int64_t)(blockIdx.x % 8) * ((nb + 7) / 8) + blockIdx.x / 8;
  if (logical >= nb || blockIdx.x / 8 >= (nb + 7) / 8) return;
  const int split = (int)(logical / p.units), u = (int)(logical % p.units);
  const int64_t s0 = (int64_t)split * p.steps, s1 = s0 + p.steps;
  constexpr int nd_frags = NF * (NF + 1);
  double* out = partial + (int64_t)split * p.frags * 256;
  if (u < p.t) {
    gf_unit<NF, true>(X, Y, nd, ns, u, u, s0, s1, out + (int64_t)u * nd_frags * 256, red);
  } else {
    const int v = u - p.t;
    int i, j;
    upper_pair(v >> 1, p.t, i, j);
    gf_unit<NF, false>(X, (v & 1) ? X : Y, nd, ns, i, j, s0, s1,
                       out + ((int64_t)p.t * nd_frags + (int64_t)v * NF * NF) * 256, red);
  }
}

// One fragment of one product: the splits' partials in four interleaved sums, added in order;
// entries above the diagonal are mirrored.
__global__ __launch_bounds__(1024) void gram_both_sum_kernel(const double* __restrict__ partial, GramBothPlan p, int ns,
                                                             double* __restrict__ Hs, double* __restrict__ Ms) {
  __shared__ double red[4][256];
  const int e = threadIdx.x & 255, q = threadIdx.x >> 8;
  const double* src = partial + (int64_t)blockIdx.x * 256 + e;
  const int64_t stride = (int64_t)p.frags * 256;
  double sum = 0.0;
#pragma unroll 4
  for (int s = q; s < p.splits; s += 4) sum += src[s * stride];
  red[q][e] = sum;
  __syncthreads();
  if (q != 0) return;
  sum = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
  const int nf = p.nf, ndf = nf * (nf + 1);
  int f = blockIdx.x, ti, tj, a, b, prod;
  if (f < p.t * ndf) {
    ti = tj = f / ndf;
    f -= ti * ndf;
    prod = f >= ndf / 2;
    f -= prod * (ndf / 2);
    a = 0;
    while (f >= nf - a) {
      f -= nf - a;
      ++a;
    }
    b = a + f;
  } else {
    f -= p.t * ndf;
    const int v = f / (nf * nf);
    f -= v * nf * nf;
    prod = v & 1;
    upper_pair(v >> 1, p.t, ti, tj);
    a = f / nf;
    b = f % nf;
  }
  // D[i][j] of a fragment: lane j + 16 (i % 4), register i / 4
  const int lane = e >> 2, reg = e & 3;
  const int i = (ti * nf + a) * 16 + (lane >> 4) + 4 * reg, j = (tj * nf + b) * 16 + (lane & 15);
  if (i >= ns || j >= ns || i > j) return;
  double* C = prod ? Ms : Hs;
  C[(int64_t)i + (int64_t)j * ns] = sum;
  C[(int64_t)j + (int64_t)i * ns] = sum;
}

}  // namespace

GramBothPlan plan_gram_both(int64_t nd, int ns) {
  GramBothPlan p;
  const int frags = (ns + 15) / 16;
  p.t = (frags + 3) / 4;
  p.nf = (frags + p.t - 1) / p.t;
  p.units = p.t * p.t;
  p.frags = p.t * p.nf * (p.nf + 1) + p.t * (p.t - 1) * p.nf * p.nf;
  const int64_t steps = (nd + kGfStep - 1) / kGfStep;
  // K splits: two blocks on every CU (one unit: one), and beyond that as many as keep 96 steps
  // in a chunk, up to 160 (96 from 16 units on, where more only adds partials: 72^3, 600
  // orbitals 5290 / 5220 us at 96 / 160); then down to the next count whose last round of
  // blocks is nearly full (72^3, 100 orbitals: 160 splits 304 us, 128 266).  One unit: 72^3, 40
  // orbitals 98 / 63 / 71 us at 128 / 256 / 384 splits.
  int64_t splits;
  if (p.units == 1) {
    splits = 256;
  } else {
    const int64_t most = std::min<int64_t>({p.units < 16 ? 160 : 96, steps / 96, 12288 / p.units});
    const int64_t target = std::max<int64_t>({1, kGfRound / p.units, most});
    auto fill = [&](int64_t n) { return (double)(n * p.units) / (double)((n * p.units + kGfRound - 1) / kGfRound * kGfRound); };
    splits = target;
    for (int64_t n = target; 5 * n >= 3 * target && n >= 1; --n) {
      if (fill(n) > fill(splits)) splits = n;
      if (fill(splits) >= 0.93) break;
    }
  }
  splits = std::max<int64_t>(1, std::min<int64_t>(splits, steps / 8));
  p.steps = (steps + splits - 1) / splits;
  p.splits = (int)((steps + p.steps - 1) / p.steps);
  p.bytes = (size_t)p.splits * p.frags * 256 * sizeof(double);
  return p;
}

hipError_t launch_gram_both(const double* X, const double* Y, int64_t nd, int ns, const GramBothPlan& p,
                            double* partial, double* Hs, double* Ms, hipStream_t s) {
  const int64_t nb = (int64_t)p.units * p.splits;
  const dim3 grid((unsigned)((nb + 7) / 8 * 8)), block(64 * kGfWaves);
  switch (p.nf) {
    case 1: hipLaunchKernelGGL(gram_both_kernel<1>, grid, block, 0, s, X, Y, nd, ns, p, partial); break;
    case 2: hipLaunchKernelGGL(gram_both_kernel<2>, grid, block, 0, s, X, Y, nd, ns, p, partial); break;
    case 3: hipLaunchKernelGGL(gram_both_kernel<3>, grid, block, 0, s, X, Y, nd, ns, p, partial); break;
    case 4: hipLaunchKernelGGL(gram_both_kernel<4>, grid, block, 0, s, X, Y, nd, ns, p, partial); break;
    default: return hipErrorInvalidConfiguration;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_both_sum_kernel, dim3((unsigned)p.frags), dim3(1024), 0, s, partial, p, ns, Hs, Ms);
  return hipGetLastError();
}

}  // namespace chefsi
