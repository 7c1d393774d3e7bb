// Split-bf16 contractions of the mixed-precision projection and rotation (gfx950 MFMA).
//
// Each FP32 operand value x is written as x = hi + lo + O(2^-17 |x|) with
// hi = bf16(x) and lo = bf16(x - hi) (round to nearest even), and a product as
// a b ~ a_hi b_hi + a_hi b_lo + a_lo b_hi: three bf16 MFMAs with FP32
// accumulation, error about 2^-15 |a b| per product (the dropped a_lo b_lo term
// and the two representation errors).  The Cholesky of Ms, the eigensolve and the
// final Rayleigh-Ritz pass stay in FP64 elsewhere.
//
// v_mfma_f32_32x32x16_bf16 lane layout (measured): A[i][k] comes from lane
// i + 32 (k / 8), element k % 8; B[k][j] from lane j + 32 (k / 8), element k % 8;
// D[i][j] lands in lane j + 32 ((i / 4) % 2), register 4 (i / 8) + i % 4, i.e.
// lane l, register v holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.
//
// Projection (Alg. 1; Sec. 2.2): partial[split][tile] = A(:, I)^T B(:, J) over one
//   K chunk, 128 x 128 upper tiles, the same split-K plan and partial layout as the
//   FP64 kernel (so the FP64 fixed-order reduction is shared).  Both operands are
//   contiguous along K, so 32-wide K stages of both tiles are split into hi/lo and
//   staged through double-buffered LDS (one barrier per stage).
// Rotation (Alg. 1; Sec. 2.4): O = X Z computed as O^T = Z^T X^T.  Z is split once
//   into bf16 hi/lo arrays (zero padded, so the K tail needs no masking); a block
//   stages a 128-column slice of Z through LDS and every wave gathers the MFMA B
//   operand straight from X: lane l reads grid point p = l % 32 of 8 consecutive
//   columns, so each load instruction covers 128 contiguous bytes of two columns and
//   no transpose is needed.  Results leave as 128-byte rows of O.  A stage's 48 MFMA take
//   1536 cycles of a SIMD; the vector work beside them has to stay below that (addresses
//   formed per lane, single conversions and the copy of the next stage's values made it 1900,
//   now 400), after which the power limit holds the clock near 1.6 GHz.  60x60x180, 1200
//   orbitals: 6.6 -> 5.7 ms, 0.85 -> 0.98 PFLOP/s executed.
#include "common.h"

#include <algorithm>

namespace chefsi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // rows of odd length are only 4-byte aligned

namespace {

constexpr int kT = 128;        // projection block tile (both dimensions)
constexpr int kKS = 32;        // K per stage
constexpr int kLd = kKS + 8;   // LDS row stride in bf16 (80 bytes: conflict-free 16-byte reads)
constexpr int kRotJ = 128;     // rotation: output columns per block
constexpr int kRotP = 256;     // rotation: grid points per block (64 per wave)
constexpr int kSubStages = 512;  // projection: K stages summed in FP32 before an FP64 flush (16384 rows)


__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// x = hi + lo with hi = bf16(x), lo = bf16(x - hi), both round-to-nearest-even; two values at a
// time, so one conversion instruction makes two (a rotation stage: 96 instead of 128).
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
  u32x4 h4, l4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x2 v = {x[2 * e], x[2 * e + 1]};
    const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
    const f32x2 r = {x[2 * e] - __builtin_bit_cast(float, h << 16),
                     x[2 * e + 1] - __builtin_bit_cast(float, h & 0xffff0000u)};
    h4[e] = h;
    l4[e] = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
  }
  hi = __builtin_bit_cast(bf16x8, h4);
  lo = __builtin_bit_cast(bf16x8, l4);
}

__device__ __forceinline__ u32x4 as_u4(bf16x8 v) { return __builtin_bit_cast(u32x4, v); }
__device__ __forceinline__ bf16x8 as_bf8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ void upper_tile_of(int t, int nt, int& ti, int& tj) {
  int i = 0;
  int row = nt;
  while (t >= row) {
    t -= row;
    ++i;
    --row;
  }
  ti = i;
  tj = i + t;
}

}  // namespace

// ---------------------------------------------------------------------------
// Projection partial tiles.
// ---------------------------------------------------------------------------
struct GramStage {
  float a[16];
  float b[16];
};

// Thread t stages row t / 2 of both tiles: the 16 elements k .. k + 15 (k = stage start
// + 16 (t % 2)) of rows pa and pb; elements at or past ke read as zero unless full.
__device__ __forceinline__ void gram_load(GramStage& st, const float* __restrict__ pa, const float* __restrict__ pb,
                                          int64_t k, int64_t ke, bool full) {
  if (full) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4u va = *reinterpret_cast<const f32x4u*>(pa + k + 4 * q);
      const f32x4u vb = *reinterpret_cast<const f32x4u*>(pb + k + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        st.a[4 * q + e] = va[e];
        st.b[4 * q + e] = vb[e];
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const bool ok = k + e < ke;
      st.a[e] = ok ? pa[k + e] : 0.f;
      st.b[e] = ok ? pb[k + e] : 0.f;
    }
  }
}

__device__ __forceinline__ void gram_store_lds(const GramStage& st, __bf16* ah, __bf16* al, __bf16* bh, __bf16* bl,
                                               int off) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float xa[8], xb[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xa[e] = st.a[8 * q + e];
      xb[e] = st.b[8 * q + e];
    }
    bf16x8 h, l;
    split8(xa, h, l);
    *reinterpret_cast<u32x4*>(ah + off + 8 * q) = as_u4(h);
    *reinterpret_cast<u32x4*>(al + off + 8 * q) = as_u4(l);
    split8(xb, h, l);
    *reinterpret_cast<u32x4*>(bh + off + 8 * q) = as_u4(h);
    *reinterpret_cast<u32x4*>(bl + off + 8 * q) = as_u4(l);
  }
}

// FP32 accumulators of a wave's 64 x 64 part into the FP64 partial tile (added to what the
// same threads stored before when `add`), then cleared.  One writer per element, fixed order.
__device__ __forceinline__ void flush_tile(f32x16 (&acc)[2][2], double* __restrict__ pt, int wm, int wn, int g,
                                           int r32, bool add) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ii = wm * 64 + i * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
        const int jj = wn * 64 + j * 32 + r32;
        double* q = pt + ii * kT + jj;
        *q = add ? *q + (double)acc[i][j][v] : (double)acc[i][j][v];
        acc[i][j][v] = 0.f;
      }
}

// two blocks per CU (80 KB of LDS each, at most 256 registers per lane): a second wave on
// every SIMD hides the global-load and LDS latency of the other (measured 14-22 % faster
// than one wave per SIMD on 72^3 to 120^3 blocks)
__global__ __launch_bounds__(256, 2) void gram_bf16x3_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                          int64_t nd, int ns, int nt, int ntiles, int64_t kchunk,
                                                          double* __restrict__ partial) {
  // [buffer][hi A, lo A, hi B, lo B][128 rows][kLd]
  __shared__ __attribute__((aligned(16))) __bf16 lds[2][4][kT * kLd];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int tile = blockIdx.x % ntiles;
  const int split = blockIdx.x / ntiles;
  int ti, tj;
  upper_tile_of(tile, nt, ti, tj);
  const int64_t kb = (int64_t)split * kchunk;
  const int64_t ke = min(nd, kb + kchunk);

  const int lrow = tid >> 1;       // staged row
  const int lhalf = tid & 1;       // staged K half
  const int ra = min(ti * kT + lrow, ns - 1);
  const int rb = min(tj * kT + lrow, ns - 1);
  const float* pa = A + (int64_t)ra * nd;
  const float* pb = B + (int64_t)rb * nd;
  const int st_off = lrow * kLd + 16 * lhalf;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nstage = (int)((ke - kb + kKS - 1) / kKS);
  // partial tile, row-major 128 x 128: element (ii, jj) at ii * 128 + jj
  double* pt = partial + ((int64_t)split * ntiles + tile) * (kT * kT);
  GramStage st;
  if (nstage > 0) {
    gram_load(st, pa, pb, kb + 16 * lhalf, ke, kb + kKS <= ke);
    gram_store_lds(st, lds[0][0], lds[0][1], lds[0][2], lds[0][3], st_off);
  }
  __syncthreads();

  const int r32 = lane & 31, g = lane >> 5;
  for (int t = 0; t < nstage; ++t) {
    const int buf = t & 1;
    const bool more = t + 1 < nstage;
    const int64_t kn = kb + (int64_t)(t + 1) * kKS;
    if (more) gram_load(st, pa, pb, kn + 16 * lhalf, ke, kn + kKS <= ke);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int oa = (wm * 64 + f * 32 + r32) * kLd + 16 * s + 8 * g;
        const int ob = (wn * 64 + f * 32 + r32) * kLd + 16 * s + 8 * g;
        ah[f] = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][0] + oa));
        al[f] = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][1] + oa));
        bh[f] = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][2] + ob));
        bl[f] = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][3] + ob));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(al[i], bh[j], acc[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(ah[i], bl[j], acc[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(ah[i], bh[j], acc[i][j]);
    }
    if (more) gram_store_lds(st, lds[buf ^ 1][0], lds[buf ^ 1][1], lds[buf ^ 1][2], lds[buf ^ 1][3], st_off);
    // every kSubStages stages the FP32 sums move into the FP64 partial tile (FP32 sums span
    // at most kSubStages * kKS rows of K)
    if ((t + 1) % kSubStages == 0 && more) {
      flush_tile(acc, pt, wm, wn, g, r32, t + 1 > kSubStages);
    }
    __syncthreads();
  }
  flush_tile(acc, pt, wm, wn, g, r32, nstage > kSubStages);
}

hipError_t launch_gram_bf16x3(const float* A, const float* B, int64_t nd, int ns, const GramPlan& p,
                              double* partial, hipStream_t s) {
  if (p.tile != kT) return hipErrorInvalidValue;
  dim3 grid((unsigned)(p.ntiles * p.splits));
  hipLaunchKernelGGL(gram_bf16x3_kernel, grid, dim3(256), 0, s, A, B, nd, ns, p.nt, p.ntiles, p.kchunk, partial);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Both products of the projection at once: a unit is 256 rows of X (block I) against 128
// columns of X and the same 128 columns of Y (block J >= 2 I), i.e. 256 x 128 elements of Ms
// and of Hs.
//
// The 128 x 128 kernel above is bound by its operand stream, not by MFMA: at 120^3, Ns 1800
// its two products read 424 GB through L2 with 80 % misses (3.9 TB/s of them) while MFMA was
// busy 24 % of the cycles.  The unit stages 512 rows for 256 x 256 results where four of the
// 128-wide tiles stage 1024, and splits each staged value half as often.
//
// One block per CU (512 threads, 128 KB of LDS, 256 registers a lane; 53 spill, which are read
// back between K loops, where sums go out, and not inside one).  Wave (wm, wn) holds
// 64 rows x 128 columns, wn = 0 the columns of X, wn = 1 those of Y.  A 32-wide K stage lies
// in LDS as 64-byte rows of hi and of lo; 16-byte chunk c of row r sits at chunk
// c ^ (r / 4) % 4, so the eight rows that a read covers at a time fall on distinct banks.
// Measured, both products with their sums: 120^3, Ns 1800: 77.3 -> 36.7 ms (1185 TF/s executed
// bf16, MFMA busy 69 % of the cycles at the 1.62 GHz the power limit leaves, L2 hits 65 %);
// 60x60x180, Ns 1200: 11.95 -> 6.83 ms; 72^3, Ns 600: 1.94 -> 1.62 ms.
// During stage t a thread splits its eight row pieces of stage t + 1 into the other buffer,
// six MFMAs apart, and refetches each piece for stage t + 2 as soon as it is split: every
// global load has a whole stage to arrive and the splits run under the MFMAs.
// ---------------------------------------------------------------------------
namespace {
constexpr int kPI = 256, kPJ = 128;
constexpr int kPairThreads = 512;
constexpr int kPairRows = kPI + 2 * kPJ;  // staged rows: X(:, I), X(:, J), Y(:, J)
constexpr int kPairPasses = 8;            // row pieces a thread stages: rows 64 q + tid / 8
constexpr int kPairSub = kSubStages * kKS;  // rows summed in FP32 before an FP64 flush

__device__ __forceinline__ void pair_unit_of(int u, int nj, int& bi, int& bj) {
  bi = 0;
  int row = nj;
  while (u >= row) {
    u -= row;
    ++bi;
    row -= 2;
  }
  bj = 2 * bi + u;
}

__device__ __forceinline__ void pair_flush(f32x16 (&acc)[2][4], double* __restrict__ pt, int wm, int wn, int g, int r32,
                                           bool add) {
  int64_t zero = 0;  // keeps the 128 addresses from being formed ahead of the K loop
  asm volatile("" : "+s"(zero));
  pt += zero;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ii = wm * 64 + i * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
        const int jj = wn * kPJ + j * 32 + r32;
        double* q = pt + ii * (2 * kPJ) + jj;
        *q = add ? *q + (double)acc[i][j][v] : (double)acc[i][j][v];
        acc[i][j][v] = 0.f;
      }
}

// hi and lo of two values at once (one packed conversion each), as split_bf16
__device__ __forceinline__ void split2(f32x2 x, bf16x2& hi, bf16x2& lo) {
  hi = __builtin_convertvector(x, bf16x2);
  lo = __builtin_convertvector(x - __builtin_convertvector(hi, f32x2), bf16x2);
}

__device__ __forceinline__ void pair_split_store(const f32x4u& x, __bf16* ph, __bf16* pl) {
  bf16x2 h0, h1, l0, l1;
  split2(f32x2{x[0], x[1]}, h0, l0);
  split2(f32x2{x[2], x[3]}, h1, l1);
  *reinterpret_cast<bf16x4*>(ph) = __builtin_shufflevector(h0, h1, 0, 1, 2, 3);
  *reinterpret_cast<bf16x4*>(pl) = __builtin_shufflevector(l0, l1, 0, 1, 2, 3);
}
}  // namespace

// First row of group g of `groups`: near g / groups of the rows, at a place where the FP32
// sums of the 128 x 128 kernel end too (a multiple of kPairSub rows inside a K chunk, or a
// chunk's end), so both kernels form the same FP32 sums.
__device__ __forceinline__ int64_t pair_bound(int g, int groups, int64_t nd, int64_t kchunk) {
  if (g <= 0) return 0;
  if (g >= groups) return nd;
  const int64_t r = nd / groups * g, c0 = r / kchunk * kchunk;
  const int64_t in = (r - c0 + kPairSub / 2) / kPairSub * kPairSub;
  return min(nd, min(c0 + in, c0 + kchunk));
}

__global__ __launch_bounds__(kPairThreads, 2) void gram_pair_kernel(const float* __restrict__ X,
                                                                    const float* __restrict__ Y, int64_t nd, int ns,
                                                                    int nj, int nunits, int nblocks, int per_xcd,
                                                                    int groups, int64_t kchunk,
                                                                    double* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) __bf16 lds[2][2][kPairRows * kKS];  // [buffer][hi, lo][row][32]
  const int logical = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (logical >= nblocks) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave & 3, wn = wave >> 2;
  const int unit = logical % nunits, group = logical / nunits;
  int bi, bj;
  pair_unit_of(unit, nj, bi, bj);

  const int lr = tid >> 3, lc = tid & 7;
  const float* col[kPairPasses];
#pragma unroll
  for (int q = 0; q < kPairPasses; ++q) {
    const int row = 64 * q + lr;
    const int c = q < 4 ? bi * kPI + row : bj * kPJ + (row - kPI) % kPJ;
    col[q] = (q < 6 ? X : Y) + (int64_t)min(c, ns - 1) * nd + 4 * lc;
  }
  const int st_off = lr * kKS + ((((lc >> 1) ^ (lr >> 2)) & 3) << 3) + 4 * (lc & 1);

  f32x16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int r32 = lane & 31, g = lane >> 5, key = (r32 >> 2) & 3;
  const int oa = (wm * 64 + r32) * kKS, ob = (kPI + wn * kPJ + r32) * kKS;
  // partial results, row-major 256 x (128 of Ms, 128 of Hs)
  double* pt = partial + ((int64_t)group * nunits + unit) * (kPI * 2 * kPJ);
  const int64_t r1 = pair_bound(group + 1, groups, nd, kchunk);
  bool flushed = false;
  f32x4u st[kPairPasses];
  for (int64_t kb = pair_bound(group, groups, nd, kchunk); kb < r1;) {
    // one FP32 sum: rows kb .. ke
    const int64_t c0 = kb / kchunk * kchunk;
    const int64_t ke = min(min(c0 + kchunk, nd), kb + kPairSub);
    const int nfull = (int)((ke - kb) / kKS);
    const float* src[kPairPasses];
#pragma unroll
    for (int q = 0; q < kPairPasses; ++q) src[q] = col[q] + kb;
    if (nfull > 0) {
#pragma unroll
      for (int q = 0; q < kPairPasses; ++q) st[q] = *reinterpret_cast<const f32x4u*>(src[q]);
#pragma unroll
      for (int q = 0; q < kPairPasses; ++q)
        pair_split_store(st[q], lds[0][0] + st_off + 64 * q * kKS, lds[0][1] + st_off + 64 * q * kKS);
      const int64_t k1 = (int64_t)min(1, nfull - 1) * kKS;
#pragma unroll
      for (int q = 0; q < kPairPasses; ++q) st[q] = *reinterpret_cast<const f32x4u*>(src[q] + k1);
    }
    __syncthreads();
    for (int t = 0; t < nfull; ++t) {
      const __bf16* lh = lds[t & 1][0];
      const __bf16* ll = lds[t & 1][1];
      __bf16* nh = lds[(t & 1) ^ 1][0];
      __bf16* nl = lds[(t & 1) ^ 1][1];
      // past the last full stage the pieces are refetched and staged again, unread
      const int64_t kn = (int64_t)min(t + 2, nfull - 1) * kKS;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int ch = ((2 * s + g) ^ key) << 3;
        bf16x8 ah[2], al[2], bh[4], bl[4];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          ah[f] = as_bf8(*reinterpret_cast<const u32x4*>(lh + oa + f * 32 * kKS + ch));
          al[f] = as_bf8(*reinterpret_cast<const u32x4*>(ll + oa + f * 32 * kKS + ch));
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          bh[f] = as_bf8(*reinterpret_cast<const u32x4*>(lh + ob + f * 32 * kKS + ch));
          bl[f] = as_bf8(*reinterpret_cast<const u32x4*>(ll + ob + f * 32 * kKS + ch));
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {  // MFMAs 6 c .. 6 c + 5 of the 24, then one staged piece
#pragma unroll
          for (int m = 6 * c; m < 6 * c + 6; ++m) {
            const int p = m / 8, i = (m % 8) / 4, j = m % 4;
            acc[i][j] = p == 0 ? mfma_bf16(al[i], bh[j], acc[i][j])
                               : (p == 1 ? mfma_bf16(ah[i], bl[j], acc[i][j]) : mfma_bf16(ah[i], bh[j], acc[i][j]));
          }
          const int q = 4 * s + c;
          pair_split_store(st[q], nh + st_off + 64 * q * kKS, nl + st_off + 64 * q * kKS);
          st[q] = *reinterpret_cast<const f32x4u*>(src[q] + kn);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    }
    if (kb + (int64_t)nfull * kKS < ke) {  // rows past the last full stage (zeros beyond ke)
      const int64_t k0 = (int64_t)nfull * kKS;
#pragma unroll
      for (int q = 0; q < kPairPasses; ++q) {
        f32x4u x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = kb + k0 + 4 * lc + e < ke ? src[q][k0 + e] : 0.f;
        pair_split_store(x, lds[0][0] + st_off + 64 * q * kKS, lds[0][1] + st_off + 64 * q * kKS);
      }
      __syncthreads();
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int ch = ((2 * s + g) ^ key) << 3;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bf16x8 ah = as_bf8(*reinterpret_cast<const u32x4*>(lds[0][0] + oa + i * 32 * kKS + ch));
          const bf16x8 al = as_bf8(*reinterpret_cast<const u32x4*>(lds[0][1] + oa + i * 32 * kKS + ch));
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bf16x8 bh = as_bf8(*reinterpret_cast<const u32x4*>(lds[0][0] + ob + j * 32 * kKS + ch));
            const bf16x8 bl = as_bf8(*reinterpret_cast<const u32x4*>(lds[0][1] + ob + j * 32 * kKS + ch));
            acc[i][j] = mfma_bf16(al, bh, acc[i][j]);
            acc[i][j] = mfma_bf16(ah, bl, acc[i][j]);
            acc[i][j] = mfma_bf16(ah, bh, acc[i][j]);
          }
        }
      }
      __syncthreads();  // the next sum stages into the same buffer
    }
    pair_flush(acc, pt, wm, wn, g, r32, flushed);
    flushed = true;
    kb = ke;
  }
  if (!flushed) pair_flush(acc, pt, wm, wn, g, r32, false);  // a group without rows: zeros
}

// Hs(i, j) = Hs(j, i) and Ms(i, j) = Ms(j, i): the units' partial results of element (i, j),
// i <= j, summed over the K chunks in a fixed order.
__global__ __launch_bounds__(256) void gram_pair_reduce_kernel(const double* __restrict__ partial, int ns, int nj,
                                                               int nunits, int splits, double* __restrict__ Hs,
                                                               double* __restrict__ Ms) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  int bi, bj;
  pair_unit_of(blockIdx.y, nj, bi, bj);
  const int i = bi * kPI + e / (2 * kPJ), jj = e % (2 * kPJ), j = bj * kPJ + jj % kPJ;
  if (i > j || j >= ns) return;
  double s = 0.0;
  for (int q = 0; q < splits; ++q) s += partial[((int64_t)q * nunits + blockIdx.y) * (kPI * 2 * kPJ) + e];
  double* C = jj < kPJ ? Ms : Hs;
  C[(int64_t)j * ns + i] = s;
  C[(int64_t)i * ns + j] = s;
}

PairPlan plan_gram_pair(int64_t nd, int ns, const GramPlan& gp, size_t bytes) {
  PairPlan p;
  p.nj = (ns + kPJ - 1) / kPJ;
  p.nunits = 0;
  for (int j = p.nj; j > 0; j -= 2) p.nunits += j;
  // groups of rows: whole rounds of one block per CU, no shorter than the FP32 sums allow,
  // partial results within the given bytes.  The longest group decides a round's length.
  const size_t unit_bytes = (size_t)kPI * 2 * kPJ * sizeof(double);
  const int64_t seg = std::min<int64_t>(gp.kchunk, kPairSub);
  const int64_t most = std::min<int64_t>((int64_t)(bytes / (unit_bytes * p.nunits)), (nd + seg - 1) / seg);
  for (int64_t s = 1; s <= most && s * p.nunits <= 1024; ++s) {
    const int64_t rounds = (s * p.nunits + 255) / 256;
    const int64_t longest = ((nd + s - 1) / s + seg - 1) / seg * seg;  // whole FP32 sums
    const double fill = (double)nd * p.nunits / ((double)rounds * 256.0 * longest);
    if (fill > p.fill + 0.02) {
      p.fill = fill;
      p.groups = (int)s;
    }
  }
  p.kchunk = gp.kchunk;
  p.fill *= (2.0 * gp.ntiles * kT * kT) / ((double)p.nunits * kPI * 2 * kPJ);
  return p;
}

hipError_t launch_gram_pair_bf16x3(const float* X, const float* Y, int64_t nd, int ns, const PairPlan& p,
                                   double* partial, double* Hs, double* Ms, hipStream_t s) {
  const int nblocks = p.nunits * p.groups;
  const int per_xcd = (nblocks + 7) / 8;
  hipLaunchKernelGGL(gram_pair_kernel, dim3((unsigned)(per_xcd * 8)), dim3(kPairThreads), 0, s, X, Y, nd, ns, p.nj,
                     p.nunits, nblocks, per_xcd, p.groups, p.kchunk, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_pair_reduce_kernel, dim3(kPI * 2 * kPJ / 256, (unsigned)p.nunits), dim3(256), 0, s, partial,
                     ns, p.nj, p.nunits, p.groups, Hs, Ms);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Rotation.
// ---------------------------------------------------------------------------
size_t zsplit_ld(int ns) { return (size_t)((ns + kKS - 1) / kKS) * kKS; }
size_t zsplit_cols(int ns) { return (size_t)((ns + kRotJ - 1) / kRotJ) * kRotJ; }
size_t zsplit_bytes(int ns) { return 2 * zsplit_cols(ns) * zsplit_ld(ns) * sizeof(__bf16); }

// zh/zl[j * ld + i] = split of Z[i + j ns] for i < ns, j < ns; zero in the padding.
__global__ void zsplit_kernel(const double* __restrict__ Z, int ns, int ld, int cols, __bf16* __restrict__ zh,
                              __bf16* __restrict__ zl) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)ld * cols) return;
  const int i = (int)(e % ld);
  const int j = (int)(e / ld);
  __bf16 h = (__bf16)0.f, l = (__bf16)0.f;
  if (i < ns && j < ns) {
    const double z = Z[i + (int64_t)j * ns];
    h = (__bf16)(float)z;
    l = (__bf16)(float)(z - (double)(float)h);
  }
  zh[e] = h;
  zl[e] = l;
}

// Lane (r32, g) of fragment f holds X[i][pcol[f]] for the 8 columns i = k0 + 16 s + 8 g + e
// of each 16-wide K step s.  A column's address is a scalar one (its first for g = 0, the base
// of a buffer) and the lane's byte offset, the same for all of them (8 g columns and the point,
// below 2^31 bytes: a handle has at most 2^31 / 48 points), so a load costs no vector
// instructions.  In the stage that passes ns the lanes form 64-bit addresses, columns past ns
// clamped (Z is zero there).
__device__ __forceinline__ void rot_load_x(float (&xv)[2][2][8], const float* __restrict__ X, int64_t nd, int ns,
                                           const int64_t (&pcol)[2], const unsigned (&voff)[2], int k0, int g) {
  if (k0 + kKS <= ns) {
    const float* row = X + (int64_t)k0 * nd;
    const int bytes = 36 * (int)nd;  // nine columns: a lane's own lies 0 or 8 further
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(row), (short)0, bytes, 0x00020000);
#pragma unroll
        for (int f = 0; f < 2; ++f)
          xv[s][f][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff[f], 0, 0));
        row += nd;
      }
      row += 8 * nd;
    }
    return;
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = min(k0 + 16 * s + 8 * g + e, ns - 1);
      const float* row = X + (int64_t)i * nd;
#pragma unroll
      for (int f = 0; f < 2; ++f) xv[s][f][e] = row[pcol[f]];
    }
}

__device__ __forceinline__ void rot_load_z(u32x4 (&zr)[4], const __bf16* __restrict__ pzh,
                                           const __bf16* __restrict__ pzl, int k0) {
  zr[0] = *reinterpret_cast<const u32x4*>(pzh + k0);
  zr[1] = *reinterpret_cast<const u32x4*>(pzh + k0 + 8);
  zr[2] = *reinterpret_cast<const u32x4*>(pzl + k0);
  zr[3] = *reinterpret_cast<const u32x4*>(pzl + k0 + 8);
}

__device__ __forceinline__ void rot_store_z(const u32x4 (&zr)[4], __bf16* sh, __bf16* sl) {
  *reinterpret_cast<u32x4*>(sh) = zr[0];
  *reinterpret_cast<u32x4*>(sh + 8) = zr[1];
  *reinterpret_cast<u32x4*>(sl) = zr[2];
  *reinterpret_cast<u32x4*>(sl + 8) = zr[3];
}

// JF: 32-wide fragments of a block's columns (4: kRotJ).  Up to 64 orbitals one block has them all,
// and a narrower one needs fewer registers (90 and 204 against 256), so more blocks hide each
// other's single or double stage: 120^3, 8 / 24 / 48 orbitals 75.7 / 97 / 186 us with four
// fragments, 26.4 / 60.2 / 149 with one or two.
template <int JF>
__global__ __launch_bounds__(256, JF == 1 ? 4 : 2) void rotate_bf16x3_kernel(
    const float* __restrict__ X, const __bf16* __restrict__ zh, const __bf16* __restrict__ zl, float* __restrict__ O,
    int64_t nd, int ns, int ld, int npt, int njt, int per_xcd) {
  __shared__ __attribute__((aligned(16))) __bf16 lds[2][2][32 * JF * kLd];  // [buffer][hi, lo][j][kLd]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // blocks are dealt to the 8 XCDs round-robin; a contiguous run of logical tiles per
  // XCD keeps the njt blocks that read one slab of X on one L2
  const int b = blockIdx.x;
  const int logical = (b % 8) * per_xcd + b / 8;
  if (logical >= npt * njt) return;
  const int ptile = logical / njt, jtile = logical % njt;
  const int j0 = jtile * kRotJ;
  const int64_t p0 = (int64_t)ptile * kRotP + wave * 64;

  // Z staging: thread t copies 16 bf16 of column j0 + t / 2 (hi and lo)
  const int zrow = min(tid >> 1, 32 * JF - 1), zhalf = tid & 1;  // (threads past the columns: the last one again)
  const __bf16* pzh = zh + (int64_t)(j0 + zrow) * ld + 16 * zhalf;
  const __bf16* pzl = zl + (int64_t)(j0 + zrow) * ld + 16 * zhalf;
  const int zoff = zrow * kLd + 16 * zhalf;

  // X gather: fragment f covers points p0 + 32 f + (lane % 32); K slot 8 (lane / 32) + e
  const int r32 = lane & 31, g = lane >> 5;
  int64_t pcol[2];
  unsigned voff[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    pcol[f] = min(p0 + 32 * f + r32, nd - 1);
    voff[f] = ((unsigned)(8 * g) * (unsigned)nd + (unsigned)pcol[f]) * 4u;
  }

  f32x16 acc[JF][2];  // [j fragment][p fragment]
#pragma unroll
  for (int i = 0; i < JF; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nstage = JF == 1 ? 1 : ld / kKS;  // one fragment: at most 32 columns
  float xa[2][2][8], xb[2][2][8];  // [k16 step][p fragment][e], a stage's and the next one's
  u32x4 zr[4];
  rot_load_z(zr, pzh, pzl, 0);
  rot_load_x(xa, X, nd, ns, pcol, voff, 0, g);
  rot_store_z(zr, lds[0][0] + zoff, lds[0][1] + zoff);
  __syncthreads();

  auto stage = [&](int t, int buf, const float (&xc)[2][2][8], float (&xn)[2][2][8]) {
    const bool more = t + 1 < nstage;
    if (more) {
      rot_load_z(zr, pzh, pzl, (t + 1) * kKS);
      rot_load_x(xn, X, nd, ns, pcol, voff, (t + 1) * kKS, g);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 xh[2], xl[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) split8(xc[s][f], xh[f], xl[f]);
#pragma unroll
      for (int jf = 0; jf < JF; ++jf) {
        const int o = (jf * 32 + r32) * kLd + 16 * s + 8 * g;
        const bf16x8 zhv = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][0] + o));
        const bf16x8 zlv = as_bf8(*reinterpret_cast<const u32x4*>(lds[buf][1] + o));
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[jf][f] = mfma_bf16(zlv, xh[f], acc[jf][f]);
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[jf][f] = mfma_bf16(zhv, xl[f], acc[jf][f]);
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[jf][f] = mfma_bf16(zhv, xh[f], acc[jf][f]);
      }
    }
    if (more) rot_store_z(zr, lds[buf ^ 1][0] + zoff, lds[buf ^ 1][1] + zoff);
    __syncthreads();
  };
  for (int t = 0; t < nstage; t += 2) {
    stage(t, 0, xa, xb);
    if (t + 1 < nstage) stage(t + 1, 1, xb, xa);
  }

  // D[j][p]: lane l, register v -> j = 8 (v / 4) + 4 (l / 32) + v % 4, p = l % 32
#pragma unroll
  for (int jf = 0; jf < JF; ++jf)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int j = j0 + jf * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
      if (j >= ns) continue;
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int64_t p = p0 + 32 * f + r32;
        if (p < nd) O[(int64_t)j * nd + p] = acc[jf][f][v];
      }
    }
}

hipError_t launch_rotate_bf16x3(const float* X, const double* Z, void* zsplit, float* O, int64_t nd, int ns,
                                hipStream_t s) {
  const int ld = (int)zsplit_ld(ns);
  const int cols = (int)zsplit_cols(ns);
  __bf16* zh = static_cast<__bf16*>(zsplit);
  __bf16* zl = zh + (size_t)ld * cols;
  const int64_t nz = (int64_t)ld * cols;
  hipLaunchKernelGGL(zsplit_kernel, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, s, Z, ns, ld, cols, zh, zl);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int npt = (int)((nd + kRotP - 1) / kRotP);
  const int njt = cols / kRotJ;
  const int64_t nb = (int64_t)npt * njt;
  const int per_xcd = (int)((nb + 7) / 8);
  const dim3 grid((unsigned)(per_xcd * 8));
  if (nd > ((int64_t)1 << 31) / 48) return hipErrorInvalidValue;
  if (ns <= 32)
    hipLaunchKernelGGL(rotate_bf16x3_kernel<1>, grid, dim3(256), 0, s, X, zh, zl, O, nd, ns, ld, npt, njt, per_xcd);
  else if (ns <= 64)
    hipLaunchKernelGGL(rotate_bf16x3_kernel<2>, grid, dim3(256), 0, s, X, zh, zl, O, nd, ns, ld, npt, njt, per_xcd);
  else
    hipLaunchKernelGGL(rotate_bf16x3_kernel<4>, grid, dim3(256), 0, s, X, zh, zl, O, nd, ns, ld, npt, njt, per_xcd);
  return hipGetLastError();
}

}  // namespace chefsi
