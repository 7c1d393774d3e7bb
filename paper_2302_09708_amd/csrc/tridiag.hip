// Householder tridiagonalisation of the reduced pencil (first third of the FP64 subspace
// eigensolve, Sec. 2.3) and the back transformation of the tridiagonal eigenvectors.
//
// tridiag_kernel: A = Q T Q^T for a symmetric n x n matrix, upper triangle read, in the
// column order and with the reflector convention of LAPACK's dsytrd (uplo U: column m from
// n - 1 down to 1, v[m - 1] = 1, beta = -sign(alpha) |x|), so any tridiagonal eigensolver
// and back transformation that expects that form can follow.
//   One launch.  The rows of A live in the LDS of G workgroups (row j in workgroup j % G) for
// the whole reduction; every workgroup keeps v and w of the current column in registers and
// forms them for itself, bit for bit the same, so one exchange per column is enough:
//   - each workgroup brings its rows up to date with the previous column's rank-2 update and
//     in the same pass forms its rows of p = A v;
//   - it publishes (p_j, A_j,m-1): the product and the next column's element of its rows;
//   - having all of p and of that column it forms w, the next column after this column's
//     update, and the next reflector, without a second exchange.
// The exchange carries its own validity: a double goes out as two 64-bit words of 32 payload
// bits and the 32-bit number of the column, written and read with relaxed device-scope
// atomics, so no fence, flag or cache maintenance is needed.  Slots alternate between two
// sets: a workgroup writes a set again only after it has read the other one whole.  That one
// holds a slot from every workgroup that reads the first set (tridiag_exchange.h), so nobody
// waits any more for what is written over; a workgroup without a row in the next column
// publishes its last rows and leaves.
//   A cooperative launch has all its workgroups resident at once among the kernels of one
// process.  Workgroups of another process' reduction may hold the compute units that some of
// these need while they wait for each other, so the wait is bounded, and
// tridiag_alone_kernel, one workgroup without an exchange, does the reduction again where it
// was not met.
// Measured (whole reduction / back transformation): n = 40 66 / 11 us, 130 0.35 / 0.04 ms,
// 600 2.18 / 0.26 ms, 1200 6.25 / 0.84 ms; rocSOLVER's blocked reduction launches four to six
// kernels a column: 9.0 / 1.2 ms at n = 600, 0.15 / 0.27 ms at n = 40.  Bound by a column's
// serial chain (two wave sums, a square root, two divisions, LDS round trips) and, with more
// than one workgroup, the exchange: 2.7 us a column at n = 130, 3.6 at 600.
// Above 1024 rows v, w and the rows under way outgrow the 256 registers (65 spilled up to 1216,
// 162 up to 1408, read back in every column); 1200 columns still take 5.2 us each.
// backtransform_kernel: C <- Q C, a wave keeping two columns of C in registers, the
// reflectors applied one after the other from LDS with the next ones already on the way.
#include "common.h"
#include "tridiag_exchange.h"

#include <algorithm>

namespace chefsi {

namespace {

constexpr int kTdThreads = 512;
constexpr int kTdWaves = kTdThreads / 64;
constexpr size_t kTdMaxLds = 160 * 1024;
constexpr int kTdMaxGroups = 192;       // of 256 CUs: one workgroup each
constexpr int kTdMaxChunks = 22;        // 64-wide chunks of a row: n <= 1408
constexpr int kBtThreads = 256;          // back transformation: two columns of C per wave
constexpr int kBtWaves = kBtThreads / 64;
constexpr int kBtRefl = 4;

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, true);
  return x + __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Sum over the 64 lanes, the same in every lane (fixed order).
__device__ __forceinline__ double wave_total(double x) {
  x = dpp_add<0x111, 0xf>(x);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds its sum
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);  // row_bcast 15 into rows 1 and 3
  x = dpp_add<0x143, 0xc>(x);  // row_bcast 31 into rows 2 and 3
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// w = tau p - h v and the next column's element after this column's rank-2 update, in one
// rounding sequence wherever an element is formed (v of the pivot row is 1).
__device__ __forceinline__ double td_w(double tau, double p, double h, double v) { return fma(-h, v, tau * p); }
__device__ __forceinline__ double td_col(double a, double v, double wm, double w) { return fma(-v, wm, a) - w; }

__device__ __forceinline__ void msg_store(unsigned long long* p, unsigned payload, unsigned tag) {
  __hip_atomic_store(p, ((unsigned long long)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// cache policy bits of a buffer load that must see other XCDs' device-scope stores (sc1);
// a 16-byte load takes two words, each of them valid by its own tag
constexpr int kDeviceScope = 16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void msg_clear_kernel(unsigned long long* __restrict__ msg, int words,
                                                        int* __restrict__ info) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) *info = 0;
  if (i < words) msg[i] = 0ull;  // tag 0: no column (columns count from 1)
}

// What a workgroup carries from column to column.  LDS rows and vectors are 64 NC wide (zero
// past n), so the code over a row's chunks has no bounds to check.
template <int NC>
struct TdState {
  double x[NC];           // column m, then its v: element lane + 64 q
  double vp[NC], wp[NC];  // the previous column's v and w
  double taup, hp;        // of the previous column: w_j = taup p_j - hp v_j
  double alpha, diag;     // elements m - 1 and m of column m
  double *rows, *pl, *al, *vl;
  double *A, *D, *E, *tau;
  unsigned long long* msg;
  __amdgpu_buffer_rsrc_t rmsg;
  unsigned max_polls;
  int* failed;
  int n, groups, me, nrow, lane, wave, tid;
};

// Columns m1 down to m0 + 1, whose active rows and columns lie in the first AC chunks.  False
// when the workgroup is through: it has no row left, or a wait has failed.
template <int NC, int AC>
__device__ __forceinline__ bool td_columns(TdState<NC>& t, int m1, int m0) {
  constexpr int LD = 64 * NC;
  constexpr int RT = (64 * AC + kTdThreads - 1) / kTdThreads;  // slots a thread waits for
  const int lane = t.lane, n = t.n;
  for (int m = m1; m > m0; --m) {
    const unsigned tag = (unsigned)(n - m);
    const int set = td_set(n, m);
    double* ps = t.pl + set * LD;
    double* as = t.al + set * LD;
    double* vs = t.vl + set * LD;
    const double* pprev = t.pl + (set ^ 1) * LD;
    const double* vprev = t.vl + (set ^ 1) * LD;
    // reflector of column m
    double xx = 0.0;
#pragma unroll
    for (int q = 0; q < AC; ++q) {
      const double c = lane + 64 * q < m - 1 ? t.x[q] : 0.0;
      xx = fma(c, c, xx);
    }
    xx = wave_total(xx);
    double beta = t.alpha, tau = 0.0, scale = 0.0;
    if (xx != 0.0) {
      beta = -copysign(sqrt(fma(t.alpha, t.alpha, xx)), t.alpha);
      tau = (beta - t.alpha) / beta;
      scale = 1.0 / (t.alpha - beta);
    }
#pragma unroll
    for (int q = 0; q < AC; ++q) {
      const int k = lane + 64 * q;
      t.x[q] = k < m - 1 ? t.x[q] * scale : (k == m - 1 ? 1.0 : 0.0);
      if (t.wave == 0) vs[k] = t.x[q];
    }
    // the workgroup's rows, two at a time: previous rank-2 update, then their products with v
    for (int r = t.wave; r < t.nrow; r += 2 * kTdWaves) {
      const int j0 = t.me + r * t.groups, j1 = j0 + kTdWaves * t.groups;
      if (j0 >= m) break;
      const bool two = j1 < m;
      double* row0 = t.rows + (size_t)r * LD;
      double* row1 = two ? row0 + (size_t)kTdWaves * LD : row0;
      const int jj = two ? j1 : j0;
      const double vj0 = vprev[j0], vj1 = vprev[jj];
      const double wj0 = td_w(t.taup, pprev[j0], t.hp, vj0), wj1 = td_w(t.taup, pprev[jj], t.hp, vj1);
      double a[AC], b[AC];
#pragma unroll
      for (int q = 0; q < AC; ++q) {
        a[q] = row0[lane + 64 * q];
        b[q] = row1[lane + 64 * q];
      }
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int q = 0; q < AC; ++q) {
        a[q] = fma(-wj0, t.vp[q], fma(-vj0, t.wp[q], a[q]));
        b[q] = fma(-wj1, t.vp[q], fma(-vj1, t.wp[q], b[q]));
        s0 = fma(a[q], t.x[q], s0);
        s1 = fma(b[q], t.x[q], s1);
        row0[lane + 64 * q] = a[q];
        row1[lane + 64 * q] = b[q];  // row0 again when there is no second row
      }
      const double p0 = wave_total(s0), p1 = wave_total(s1);
      const double n0 = row0[m - 1], n1 = row1[m - 1];
      if (t.groups == 1) {
        if (lane == 0) {
          ps[j0] = p0;
          as[j0] = n0;
          ps[jj] = p1;
          as[jj] = n1;
        }
      } else if (lane < (two ? 8 : 4)) {
        const double y = lane < 4 ? (lane < 2 ? p0 : n0) : (lane < 6 ? p1 : n1);
        const unsigned long long w = __builtin_bit_cast(unsigned long long, y);
        msg_store(t.msg + ((size_t)set * n + (lane < 4 ? j0 : j1)) * 4 + (lane & 3), (unsigned)(lane & 1 ? w : w >> 32),
                  tag);
      }
    }
    if (t.groups > 1) {
      if (!td_reads(t.me, m)) return false;
      // rows tid, tid + 512, ...: all of a thread's slots are asked for at once, and again
      // until every word carries this column's tag
      u32x4 w[RT][2];
      unsigned polls = 0;
      bool all;
      do {
        asm volatile("" ::: "memory");  // the loads are issued again on every turn
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const int j = t.tid + i * kTdThreads;
          const unsigned o = j < m ? (unsigned)((set * n + j) * 32) : 0x40000000u;  // past the end: zeros
#pragma unroll
          for (int y = 0; y < 2; ++y)
            w[i][y] = __builtin_bit_cast(u32x4,
                                         __builtin_amdgcn_raw_buffer_load_b128(t.rmsg, o + 16 * y, 0, kDeviceScope));
        }
        all = true;
#pragma unroll
        for (int i = 0; i < RT; ++i)
          if (t.tid + i * kTdThreads < m)
            all = all && w[i][0][1] == tag && w[i][0][3] == tag && w[i][1][1] == tag && w[i][1][3] == tag;
      } while (!all && ++polls < t.max_polls);
      if (!all) *t.failed = 1;
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const int j = t.tid + i * kTdThreads;
        if (j < m) {
          ps[j] = __builtin_bit_cast(double, ((unsigned long long)w[i][0][0] << 32) | w[i][0][2]);
          as[j] = __builtin_bit_cast(double, ((unsigned long long)w[i][1][0] << 32) | w[i][1][2]);
        }
      }
    }
    __syncthreads();
    if (*t.failed) return false;
    // w = tau p - (tau^2 v.p / 2) v, and column m - 1 after this column's update
    double p[AC], s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < AC; ++q) p[q] = ps[lane + 64 * q];
    const double pm = ps[m - 1], am = as[m - 1];
    const int i2 = m > 1 ? m - 2 : 0;
    const double p2 = ps[i2], a2 = as[i2], v2 = vs[i2];
#pragma unroll
    for (int q = 0; q < AC; ++q) {  // entries of p past m - 1 are an earlier column's: v is zero there
      if (q & 1)
        s1 = fma(t.x[q], p[q], s1);
      else
        s0 = fma(t.x[q], p[q], s0);
    }
    const double h = 0.5 * tau * tau * wave_total(s0 + s1);
    const double wm = td_w(tau, pm, h, 1.0);
    if (t.me == 0 && t.wave == 0) {  // every workgroup has read A: column m's results may go out
#pragma unroll
      for (int q = 0; q < AC; ++q)
        if (lane + 64 * q < m - 1) t.A[lane + 64 * q + (int64_t)m * n] = t.x[q];
      if (lane == 0) {
        t.D[m] = t.diag;
        t.E[m - 1] = beta;
        t.tau[m - 1] = tau;
      }
    }
#pragma unroll
    for (int q = 0; q < AC; ++q) {
      const int k = lane + 64 * q;
      const double w = td_w(tau, p[q], h, t.x[q]);
      t.vp[q] = t.x[q];
      t.wp[q] = k < m ? w : 0.0;
      t.x[q] = k < m ? td_col(as[k], t.x[q], wm, w) : 0.0;
    }
    t.diag = td_col(am, 1.0, wm, wm);
    if (m > 1) t.alpha = td_col(a2, v2, wm, td_w(tau, p2, h, v2));
    t.taup = tau;
    t.hp = h;
  }
  return true;
}

// The columns in stretches of shrinking row length: two chunks less each (three in long rows).
template <int NC, int AC>
__device__ __forceinline__ void td_all(TdState<NC>& t, int m1) {
  constexpr int NEXT = AC > 10 ? AC - 3 : (AC > 2 ? AC - 2 : 0);
  const int m0 = min(m1, 64 * NEXT);
  if (!td_columns<NC, AC>(t, m1, m0)) return;
  if constexpr (NEXT > 0) td_all<NC, NEXT>(t, m0);
}

// NC: 64-wide chunks of a row (n <= 64 NC).  LDS: the workgroup's rows, then p, the next
// column and v, two sets each.
template <int NC>
__global__ __launch_bounds__(kTdThreads, 2) void tridiag_kernel(double* __restrict__ A, int n, int groups,
                                                                double* __restrict__ D, double* __restrict__ E,
                                                                double* __restrict__ tau_out,
                                                                unsigned long long* __restrict__ msg,
                                                                int* __restrict__ info, unsigned max_polls) {
  extern __shared__ __align__(16) double td_lds[];
  __shared__ int failed;
  constexpr int LD = 64 * NC;
  TdState<NC> t;
  t.tid = threadIdx.x;
  t.lane = t.tid & 63;
  t.wave = t.tid >> 6;
  t.me = blockIdx.x;
  t.n = n;
  t.groups = groups;
  const int max_rows = (n + groups - 1) / groups;
  t.nrow = t.me < n ? (n - t.me + groups - 1) / groups : 0;
  t.rows = td_lds;
  t.pl = t.rows + (size_t)max_rows * LD;  // [2][LD]
  t.al = t.pl + 2 * LD;                   // [2][LD]
  t.vl = t.al + 2 * LD;                   // [2][LD]
  t.A = A;
  t.D = D;
  t.E = E;
  t.tau = tau_out;
  t.msg = msg;
  t.rmsg = __builtin_amdgcn_make_buffer_rsrc(msg, (short)0, groups > 1 ? 2 * n * 32 : 0, 0x00020000);
  t.max_polls = max_polls;
  t.failed = &failed;
  if (t.tid == 0) failed = 0;
  for (int i = t.tid; i < 6 * LD; i += kTdThreads) t.pl[i] = 0.0;
  for (int r = t.wave; r < t.nrow; r += kTdWaves) {
    const int j = t.me + r * groups;
    for (int k = t.lane; k < LD; k += 64)
      t.rows[(size_t)r * LD + k] = k >= n ? 0.0 : (k >= j ? A[j + (int64_t)k * n] : A[k + (int64_t)j * n]);
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int k = t.lane + 64 * q;
    t.x[q] = k < n ? A[k + (int64_t)(n - 1) * n] : 0.0;
    t.vp[q] = t.wp[q] = 0.0;
  }
  t.taup = t.hp = 0.0;
  t.alpha = A[n - 2 + (int64_t)(n - 1) * n];
  t.diag = A[n - 1 + (int64_t)(n - 1) * n];
  __syncthreads();
  td_all<NC, NC>(t, n - 1);
  if (t.me == 0 && t.tid == 0) D[0] = t.diag;
  if (t.tid == 0 && failed) *info = n + 1;
}

// The same results from one workgroup, with A in memory: for a launch above that could not
// finish (*info != 0) or was not possible (always).  What that launch wrote to A are reflectors
// above the first superdiagonal, so the lower triangle is still whole; its values are those of
// the upper one up to the rounding of the products that made them.  Row j of the symmetric
// matrix is column j of A.  Two passes over the active block a column: n = 130 0.7 ms, 600 29 ms,
// 1408 530 ms (the exchange: 0.35, 2.2, 8).
constexpr int kTaThreads = 1024;
constexpr int kTaWaves = kTaThreads / 64;

__global__ __launch_bounds__(kTaThreads) void tridiag_alone_kernel(double* A, int n, double* __restrict__ D,
                                                                   double* __restrict__ E, double* __restrict__ tau_out,
                                                                   int* info, int always) {
  __shared__ double v[64 * kTdMaxChunks], w[64 * kTdMaxChunks], part[kTaWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!always && *info == 0) return;
  auto block_total = [&](double x) {
    x = wave_total(x);
    __syncthreads();  // part may still be read from the sum before
    if (lane == 0) part[wave] = x;
    __syncthreads();
    double s = part[0];
    for (int i = 1; i < kTaWaves; ++i) s += part[i];
    return s;
  };
  for (int j = wave; j < n; j += kTaWaves)
    for (int k = lane; k < j; k += 64) A[k + (int64_t)j * n] = A[j + (int64_t)k * n];
  __syncthreads();
  for (int m = n - 1; m > 0; --m) {
    double* col = A + (int64_t)m * n;
    double xx = 0.0;
    for (int k = tid; k < m - 1; k += kTaThreads) xx = fma(col[k], col[k], xx);
    xx = block_total(xx);
    const double alpha = col[m - 1];
    double beta = alpha, tau = 0.0, scale = 0.0;
    if (xx != 0.0) {
      beta = -copysign(sqrt(fma(alpha, alpha, xx)), alpha);
      tau = (beta - alpha) / beta;
      scale = 1.0 / (alpha - beta);
    }
    for (int k = tid; k < m; k += kTaThreads) v[k] = k < m - 1 ? col[k] * scale : 1.0;
    __syncthreads();
    for (int j = wave; j < m; j += kTaWaves) {
      double p = 0.0;
      for (int k = lane; k < m; k += 64) p = fma(A[k + (int64_t)j * n], v[k], p);
      p = wave_total(p);
      if (lane == 0) w[j] = p;
    }
    __syncthreads();
    double vp = 0.0;
    for (int k = tid; k < m; k += kTaThreads) vp = fma(v[k], w[k], vp);
    const double h = 0.5 * tau * tau * block_total(vp);
    for (int k = tid; k < m; k += kTaThreads) {
      w[k] = td_w(tau, w[k], h, v[k]);
      if (k < m - 1) col[k] = v[k];
    }
    if (tid == 0) {
      D[m] = col[m];
      E[m - 1] = beta;
      tau_out[m - 1] = tau;
    }
    __syncthreads();
    for (int j = wave; j < m; j += kTaWaves)
      for (int k = lane; k < m; k += 64) {
        double* a = A + k + (int64_t)j * n;
        *a = fma(-w[j], v[k], fma(-v[j], w[k], *a));
      }
    __syncthreads();
  }
  if (tid == 0) {
    D[0] = A[0];
    *info = 0;
  }
}

// C <- Q C for the reflectors that tridiag_kernel left in A: column m holds v[0 .. m - 2],
// v[m - 1] = 1, factor tau[m - 1]; applied from m = 2 up (column 1 has factor zero).  A wave
// keeps two columns of C in registers; the block stages kBtRefl reflectors at a time in LDS
// (zero outside 0 .. m - 1), the next ones already in registers while these are applied.
template <int NC>
__global__ __launch_bounds__(kBtThreads) void backtransform_kernel(const double* __restrict__ A,
                                                                   const double* __restrict__ tau, int n,
                                                                   double* __restrict__ C) {
  constexpr int LD = 64 * NC;
  __shared__ double vs[2][kBtRefl][LD];
  __shared__ double ts[2][kBtRefl];
  constexpr int PT = kBtRefl * LD / kBtThreads;  // staged values per thread
  const int tid = threadIdx.x, lane = tid & 63;
  const int col = 2 * (blockIdx.x * kBtWaves + (tid >> 6));
  double c0[NC], c1[NC], st[PT], tst = 0.0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int k = lane + 64 * q;
    c0[q] = k < n && col < n ? C[k + (int64_t)col * n] : 0.0;
    c1[q] = k < n && col + 1 < n ? C[k + (int64_t)(col + 1) * n] : 0.0;
  }
  auto load = [&](int m0) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int e = tid + i * kBtThreads, m = m0 + e / LD, k = e % LD;
      st[i] = m < n && k < m - 1 ? A[k + (int64_t)m * n] : (m < n && k == m - 1 ? 1.0 : 0.0);
    }
    tst = tid < kBtRefl && m0 + tid < n ? tau[m0 + tid - 1] : 0.0;
  };
  auto stage = [&](int b) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int e = tid + i * kBtThreads;
      vs[b][e / LD][e % LD] = st[i];
    }
    if (tid < kBtRefl) ts[b][tid] = tst;
  };
  load(2);
  stage(0);
  __syncthreads();
  for (int m0 = 2, b = 0; m0 < n; m0 += kBtRefl, b ^= 1) {
    load(m0 + kBtRefl);
    for (int r = 0; r < kBtRefl; ++r) {
      double v[NC], s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int q = 0; q < NC; ++q) v[q] = vs[b][r][lane + 64 * q];
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        s0 = fma(v[q], c0[q], s0);
        s1 = fma(v[q], c1[q], s1);
      }
      const double tr = ts[b][r], f0 = tr * wave_total(s0), f1 = tr * wave_total(s1);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        c0[q] = fma(-f0, v[q], c0[q]);
        c1[q] = fma(-f1, v[q], c1[q]);
      }
    }
    stage(b ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int k = lane + 64 * q;
    if (k < n && col < n) C[k + (int64_t)col * n] = c0[q];
    if (k < n && col + 1 < n) C[k + (int64_t)(col + 1) * n] = c1[q];
  }
}

// 64-wide chunks of the rows: the kernels' instances
int chunks_of(int n) {
  for (int c : {2, 4, 6, 8, 10, 13, 16, 19, kTdMaxChunks})
    if (n <= 64 * c) return c;
  return 0;
}

size_t tridiag_lds(int n, int groups) {
  return ((size_t)((n + groups - 1) / groups) + 6) * 64 * chunks_of(n) * sizeof(double);
}

template <int NC>
hipError_t launch_td(double* A, int n, int groups, double* D, double* E, double* tau, void* msg, int* info,
                     hipStream_t s, unsigned max_polls) {
  unsigned long long* m = static_cast<unsigned long long*>(msg);
  const size_t lds = tridiag_lds(n, groups);
  if (groups == 1) {
    hipLaunchKernelGGL(tridiag_kernel<NC>, dim3(1), dim3(kTdThreads), lds, s, A, n, groups, D, E, tau, m, info,
                       max_polls);
    return hipGetLastError();
  }
  const int words = 2 * n * 4;
  hipLaunchKernelGGL(msg_clear_kernel, dim3((words + 255) / 256), dim3(256), 0, s, m, words, info);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the workgroups wait for each other: a cooperative launch, so all of them are resident
  void* args[] = {&A, &n, &groups, &D, &E, &tau, &m, &info, &max_polls};
  e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(&tridiag_kernel<NC>), dim3(groups), dim3(kTdThreads),
                                 args, (unsigned)lds, s);
  const int refused = e == hipErrorCooperativeLaunchTooLarge;  // fewer compute units than the device reports
  if (refused) (void)hipGetLastError();
  if (e != hipSuccess && !refused) return e;
  hipLaunchKernelGGL(tridiag_alone_kernel, dim3(1), dim3(kTaThreads), 0, s, A, n, D, E, tau, info, refused);
  return hipGetLastError();
}

template <int NC>
hipError_t launch_bt(const double* A, const double* tau, int n, double* C, hipStream_t s) {
  hipLaunchKernelGGL(backtransform_kernel<NC>, dim3((n + 2 * kBtWaves - 1) / (2 * kBtWaves)), dim3(kBtThreads), 0,
                     s, A, tau, n, C);
  return hipGetLastError();
}

}  // namespace

// Workgroups: one while the rows fit its LDS beside the six vectors (n <= 128: no exchange, an
// ordinary launch); beyond, enough to hold the rows, and no more than 16 rows each, so a
// workgroup's eight waves pass over their rows once, two at a time (n = 600: 24 workgroups
// 7.30 ms for the whole subspace problem, 38 7.24, 64 7.18, 128 7.27; n = 300: 6 / 19 / 64
// 3.77 / 3.68 / 3.58).
int tridiag_groups(int n) {
  if (n < 2 || chunks_of(n) == 0) return 0;
  if (n <= 128) return 1;
  for (int g = (n + 15) / 16; g <= kTdMaxGroups; ++g)
    if (tridiag_lds(n, g) + 64 <= kTdMaxLds) return g;
  return 0;
}

size_t tridiag_msg_bytes(int n) { return (size_t)2 * n * 4 * sizeof(unsigned long long); }

hipError_t launch_tridiag(double* A, int n, double* D, double* E, double* tau, void* msg, int* info, hipStream_t s,
                          unsigned max_polls) {
  const int g = tridiag_groups(n);
  if (g == 0) return hipErrorInvalidValue;
  switch (chunks_of(n)) {
    case 2: return launch_td<2>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 4: return launch_td<4>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 6: return launch_td<6>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 8: return launch_td<8>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 10: return launch_td<10>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 13: return launch_td<13>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 16: return launch_td<16>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case 19: return launch_td<19>(A, n, g, D, E, tau, msg, info, s, max_polls);
    case kTdMaxChunks: return launch_td<kTdMaxChunks>(A, n, g, D, E, tau, msg, info, s, max_polls);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_backtransform(const double* A, const double* tau, int n, double* C, hipStream_t s) {
  switch (chunks_of(n)) {
    case 2: return launch_bt<2>(A, tau, n, C, s);
    case 4: return launch_bt<4>(A, tau, n, C, s);
    case 6: return launch_bt<6>(A, tau, n, C, s);
    case 8: return launch_bt<8>(A, tau, n, C, s);
    case 10: return launch_bt<10>(A, tau, n, C, s);
    case 13: return launch_bt<13>(A, tau, n, C, s);
    case 16: return launch_bt<16>(A, tau, n, C, s);
    case 19: return launch_bt<19>(A, tau, n, C, s);
    case kTdMaxChunks: return launch_bt<kTdMaxChunks>(A, tau, n, C, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace chefsi
