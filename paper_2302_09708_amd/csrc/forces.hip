// Nonlocal Hellmann-Feynman forces and the kinetic and nonlocal stresses (Sec. 2: the
// filter's stencil and projector routines reused for the force: the gradient operator on
// the orbitals, then the nonlocal projectors on the result).
//
// nl_grad_kernel: with a = dV chi^T psi and b_d = dV chi^T (d psi / dx_d), per atom J and
//   orbital n the sums  sum_k gamma_k a_k b_d,k  of the forces, or  sum_k gamma_k a_k^2  and
//   sum_k gamma_k a_k dV (chi_k d_b)^T (d psi / dx_a)  of the nonlocal stress, times the
//   occupation.  The gradient is formed only where a projector reads it, from the 6r
//   neighbours of each support point, and never leaves registers.  atom_sums_kernel adds
//   the orbitals of an atom in a fixed order.
// kinetic_stress_kernel: the six products of the gradient's components summed over the
//   grid in one z march over each orbital (the layout of the filter's stencil pass).
// Every sum has a fixed order (bitwise reproducible); FP64 arithmetic.
#include <algorithm>

#include "reduce.h"
#include "stencil.h"

namespace chefsi {

namespace {

constexpr int kNgWaves = 8;  // waves per block, sharing an atom's support
constexpr int kNgP = 4;      // projectors per pass

// One block = one atom x V orbitals; a thread owns every 512th support point.  A point's 6r + 1
// byte offsets are computed once and serve the V orbitals (Dirichlet ghosts are offsets
// past the end, which load zero).  For supports too large for the kernel below.  Bound by the
// 6r + 1 cached loads per (support point, orbital), about 58 cycles of a CU each (eight to twelve
// lines, mostly from L2), and with few atoms and orbitals by the chain of a thread's points: 8
// waves share it.  40x37x33, 4 atoms of 8200 points, order 12, forces of 1 / 10 / 40 orbitals
// FP64 (us): whole gradients written and re-read 315 / 476 / 590, one wave for two orbitals of an
// atom 768 / 948 / 1313, now 108 / 109 / 111.
// The stress keeps 40 sums per orbital, so its blocks own one orbital, the forces' two.
// XCD mapping: each XCD takes a contiguous run of (orbital group, atom), atom fastest, so
// neighbouring atoms read an orbital's shared points through one L2.
template <typename TV, int R, bool STRESS>
__global__ __launch_bounds__(64 * kNgWaves) void nl_grad_kernel(NlGradArgs<TV> a) {
  constexpr int V = STRESS ? 1 : 2;
  constexpr int NB = STRESS ? 9 : 3;         // gathers of the gradient per projector
  constexpr int NS = NB * kNgP;              // their sums; the kNgP sums of psi beside them
  constexpr int NR = STRESS ? 32 : 16;       // power of two of the first reduction
  constexpr int NO = STRESS ? 10 : 3;        // results per (atom, orbital)
  constexpr int NA = kNgP + NS;              // 16 or 40 sums per orbital
  __shared__ double red[kNgWaves][V][NA];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t logical = (int64_t)(blockIdx.x % 8) * a.per_xcd + blockIdx.x / 8;
  if (logical >= (int64_t)a.n_atoms * a.ngroups) return;
  const int atom = (int)(logical % a.n_atoms);
  const int v0 = (int)(logical / a.n_atoms) * V;
  const int s0 = a.supp_off[atom];
  const int n = a.supp_off[atom + 1] - s0;
  const int npj = a.nproj[atom];
  const double* chi = a.chi + a.chi_off[atom];
  const int nx = a.nx, ny = a.ny, nz = a.nz, nplane = nx * ny;
  const int nbytes = (int)(a.nd * (int64_t)sizeof(TV));
  __amdgpu_buffer_rsrc_t rx[V];
#pragma unroll
  for (int u = 0; u < V; ++u) rx[u] = make_rsrc(a.x + (int64_t)min(v0 + u, a.ns - 1) * a.nd, nbytes);
  double tot = 0.0;  // thread u NO + d: result d of orbital u
  const int ou = tid / NO, od = tid % NO;

  for (int a0 = 0; a0 < npj; a0 += kNgP) {
    double acc[V][NA];
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int k = 0; k < NA; ++k) acc[u][k] = 0.0;
    for (int s = tid; s < n; s += 64 * kNgWaves) {
      const int i = a.supp_idx[s0 + s];
      const int z = i / nplane, yx = i - z * nplane, y = yx / nx, x = yx - y * nx;
      unsigned off[3][2][R];
#pragma unroll
      for (int p = 1; p <= R; ++p) {
        const int cp[3] = {x + p, y + p, z + p}, cm[3] = {x - p, y - p, z - p};
        const int ext[3] = {nx, ny, nz}, str[3] = {1, nx, nplane};
#pragma unroll
        for (int d = 0; d < 3; ++d) {  // n >= r in a periodic direction: one wrap
          const int jp = i + p * str[d], jm = i - p * str[d];
          const bool op = cp[d] >= ext[d], om = cm[d] < 0;
          off[d][0][p - 1] = lane_off<TV>(!op ? jp : (a.periodic[d] ? jp - ext[d] * str[d] : -1));
          off[d][1][p - 1] = lane_off<TV>(!om ? jm : (a.periodic[d] ? jm + ext[d] * str[d] : -1));
        }
      }
      double c[kNgP];
#pragma unroll
      for (int k = 0; k < kNgP; ++k) c[k] = a0 + k < npj ? chi[(int64_t)(a0 + k) * n + s] : 0.0;
      double w[3] = {1.0, 1.0, 1.0};
      if (STRESS) {
#pragma unroll
        for (int b = 0; b < 3; ++b) w[b] = a.disp[3 * (int64_t)(s0 + s) + b];
      }
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const double yv = double(bload<TV>(rx[u], lane_off<TV>(i), 0u));
#pragma unroll
        for (int k = 0; k < kNgP; ++k) acc[u][k] += c[k] * yv;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          double g = 0.0;
#pragma unroll
          for (int p = 0; p < R; ++p)
            g += a.c[d][p + 1] * (double(bload<TV>(rx[u], off[d][0][p], 0u)) - double(bload<TV>(rx[u], off[d][1][p], 0u)));
          if (STRESS) {
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
              for (int k = 0; k < kNgP; ++k) acc[u][kNgP + (3 * d + b) * kNgP + k] += (c[k] * w[b]) * g;
          } else {
#pragma unroll
            for (int k = 0; k < kNgP; ++k) acc[u][kNgP + d * kNgP + k] += c[k] * g;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      double h[NR];
#pragma unroll
      for (int k = 0; k < NR; ++k) h[k] = acc[u][k];
      wave_sums(h, lane);
      if (lane % (64 / NR) == 0) red[wave][u][lane / (64 / NR)] = h[0];
      if constexpr (STRESS) {  // the other eight of the forty
        double g[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = acc[u][NR + k];
        wave_sums(g, lane);
        if (lane % 8 == 0) red[wave][u][NR + lane / 8] = g[0];
      }
    }
    __syncthreads();
    if (tid < V * NO) {
      auto sum = [&](int k) {
        double r = red[0][ou][k];
#pragma unroll
        for (int w = 1; w < kNgWaves; ++w) r += red[w][ou][k];
        return r;
      };
      // the energy sum gamma a^2 (stress, result 0), else sum gamma a b
      const int b = STRESS ? od : od + 1;  // block of kNgP sums in red
      for (int k = 0; k < kNgP && a0 + k < npj; ++k)
        tot += a.gdv[a.poff[atom] + a0 + k] * (sum(k) * sum(b * kNgP + k));
    }
    __syncthreads();
  }
  if (tid < V * NO && v0 + ou < a.ns)  // gdv holds gamma dV: two factors dV, one taken from gdv
    a.part[((int64_t)atom * a.ns + v0 + ou) * NO + od] = a.occ[v0 + ou] * tot * a.dv;
}

// The same results with the gradient's neighbourhood in LDS.  One block = one atom x kBoxOrb
// orbitals, one orbital after the other.  The atom's support lies in a box of grid points
// (wrapped in periodic directions); for each direction the block stages the box, longer by r
// at both ends of that direction, and every thread forms the derivative at its (at most
// kBoxPts) support points from LDS.  The staged values' source offsets, the points' places
// in the box and their projector values stay in registers for all orbitals; the next
// direction's values are in flight while one is summed.  Where the support or the box is
// larger than the registers hold, nl_grad_kernel above does the work.
// The wave sums of all the block's orbitals wait in LDS and are combined at its end: combined
// orbital by orbital they were a third of the time (2.36 and 2.95 ms).
// 72^3, 128 atoms (905 points, a box of 12^3), 600 orbitals, order 12, FP64: forces 3.8 ->
// 1.95 ms, stress 3.9 -> 2.5 ms; bound by latency at one block per CU (LDS busy 31 % of the
// cycles, VALU 30 %): the registers leave no room for a second.
constexpr int kBoxThreads = 512;
constexpr int kBoxWaves = kBoxThreads / 64;
constexpr int kBoxPts = kGradBoxPoints / kBoxThreads;    // support points per thread
constexpr int kBoxStage = kGradBoxValues / kBoxThreads;  // staged values per thread and direction
constexpr int kBoxOrb = 16;

template <typename TV, int R, bool STRESS>
__global__ __launch_bounds__(kBoxThreads, 2) void nl_grad_box_kernel(NlGradArgs<TV> a) {
  constexpr int NO = STRESS ? 10 : 3;
  constexpr int NR = STRESS ? 3 : 1;  // reductions of 16 sums per orbital
  __shared__ TV box[2][kGradBoxValues];
  __shared__ double red[kBoxOrb][kBoxWaves][16 * NR];  // every orbital's sums, combined at the end
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t logical = (int64_t)(blockIdx.x % 8) * a.per_xcd + blockIdx.x / 8;
  if (logical >= (int64_t)a.n_atoms * a.ngroups) return;
  const int atom = (int)(logical % a.n_atoms);
  const int v0 = (int)(logical / a.n_atoms) * a.gpo, v1 = min(v0 + a.gpo, a.ns);
  const int s0 = a.supp_off[atom], n = a.supp_off[atom + 1] - s0;
  const int npj = a.nproj[atom];
  const double* chi = a.chi + a.chi_off[atom];
  const int ext[3] = {a.nx, a.ny, a.nz}, str[3] = {1, a.nx, a.nx * a.ny};
  int lo[3], len[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = a.box[6 * atom + d];
    len[d] = a.box[6 * atom + 3 + d];
  }
  // source offset of every staged value (past the end: a zero)
  unsigned off[3][kBoxStage];
  int count[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int e0 = len[0] + (d == 0 ? 2 * R : 0), e1 = len[1] + (d == 1 ? 2 * R : 0), e2 = len[2] + (d == 2 ? 2 * R : 0);
    count[d] = e0 * e1 * e2;
#pragma unroll
    for (int i = 0; i < kBoxStage; ++i) {
      const int e = tid + i * kBoxThreads;
      int src = -1;
      if (e < count[d]) {
        const int q = e / e0;
        int c[3] = {lo[0] + e - q * e0, lo[1] + q % e1, lo[2] + q / e1};
        c[d] -= R;
        src = 0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          if (a.periodic[b]) {  // the box is no longer than the period, r no longer than it
            c[b] = c[b] < 0 ? c[b] + ext[b] : c[b];
            c[b] = c[b] >= ext[b] ? c[b] - ext[b] : c[b];
            c[b] = c[b] >= ext[b] ? c[b] - ext[b] : c[b];
          }
          src = c[b] < 0 || c[b] >= ext[b] || src < 0 ? -1 : src + c[b] * str[b];
        }
      }
      off[d][i] = lane_off<TV>(src);
    }
  }
  // the thread's support points: place in the box, displacement
  int place[kBoxPts][3];
  double w[kBoxPts][3];
#pragma unroll
  for (int t = 0; t < kBoxPts; ++t) {
    const int s = tid + t * kBoxThreads;
    // past the end the last point again, with zero weights: no value is read that the sums do
    // not contain (0 times a non-finite one would be NaN)
    const int i = n > 0 ? a.supp_idx[s0 + min(s, n - 1)] : 0;
    const int z = i / str[2], yx = i - z * str[2], y = yx / a.nx;
    int c[3] = {yx - y * a.nx, y, z};
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      c[b] -= lo[b];
      c[b] = c[b] < 0 ? c[b] + ext[b] : c[b];
      place[t][b] = n > 0 ? c[b] : 0;
      w[t][b] = STRESS && s < n ? a.disp[3 * (int64_t)(s0 + s) + b] : 0.0;
    }
  }
  const int nbytes = (int)(a.nd * (int64_t)sizeof(TV));
  TV st[kBoxStage];
  auto fetch = [&](int v, int d) {
    const __amdgpu_buffer_rsrc_t r = make_rsrc(a.x + (int64_t)v * a.nd, v < v1 ? nbytes : 0);
#pragma unroll
    for (int i = 0; i < kBoxStage; ++i)
      st[i] = bload<TV>(r, d == 0 ? off[0][i] : (d == 1 ? off[1][i] : off[2][i]), 0u);
  };

  for (int a0 = 0; a0 < npj; a0 += kNgP) {
    double c[kBoxPts][kNgP];
#pragma unroll
    for (int t = 0; t < kBoxPts; ++t)
#pragma unroll
      for (int k = 0; k < kNgP; ++k) {
        const int s = tid + t * kBoxThreads;
        c[t][k] = s < n && a0 + k < npj ? chi[(int64_t)(a0 + k) * n + s] : 0.0;
      }
    auto stage = [&](int d, int buf) {
      const int cnt = d == 0 ? count[0] : (d == 1 ? count[1] : count[2]);
#pragma unroll
      for (int i = 0; i < kBoxStage; ++i)
        if (wave * 64 + i * kBoxThreads < cnt) box[buf][tid + i * kBoxThreads] = st[i];
    };
    fetch(v0, 0);
    stage(0, 0);
    fetch(v0, 1);
    int buf = 0;
    for (int v = v0; v < v1; ++v) {
      double acc[16];  // forces: four sums of psi, then of each derivative; stress: those of one direction
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[k] = 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d, buf ^= 1) {
        __syncthreads();  // this direction's box is staged, the other buffer is no longer read
        stage(d < 2 ? d + 1 : 0, buf ^ 1);
        fetch(d < 1 ? v : v + 1, d < 1 ? 2 : d - 1);
        const int e0 = len[0] + (d == 0 ? 2 * R : 0), e1 = len[1] + (d == 1 ? 2 * R : 0);
        const int step = d == 0 ? 1 : (d == 1 ? e0 : e0 * e1);
#pragma unroll
        for (int t = 0; t < kBoxPts; ++t) {
          if (wave * 64 + t * kBoxThreads >= n) continue;
          const TV* p0 = box[buf] + place[t][0] + e0 * (place[t][1] + e1 * place[t][2]) + R * step;
          double g = 0.0;
#pragma unroll
          for (int p = 1; p <= R; ++p) g += a.c[d][p] * (double(p0[p * step]) - double(p0[-p * step]));
          if (d == 0) {
            const double yv = double(p0[0]);
#pragma unroll
            for (int k = 0; k < kNgP; ++k) acc[k] += c[t][k] * yv;
          }
          if (STRESS) {
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
              for (int k = 0; k < kNgP; ++k) acc[kNgP + b * kNgP + k] += (c[t][k] * w[t][b]) * g;
          } else {
#pragma unroll
            for (int k = 0; k < kNgP; ++k) acc[kNgP + d * kNgP + k] += c[t][k] * g;
          }
        }
        if (STRESS || d == 2) {
          wave_sums(acc, lane);
          if (lane % 4 == 0) red[v - v0][wave][(STRESS ? 16 * d : 0) + lane / 4] = acc[0];
#pragma unroll
          for (int k = 0; k < 16; ++k) acc[k] = 0.0;
        }
      }
    }
    __syncthreads();
    for (int e = tid; e < (v1 - v0) * NO; e += kBoxThreads) {
      const int v = e / NO, i = e % NO;
      auto sum = [&](int k) {
        double r = red[v][0][k];
        for (int j = 1; j < kBoxWaves; ++j) r += red[v][j][k];
        return r;
      };
      // result i: the energy (stress, 0), else direction pair 3 d + b = i - 1; forces: direction i
      const int at = !STRESS ? kNgP * (i + 1) : (i == 0 ? 0 : 16 * ((i - 1) / 3) + kNgP * (1 + (i - 1) % 3));
      double tot = 0.0;
      for (int k = 0; k < kNgP && a0 + k < npj; ++k) tot += a.gdv[a.poff[atom] + a0 + k] * (sum(k) * sum(at + k));
      double* out = a.part + ((int64_t)atom * a.ns + v0 + v) * NO + i;
      tot *= a.occ[v0 + v] * a.dv;
      *out = a0 == 0 ? tot : *out + tot;
    }
    __syncthreads();  // the sums are read before another pass of projectors writes its own
  }
}

// out[J * no + d] = scale * sum over orbitals of part[(J * ns + v) * no + d], one block per
// atom: thread t adds orbitals t, t + 256, ..., then a tree over the threads.
__global__ __launch_bounds__(256) void atom_sums_kernel(const double* __restrict__ part, int ns, int no, double scale,
                                                        double* __restrict__ out) {
  __shared__ double red[256];
  const int J = blockIdx.x;
  for (int d = 0; d < no; ++d) {
    double s = 0.0;
    for (int v = threadIdx.x; v < ns; v += 256) s += part[((int64_t)J * ns + v) * no + d];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[(int64_t)J * no + d] = scale * red[0];
    __syncthreads();
  }
}

// Kinetic stress: sum_v occ[v] sum_i g_a g_b (ab = xx, yy, zz, xy, xz, yz).  A unit is one
// orbital x a tile of whole x rows x a z chunk, marched as in the filter's stencil pass (z
// neighbours in a register queue, the plane and its halo in double-buffered LDS, one
// barrier per plane, the next plane's values one iteration ahead); block b takes units b,
// b + grid, ... and writes its six sums.  Reads the block once: bound by LDS reads and
// memory latency like the stencil pass.  72^3, 600 orbitals FP64 measured 1.16 ms; one
// thread per point with every neighbour through the caches took 9.7 ms.
template <typename TV, int R, int PY, int KH>
__global__ __launch_bounds__(hx_max_threads(PY)) void kinetic_stress_kernel(StressArgs<TV> a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  constexpr int Q = 2 * R + 1;
  const int nx = a.nx, ny = a.ny, nz = a.nz, nplane = nx * ny;
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
  const int pitch = a.pitch;
  const int tile_elems = (a.ty + 2 * R) * pitch;
  const int tile_buf = tile_elems + kHxDummy;
  TV* s_tile = reinterpret_cast<TV*>(lds_raw);
  const bool active = tid < nx * a.nyg;
  const int x = active ? tid % nx : 0;
  const int ly0 = active ? (tid / nx) * PY : 0;
  const int nbytes = (int)(a.nd * (int64_t)sizeof(TV));
  const unsigned plane_bytes = (unsigned)nplane * (unsigned)sizeof(TV);
  if (!a.periodic[0]) {  // Dirichlet x: the halo columns of both tile buffers hold zeros
    const int nrows = 2 * (a.ty + 2 * R);
    for (int i = tid; i < nrows * 2 * R; i += nthr) {
      const int row = i / (2 * R), c = i % (2 * R);
      const int buf = row / (a.ty + 2 * R), rr = row % (a.ty + 2 * R);
      s_tile[buf * tile_buf + rr * pitch + (c < R ? c : nx + c)] = TV(0);
    }
  }
  double tot[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const int per_vec = a.nty * a.nzc;
  for (int64_t unit = blockIdx.x; unit < a.nunits; unit += gridDim.x) {
    const int vec = (int)(unit / per_vec), rem = (int)(unit % per_vec);
    const int y0 = (rem % a.nty) * a.ty, z0 = (rem / a.nty) * a.zc;
    const int nzl = min(a.zc, nz - z0);
    const TV* xv = a.x + (int64_t)vec * a.nd;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(xv, nbytes);
    const __amdgpu_buffer_rsrc_t rz = make_rsrc(xv, 0);
    unsigned vq[PY];
    int sown[PY];
    bool valid[PY];
#pragma unroll
    for (int j = 0; j < PY; ++j) {
      const int gy = y0 + ly0 + j;
      vq[j] = lane_off<TV>(active ? row_offset(x, gy, nx, ny, a.periodic[1]) : -1);
      valid[j] = active && gy < ny;
      sown[j] = active ? (R + ly0 + j) * pitch + R + x : tile_elems + lane;
    }
    int sdst[KH];
    unsigned vh[KH];
    const int nslots = hx_halo_slots(nx, a.ty, R, a.periodic[0]);
#pragma unroll
    for (int k = 0; k < KH; ++k) {
      const int e = tid + k * nthr;
      int dst = tile_elems + lane, src = -1;
      if (e < nslots) halo_slot(e, nx, ny, a.ty, y0, R, pitch, a.periodic[0], a.periodic[1], dst, src);
      sdst[k] = dst;
      vh[k] = lane_off<TV>(src);
    }
    TV q[Q][PY], pf[PY], hp[KH];
#pragma unroll
    for (int j = 0; j < PY; ++j) q[0][j] = TV(0);
#pragma unroll
    for (int s = 1; s < Q; ++s) {
      const int po = plane_offset(z0 - R - 1 + s, nplane, nz, a.periodic[2]);
#pragma unroll
      for (int j = 0; j < PY; ++j) q[s][j] = pload<TV>(xv, nbytes, vq[j], po);
    }
    {
      const int po = plane_offset(z0 + R, nplane, nz, a.periodic[2]);
#pragma unroll
      for (int j = 0; j < PY; ++j) pf[j] = pload<TV>(xv, nbytes, vq[j], po);
      const int ph = plane_offset(z0, nplane, nz, a.periodic[2]);
#pragma unroll
      for (int k = 0; k < KH; ++k) hp[k] = pload<TV>(xv, nbytes, vh[k], ph);
    }
    int pb = z0 + R + 1, ph = z0 + 1;
    if (a.periodic[2]) {
      pb %= nz;
      ph %= nz;
    }
    double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // the previous unit's last plane may still be read by slower waves
    __syncthreads();
    for (int zl = 0; zl < nzl; ++zl) {
      TV* tl = s_tile + (zl & 1) * tile_buf;
      const bool more = zl + 1 < nzl;
#pragma unroll
      for (int s = 0; s < Q - 1; ++s)
#pragma unroll
        for (int j = 0; j < PY; ++j) q[s][j] = q[s + 1][j];
#pragma unroll
      for (int j = 0; j < PY; ++j) q[Q - 1][j] = pf[j];
      {
        const bool ok = more && pb < nz;
        const __amdgpu_buffer_rsrc_t r = ok ? rx : rz;
        const unsigned so = ok ? (unsigned)pb * plane_bytes : 0u;
#pragma unroll
        for (int j = 0; j < PY; ++j) pf[j] = bload<TV>(r, vq[j], so);
      }
#pragma unroll
      for (int j = 0; j < PY; ++j) tl[sown[j]] = q[R][j];
#pragma unroll
      for (int k = 0; k < KH; ++k) tl[sdst[k]] = hp[k];
      {
        const bool ok = more && ph < nz;
        const __amdgpu_buffer_rsrc_t r = ok ? rx : rz;
        const unsigned so = ok ? (unsigned)ph * plane_bytes : 0u;
#pragma unroll
        for (int k = 0; k < KH; ++k) hp[k] = bload<TV>(r, vh[k], so);
      }
      ++pb;
      ++ph;
      if (a.periodic[2]) {
        pb = pb == nz ? 0 : pb;
        ph = ph == nz ? 0 : ph;
      }
      __syncthreads();
      double gx[PY], gy[PY], gz[PY];
#pragma unroll
      for (int j = 0; j < PY; ++j) {
        gx[j] = gy[j] = gz[j] = 0.0;
#pragma unroll
        for (int p = 1; p <= R; ++p) gz[j] += a.c[2][p] * (double(q[R + p][j]) - double(q[R - p][j]));
      }
#pragma unroll
      for (int t = 0; t < PY + 2 * R; ++t) {  // each LDS row of the column feeds every row it neighbours
        const double v = double(tl[(ly0 + t) * pitch + R + x]);
#pragma unroll
        for (int j = 0; j < PY; ++j) {
          const int p = t - R - j;
          if (p > 0 && p <= R) gy[j] += a.c[1][p] * v;
          if (p < 0 && p >= -R) gy[j] -= a.c[1][-p] * v;
        }
      }
#pragma unroll
      for (int j = 0; j < PY; ++j) {
        const TV* row = tl + (R + ly0 + j) * pitch + R + x;
#pragma unroll
        for (int p = 1; p <= R; ++p) gx[j] += a.c[0][p] * (double(row[p]) - double(row[-p]));
        if (!valid[j]) gx[j] = gy[j] = gz[j] = 0.0;  // idle lanes and rows past ny
        sum[0] += gx[j] * gx[j];
        sum[1] += gy[j] * gy[j];
        sum[2] += gz[j] * gz[j];
        sum[3] += gx[j] * gy[j];
        sum[4] += gx[j] * gz[j];
        sum[5] += gy[j] * gz[j];
      }
    }
    const double w = a.occ[vec];
#pragma unroll
    for (int k = 0; k < 6; ++k) tot[k] += w * sum[k];
  }
  __syncthreads();
  double* red = reinterpret_cast<double*>(lds_raw);  // [waves][6]; the tile is larger
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double v = tot[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) red[(tid >> 6) * 6 + k] = v;
  }
  __syncthreads();
  if (tid < 6) {
    double s = 0.0;
    for (int wv = 0; wv < nthr / 64; ++wv) s += red[wv * 6 + tid];
    a.partial[(int64_t)blockIdx.x * 6 + tid] = s;
  }
}

// out[k] = sum over nblocks of partial[b * 6 + k], one block per k (fixed order).
__global__ __launch_bounds__(256) void stress_sum_kernel(const double* __restrict__ partial, int nblocks,
                                                         double* __restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += 256) s += partial[(int64_t)b * 6 + blockIdx.x];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

template <typename TV, int R, int PY>
hipError_t launch_stress_kh(const StressArgs<TV>& a, int kh, int grid, int threads, size_t lds, hipStream_t s) {
  switch (kh) {
    case 2: hipLaunchKernelGGL((kinetic_stress_kernel<TV, R, PY, 2>), dim3(grid), dim3(threads), lds, s, a); break;
    case 3: hipLaunchKernelGGL((kinetic_stress_kernel<TV, R, PY, 3>), dim3(grid), dim3(threads), lds, s, a); break;
    case 4: hipLaunchKernelGGL((kinetic_stress_kernel<TV, R, PY, 4>), dim3(grid), dim3(threads), lds, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename TV, int R>
hipError_t launch_stress_r(const StressArgs<TV>& a, const HxPlan& p, int grid, size_t lds, hipStream_t s) {
  if (p.py == 1) return launch_stress_kh<TV, R, 1>(a, p.kh, grid, p.threads, lds, s);
  if (p.py == 2) return launch_stress_kh<TV, R, 2>(a, p.kh, grid, p.threads, lds, s);
  return hipErrorInvalidValue;
}

template <typename TV, int R>
hipError_t launch_ng(const NlGradArgs<TV>& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.per_xcd * 8)), block(64 * kNgWaves);
  if (a.box != nullptr) {
    if (a.disp != nullptr)
      hipLaunchKernelGGL((nl_grad_box_kernel<TV, R, true>), grid, dim3(kBoxThreads), 0, s, a);
    else
      hipLaunchKernelGGL((nl_grad_box_kernel<TV, R, false>), grid, dim3(kBoxThreads), 0, s, a);
    return hipGetLastError();
  }
  if (a.disp != nullptr)
    hipLaunchKernelGGL((nl_grad_kernel<TV, R, true>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((nl_grad_kernel<TV, R, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace

template <typename TV>
hipError_t launch_nl_grad(const NlGradArgs<TV>& a0, int radius, double* out, double scale, hipStream_t s) {
  if (a0.n_atoms <= 0 || a0.ns <= 0) return hipSuccess;
  NlGradArgs<TV> a = a0;
  const int per_block = a.disp != nullptr ? 1 : 2;
  const int no = a.disp != nullptr ? 10 : 3;
  a.ngroups = (a.ns + per_block - 1) / per_block;
  if (a.box != nullptr) {  // as many orbitals per block as leave about four blocks per CU
    a.gpo = (int)std::max<int64_t>(1, std::min<int64_t>(kBoxOrb, (int64_t)a.n_atoms * a.ns / 1024));
    a.ngroups = (a.ns + a.gpo - 1) / a.gpo;
  }
  a.per_xcd = (int)(((int64_t)a.n_atoms * a.ngroups + 7) / 8);
  hipError_t e;
  switch (radius) {
    case 1: e = launch_ng<TV, 1>(a, s); break;
    case 2: e = launch_ng<TV, 2>(a, s); break;
    case 3: e = launch_ng<TV, 3>(a, s); break;
    case 4: e = launch_ng<TV, 4>(a, s); break;
    case 5: e = launch_ng<TV, 5>(a, s); break;
    case 6: e = launch_ng<TV, 6>(a, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(atom_sums_kernel, dim3((unsigned)a.n_atoms), dim3(256), 0, s, a.part, a.ns, no, scale, out);
  return hipGetLastError();
}

template <typename TV>
hipError_t launch_stress_sums(const StressArgs<TV>& a0, int radius, int64_t max_partials, hipStream_t s) {
  StressArgs<TV> a = a0;
  // FP64 queue values at two rows per thread and more cost occupancy here as in the filter:
  // the planner's default tiling (one or two rows) serves
  const HxPlan p = plan_hx(a.nx, a.ny, a.nz, a.ns, radius, (int)sizeof(TV), 0, 0);
  if (!p.ok) return hipErrorInvalidConfiguration;
  a.nyg = p.nyg;
  a.ty = p.ty;
  a.nty = p.nty;
  a.zc = p.zc;
  a.nzc = p.nzc;
  a.nunits = (int64_t)p.nty * p.nzc * a.ns;
  a.pitch = hx_pitch(a.nx, radius, (int)sizeof(TV), p.py);
  const int grid = (int)std::min<int64_t>({a.nunits, std::max<int64_t>(1, max_partials), 65535});
  const size_t lds = std::max<size_t>(hx_lds_bytes(p, a.nx, radius, (int)sizeof(TV), -1, 8), 16 * 6 * sizeof(double));
  hipError_t e;
  switch (radius) {
    case 1: e = launch_stress_r<TV, 1>(a, p, grid, lds, s); break;
    case 2: e = launch_stress_r<TV, 2>(a, p, grid, lds, s); break;
    case 3: e = launch_stress_r<TV, 3>(a, p, grid, lds, s); break;
    case 4: e = launch_stress_r<TV, 4>(a, p, grid, lds, s); break;
    case 5: e = launch_stress_r<TV, 5>(a, p, grid, lds, s); break;
    case 6: e = launch_stress_r<TV, 6>(a, p, grid, lds, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(stress_sum_kernel, dim3(6), dim3(256), 0, s, a.partial, grid, a.out);
  return hipGetLastError();
}

template hipError_t launch_stress_sums<double>(const StressArgs<double>&, int, int64_t, hipStream_t);
template hipError_t launch_stress_sums<float>(const StressArgs<float>&, int, int64_t, hipStream_t);
template hipError_t launch_nl_grad<double>(const NlGradArgs<double>&, int, double*, double, hipStream_t);
template hipError_t launch_nl_grad<float>(const NlGradArgs<float>&, int, double*, double, hipStream_t);

}  // namespace chefsi
