// Host runtime of libchefsi: handle, validation, workspace plan, CheFSI step orchestration,
// FP64 dense stage (rocSOLVER) and the C-ABI declared in include/chefsi.h.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <future>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/chefsi.h"
#include "common.h"

using namespace chefsi;

namespace {

constexpr int kNumProf = 8;
// P_FALLBACK counts mixed steps whose projection and rotation were redone in FP64 (no time)
enum ProfId { P_HX = 0, P_NL = 1, P_GRAM = 2, P_REDUCE = 3, P_ROT = 4, P_EIG = 5, P_COPY = 6, P_FALLBACK = 7 };

// A mixed step whose scaled overlap matrix has a Cholesky pivot below this (relative to its
// unit diagonal, i.e. cond(S Ms S) beyond ~1e4) redoes projection and rotation in FP64:
// the split-bf16 products (~1e-5 relative) cannot resolve the weakest filtered directions,
// and the rotation would amplify their error by the inverse pivot.
constexpr double kMixedMinPivot = 1e-4;

struct Error {
  int status;
  std::string msg;
};

// True where an allocation (or the copy into it) failed; the error is not left for the next
// launch to report.
bool no_memory(hipError_t e) {
  if (e != hipSuccess) (void)hipGetLastError();
  return e != hipSuccess;
}

#define HIP_TRY(expr)                                                                         \
  do {                                                                                        \
    hipError_t e_ = (expr);                                                                   \
    if (e_ != hipSuccess) throw Error{CHEFSI_ERR_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)}; \
  } while (0)

#define BLAS_TRY(expr)                                                                         \
  do {                                                                                         \
    rocblas_status s_ = (expr);                                                                \
    if (s_ != rocblas_status_success)                                                          \
      throw Error{CHEFSI_ERR_SOLVER, std::string(#expr) + ": " + rocblas_status_to_string(s_)}; \
  } while (0)

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Central second-derivative weights of even order 2r (closed form of the
// Lagrange-interpolation stencil); Sec. 2.1 names only the order n0.
std::vector<double> fd_weights(int order) {
  const int r = order / 2;
  std::vector<double> w(r + 1, 0.0);
  long double s = 0.0L;
  for (int p = 1; p <= r; ++p) s += 1.0L / ((long double)p * p);
  w[0] = (double)(-2.0L * s);
  auto fact = [](int n) {
    long double f = 1.0L;
    for (int i = 2; i <= n; ++i) f *= i;
    return f;
  };
  for (int p = 1; p <= r; ++p) {
    long double num = 2.0L * fact(r) * fact(r);
    long double den = (long double)p * p * fact(r - p) * fact(r + p);
    w[p] = (double)((p % 2 ? 1.0L : -1.0L) * num / den);
  }
  return w;
}

struct EventPair {
  int id;
  hipEvent_t b, e;
};

}  // namespace

// Scratch of chefsi_apply_h_static: the projector coefficients alpha (np_tot x ns of the
// handle's compute type) live in this file-scope device array instead of a caller
// workspace.  Every GPU the library runs on holds its own copy until the process ends.
// In host code `scratch` names a host-side stand-in, never the device memory: its device
// address is looked up once per device (hipGetSymbolAddress, that device current) and
// only that address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[CHEFSI_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices] = {};

// device address of `scratch` on the current device (looked up on first use per device)
void* scratch_address(int dev) {
  if (dev < 0 || dev >= kMaxScratchDevices) throw Error{CHEFSI_ERR_HIP, "device ordinal out of range"};
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      throw Error{CHEFSI_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
    g_scratch_dev[dev] = p;
  }
  return g_scratch_dev[dev];
}
}  // namespace

namespace {
// plans of the FP64 Gram products through rocBLAS, of the widened row panels, and a call's workspace
// (see plan_blas_gram, plan_panels, layout)
constexpr int kMaxGramBlocks = 8;

struct BlasGram {
  int splits = 1;
  int64_t kc = 0, tail = 0;
  int nparts = 1;
  size_t bytes = 0;
  int nblk = 1;                         // column blocks
  int start[kMaxGramBlocks + 1] = {0};  // block b is columns [start[b], start[b+1])
};

struct PanelPlan {
  int splits = 1;
  int64_t kc = 0, rows = 0;
  size_t part_bytes = 0;   // one set of Gram partials
  size_t panel_bytes = 0;  // one rows x ns FP64 panel
};

struct WsLayout {
  size_t bufB = 0, alpha = 0, hs = 0, ms = 0, d = 0, e = 0, sc = 0, info = 0, msg = 0, partial = 0, zsplit = 0,
         panel = 0, panel_out = 0, band = 0, chol = 0, solver = 0, total = 0;
  size_t bufB_bytes = 0, solver_bytes = 0, band_bytes = 0;
  GramPlan gram;
  BlasGram bgram;   // FP64 handles: Gram products of FP64 blocks
  GramBothPlan both;  // the same in one launch
  PanelPlan pan;    // mixed handles: FP64 products of the FP32 block
  PairPlan pair;    // mixed handles: both split-bf16 Gram products at once
};

}  // namespace

constexpr int kNoBand = INT32_MAX;

// Band-pass tables on the device (built while rec_max == 0, or for band_apply and band_filter).
struct BandDevice {
  int nb_reg = 0, nb_pts = 0, nb_slots = 0;
  int* nb_reg_pt = nullptr;
  int* nb_pt_idx = nullptr;
  int* nb_pt_ent = nullptr;
  int* nb_ent_ls = nullptr;
  int* nb_slot_q = nullptr;
  double* nb_ent_chi64 = nullptr;
  float* nb_ent_chi32 = nullptr;
  int* nb_reg_slot = nullptr;
  int* nb_slot_ent = nullptr;
  int* nb_gent_loc = nullptr;
  double* nb_gent_chi64 = nullptr;
  float* nb_gent_chi32 = nullptr;
  int* nb_q_slot_ptr = nullptr;
  int* nb_q_slot = nullptr;
  void* nb_partial = nullptr;     // nb_slots x (a run of orbitals) values
  size_t nb_partial_bytes = 0;
  size_t nb_bytes = 0;  // of all of them
};

struct chefsi_handle : BandDevice {
  int device = 0;
  int cus = 0;              // compute units of the device
  size_t device_bytes = 0;  // sum of the handle's own device arrays
  int precision = CHEFSI_FP64;
  int n[3] = {0, 0, 0};
  double h[3] = {0, 0, 0};
  int bc[3] = {0, 0, 0};
  int order = 12, radius = 6;
  int64_t nd = 0;
  int max_ns = 0;
  double dv = 0.0;
  std::vector<double> w;

  // host copies kept for the spectral bounds
  std::vector<double> veff_h;
  int n_atoms = 0;
  int np_tot = 0;
  std::vector<int64_t> supp_ptr_h;
  std::vector<int> supp_idx_h, nproj_h;
  std::vector<double> chi_h, gamma_h;

  // device data
  double* veff64 = nullptr;
  float* veff32 = nullptr;
  int* supp_off = nullptr;
  int* supp_idx = nullptr;
  int64_t* chi_off = nullptr;
  int* nproj = nullptr;
  int* poff = nullptr;
  int* supp_box = nullptr;  // 6 per atom; null when an atom's support is too large for the LDS gradient
  double* chi64 = nullptr;
  float* chi32 = nullptr;
  double* gdv64 = nullptr;
  float* gdv32 = nullptr;
  // projector entries grouped by (y tile, z plane) of the stencil tiling: one record per touched point
  HxPlan hx_plan;  // tiling for ns = 1 (checked at create; the z chunking depends on ns)
  int4* rec = nullptr;           // scatter records (points with more than four entries)
  int* hx_rec_ptr = nullptr;     // stencil-pass records (points with at most four entries)
  HxRec<double>* hx_rec64 = nullptr;
  HxRec<float>* hx_rec32 = nullptr;
  int* ent_col = nullptr;
  double* ent_val64 = nullptr;
  float* ent_val32 = nullptr;
  // pinned host staging for the small device-to-host reads (Ritz values, dense-stage status,
  // Cholesky pivots: max_ns doubles + 16 status words; force and stress sums: 10 per atom;
  // Lanczos coefficients)
  double* pinned = nullptr;
  int n_pts = 0;     // scatter records
  int n_hxrec = 0;   // stencil-pass records
  size_t hx_rec_bytes = 0;   // device bytes of the stencil-pass records
  size_t scatter_bytes = 0;  // device bytes of the scatter records and entries
  // points in at most this many projector entries take their projector term inside the
  // stencil pass (4: the record width), the others in the scatter pass; 0: every term in
  // the band pass (nl_band) instead
  int rec_max = 4;
  // a handle as created has the band pass beside the records for calls on at least this many
  // orbitals: single applications, and filters (band_from)
  int band_apply = kNoBand, band_filter = kNoBand;
  // slots of a handle that was created with the band pass (0: it was not): its workspaces carry
  // the partials, nb_partial serves only the calls without one
  int ws_band_slots = 0;

  rocblas_handle blas = nullptr;
  std::map<int, WsLayout> layouts;  // by ns: the plans cost a small call more than its launches
  // point-major projector table (host): point i lists pt_col/pt_val[pt_cnt[i] .. pt_cnt[i+1]),
  // kept so the stencil-pass records can be rebuilt for another tiling
  std::vector<int> pt_cnt, pt_col;
  std::vector<double> pt_val;

  bool prof_on = false;
  std::vector<hipEvent_t> ev_pool;
  std::vector<EventPair> ev_pending;
  double prof_ms[kNumProf] = {0};
  int64_t prof_n[kNumProf] = {0};

  int last_info = 0;
  std::string last_error;
};

namespace {

// FP64 Gram products through rocBLAS as split-K: `splits` K chunks of kc rows as one
// strided-batched dgemm, the tail rows (fewer than splits) as one more dgemm, and the
// partial products summed in a fixed order.  Chunks are no shorter than 2048 rows and
// about 4096 output tiles of 128 x 128 are in flight over all chunks.
// Only the upper triangle of the symmetric product is needed: the columns are cut into
// blocks and block row i is formed against columns [start_i, ns) alone, which skips most
// of the lower triangle's work.
// Column blocks of the upper-triangle Gram (split-K batches of rocBLAS dgemm, measured at
// ns = 600 and 1200): up to ns = 1024, blocks of 128 columns (ns = 600: 2.6 vs 4.2 ms for
// the full product); above, three blocks cut near 0.43 ns and 0.75 ns (ns = 1200 at 512
// and 896: 21.0 vs 28.8 ms); small blocks run too few tiles to pay.
void gram_blocks(int ns, int& nblk, int* start) {
  nblk = 0;
  start[0] = 0;
  if (ns < 256) {
    nblk = 1;
  } else if (ns <= 128 * kMaxGramBlocks) {
    for (int c = 128; c < ns; c += 128) start[++nblk] = c;
    ++nblk;
  } else {
    start[1] = (int)std::lround(0.43 * ns / 128.0) * 128;
    start[2] = (int)std::lround(0.75 * ns / 128.0) * 128;
    nblk = 3;
  }
  start[nblk] = ns;
}

BlasGram plan_blas_gram(int64_t nd, int ns) {
  BlasGram b;
  const int64_t tiles = ((int64_t)(ns + 127) / 128) * ((ns + 127) / 128);
  b.splits = (int)std::max<int64_t>(1, std::min<int64_t>({128, 4096 / tiles, nd / 2048}));
  b.kc = nd / b.splits;
  b.tail = nd - b.kc * b.splits;
  b.nparts = b.splits + (b.tail > 0 ? 1 : 0);
  b.bytes = (size_t)b.nparts * ns * ns * sizeof(double);
  gram_blocks(ns, b.nblk, b.start);
  return b;
}

// gram_f64.hip forms both products in one launch and is the faster of the two everywhere but
// on columns a multiple of 2 MiB apart: there the columns' lines of one row all fall into one
// set of the L2 and the 64-wide tiles lose their reuse.  rocBLAS's 128-wide ones win above 512
// orbitals, and on strides of 4 MiB and more from 353 on where their last tile is more than seven
// eighths full.  One projection, own / rocBLAS (ms): 64^3 (2 MiB) 500 orbitals 3.49 / 3.68, 600
// 4.77 / 4.34 (products alone), 900 11.7 / 10.5; 64x128x64 (4 MiB) 300 3.35 / 3.94, 384 4.99 /
// 4.44, 448 6.15 / 6.39, 500 7.63 / 6.94; 64x160x128 (10 MiB) 448 17.5 / 18.0, 460 20.9 / 18.0;
// 96x128x64 (6 MiB) 384 8.10 / 8.08, 500 12.9 / 12.3; 128x128x64 (8 MiB) 400 12.7 / 12.5, 448 13.7
// / 13.5, 500 17.3 / 15.8; strides of an odd multiple of 1 MiB 0.7 to 0.9; 72^3 600 5.3 / 6.2
// (products alone), 24^3 40 17 / 274 us.
bool blas_gram_faster(int64_t nd, int ns) {
  const int64_t stride = 1 << 18;  // 2 MiB of doubles
  if (nd % stride != 0) return false;
  return ns > 512 || (nd > stride && ns > 352 && 8 * ns > 7 * ((ns + 127) / 128 * 128));
}

// FP64 products of the FP32 block of a mixed handle (its FP64 Rayleigh-Ritz pass): the
// block is widened to FP64 one row panel at a time and each panel goes to rocBLAS dgemm.
// A panel is `splits` chunks of kc rows; the Gram partials of chunk q of every panel
// accumulate into partial q in panel order, then the partials are summed in a fixed
// order.  A panel holds at most kPanelBytes and a quarter of the rows, so it fits beside
// the FP32 result in the upper half of the FP64 scratch block.
constexpr int64_t kPanelBytes = (int64_t)512 << 20;

PanelPlan plan_panels(int64_t nd, int ns) {
  PanelPlan p;
  const int64_t tiles = ((int64_t)(ns + 127) / 128) * ((ns + 127) / 128);
  const int64_t budget = std::max<int64_t>(1, std::min<int64_t>(kPanelBytes / ((int64_t)ns * 8), nd / 4));
  int64_t splits = std::max<int64_t>(1, std::min<int64_t>({128, 4096 / tiles, budget / 2048}));
  const int64_t kc = std::max<int64_t>(1, budget / splits);
  p.splits = (int)splits;
  p.kc = kc;
  p.rows = splits * kc;
  p.part_bytes = (size_t)splits * ns * ns * sizeof(double);
  p.panel_bytes = (size_t)p.rows * ns * sizeof(double);
  return p;
}

// status words in the pinned staging buffer, after max_ns doubles
rocblas_int* pinned_info(chefsi_handle* h) { return reinterpret_cast<rocblas_int*>(h->pinned + h->max_ns); }

size_t elem_bytes(const chefsi_handle* h) { return h->precision == CHEFSI_FP64 ? 8 : 4; }


// The subspace eigensolve tridiagonalises with the library's own kernel where its workgroups
// (one per compute unit, waiting for each other) are all resident at once; above its sizes
// rocSOLVER's syevd does the whole eigensolve.  n = 600: 7.2 against 14.8 ms for the subspace
// problem; 1200: 16.2 / 30.8; 40: 0.63 / 1.10.
bool own_tridiag(const chefsi_handle* h, int ns) {
  const int g = tridiag_groups(ns);
  return g > 0 && g <= h->cus;
}

// Bytes of the band pass's slot partials (a block with more orbitals forms them in runs of
// kBandRunStep orbitals' multiples), and the fewest orbitals a run has to hold.
constexpr size_t kBandPartialBytes = (size_t)256 << 20;
constexpr size_t kBandMinOrbitals = 64;
constexpr int kBandRunStep = 32;

// Slot partials of the band pass over ns orbitals (one FP64 orbital at least: the FP64 pass of
// a mixed handle uses the same bytes).
size_t band_partial_bytes(const chefsi_handle* h, int slots, int ns) {
  const size_t per = (size_t)std::max(1, slots) * elem_bytes(h);
  const size_t cap = std::max(kBandPartialBytes, per * kBandMinOrbitals);
  return std::max(std::min(per * ns, cap), (size_t)std::max(1, slots) * 8);
}

// Device workspace of the FP64 dense stage (Cholesky, two triangular solves for the
// reduced matrix, symmetric eigensolve, back substitution); the calls run in sequence,
// so the largest single request is enough.
size_t solver_workspace(chefsi_handle* h, int ns) {
  const double one = 1.0;
  size_t best = 0, sz = 0;
  auto query = [&](auto&& call) {
    BLAS_TRY(rocblas_start_device_memory_size_query(h->blas));
    call();
    BLAS_TRY(rocblas_stop_device_memory_size_query(h->blas, &sz));
    best = std::max(best, sz);
  };
  if (ns > kCholMax) {
    query([&] { rocsolver_dpotrf(h->blas, rocblas_fill_upper, ns, nullptr, ns, nullptr); });
    query([&] {
      rocblas_dtrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_transpose,
                    rocblas_diagonal_non_unit, ns, ns, &one, nullptr, ns, nullptr, ns);
    });
    query([&] {
      rocblas_dtrsm(h->blas, rocblas_side_right, rocblas_fill_upper, rocblas_operation_none,
                    rocblas_diagonal_non_unit, ns, ns, &one, nullptr, ns, nullptr, ns);
    });
    query([&] {
      rocblas_dtrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_none,
                    rocblas_diagonal_non_unit, ns, ns, &one, nullptr, ns, nullptr, ns);
    });
  }
  if (own_tridiag(h, ns))
    query([&] { rocsolver_dstedc(h->blas, rocblas_evect_tridiagonal, ns, nullptr, nullptr, nullptr, ns, nullptr); });
  else
    query([&] {
      rocsolver_dsyevd(h->blas, rocblas_evect_original, rocblas_fill_upper, ns, nullptr, ns, nullptr, nullptr,
                       nullptr);
    });
  if (h->precision == CHEFSI_FP64) {
    const BlasGram b = plan_blas_gram(h->nd, ns);
    if (blas_gram_faster(h->nd, ns)) query([&] {
      rocblas_dgemm_strided_batched(h->blas, rocblas_operation_transpose, rocblas_operation_none, ns, ns,
                                    (rocblas_int)b.kc, &one, nullptr, (rocblas_int)h->nd, b.kc, nullptr,
                                    (rocblas_int)h->nd, b.kc, &one, nullptr, ns, (rocblas_stride)ns * ns, b.splits);
    });
  } else {
    const PanelPlan p = plan_panels(h->nd, ns);
    query([&] {
      rocblas_dgemm_strided_batched(h->blas, rocblas_operation_transpose, rocblas_operation_none, ns, ns,
                                    (rocblas_int)p.kc, &one, nullptr, (rocblas_int)p.rows, p.kc, nullptr,
                                    (rocblas_int)h->nd, p.kc, &one, nullptr, ns, (rocblas_stride)ns * ns, p.splits);
    });
    query([&] {
      rocblas_dgemm(h->blas, rocblas_operation_none, rocblas_operation_none, (rocblas_int)p.rows, ns, ns, &one,
                    nullptr, (rocblas_int)p.rows, nullptr, ns, &one, nullptr, (rocblas_int)p.rows);
    });
  }
  if ((int64_t)h->nd * ns < ((int64_t)1 << 31))
    query([&] {
      rocblas_dgemm(h->blas, rocblas_operation_none, rocblas_operation_none, (rocblas_int)h->nd, ns, ns, &one,
                    nullptr, (rocblas_int)h->nd, nullptr, ns, &one, nullptr, (rocblas_int)h->nd);
    });
  return best;
}

const WsLayout& layout(chefsi_handle* h, int ns) {
  const auto known = h->layouts.find(ns);
  if (known != h->layouts.end()) return known->second;
  WsLayout L;
  size_t off = 0;
  L.bufB = off;
  // mixed handles need an FP64 Nd x ns scratch for the FP64 Rayleigh-Ritz pass: same bytes as FP64 X
  L.bufB_bytes = (size_t)h->nd * ns * 8;
  off += align256(L.bufB_bytes);
  L.alpha = off;
  off += align256((size_t)std::max(1, h->np_tot) * ns * 8);
  L.hs = off;
  off += align256((size_t)ns * ns * 8);
  L.ms = off;
  off += align256((size_t)ns * ns * 8);
  L.d = off;
  off += align256((size_t)ns * 8);
  L.e = off;
  off += align256((size_t)ns * 8);
  L.sc = off;
  off += align256((size_t)ns * 8);
  L.info = off;
  off += 256;
  L.msg = off;
  off += align256(tridiag_msg_bytes(ns));
  L.gram = plan_gram(h->nd, ns);
  L.bgram = plan_blas_gram(h->nd, ns);
  L.both = plan_gram_both(h->nd, ns);
  L.pan = plan_panels(h->nd, ns);
  L.partial = off;
  // (the eigensolve also keeps ns^2 values there)
  const size_t part_bytes = h->precision == CHEFSI_FP64
                                ? std::max({L.both.bytes, blas_gram_faster(h->nd, ns) ? L.bgram.bytes : 0,
                                            (size_t)ns * ns * sizeof(double)})
                                : std::max(L.gram.partial_bytes, 2 * L.pan.part_bytes);
  if (h->precision == CHEFSI_MIXED) {
    L.pair = plan_gram_pair(h->nd, ns, L.gram, part_bytes);
  }
  off += align256(part_bytes);
  L.zsplit = off;
  if (h->precision == CHEFSI_MIXED) off += align256(zsplit_bytes(ns));
  L.panel = off;
  if (h->precision == CHEFSI_MIXED) {
    off += align256(L.pan.panel_bytes);
    // the rotation's FP64 result panel: above the FP32 result in the FP64 scratch block
    // (it fits there unless the grid is tiny), else a region of its own
    L.panel_out = L.bufB + align256((size_t)h->nd * ns * 4);
    if (L.panel_out + L.pan.panel_bytes > L.bufB + align256(L.bufB_bytes)) {
      L.panel_out = off;
      off += align256(L.pan.panel_bytes);
    }
  }
  L.chol = off;
  off += align256(chol_scratch_bytes(ns));
  L.band = off;
  if (h->ws_band_slots > 0) L.band_bytes = band_partial_bytes(h, h->ws_band_slots, ns);
  off += align256(L.band_bytes);
  L.solver = off;
  L.solver_bytes = solver_workspace(h, ns);
  off += align256(std::max<size_t>(L.solver_bytes, 256));
  L.total = off;
  return h->layouts.emplace(ns, L).first->second;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// ---- profiling -------------------------------------------------------------
// HIP events around the launches of one kernel class on the call's stream (any handle type
// with prof_on, ev_pool, ev_pending, prof_ms and prof_n).
template <typename H>
struct ProfScopeT {
  H* h;
  hipStream_t s;
  int id;
  hipEvent_t b = nullptr, e = nullptr;
  ProfScopeT(H* h_, int id_, hipStream_t s_) : h(h_), s(s_), id(id_) {
    if (!h->prof_on) return;
    b = take();
    e = take();
    HIP_TRY(hipEventRecord(b, s));
  }
  hipEvent_t take() {
    if (!h->ev_pool.empty()) {
      hipEvent_t ev = h->ev_pool.back();
      h->ev_pool.pop_back();
      return ev;
    }
    hipEvent_t ev;
    HIP_TRY(hipEventCreate(&ev));
    return ev;
  }
  void done() {
    if (!h->prof_on || b == nullptr) return;
    HIP_TRY(hipEventRecord(e, s));
    h->ev_pending.push_back({id, b, e});
    b = e = nullptr;
  }
  ~ProfScopeT() {
    if (b) h->ev_pool.push_back(b);
    if (e) h->ev_pool.push_back(e);
  }
};
using ProfScope = ProfScopeT<chefsi_handle>;

template <typename H>
void prof_collect(H* h) {
  for (auto& p : h->ev_pending) {
    HIP_TRY(hipEventSynchronize(p.e));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, p.b, p.e));
    h->prof_ms[p.id] += ms;
    h->prof_n[p.id] += 1;
    h->ev_pool.push_back(p.b);
    h->ev_pool.push_back(p.e);
  }
  h->ev_pending.clear();
}

// ---- argument checks -------------------------------------------------------
void check(bool ok, const char* what) {
  if (!ok) throw Error{CHEFSI_ERR_INVALID_ARG, what};
}

void check_ns(const chefsi_handle* h, int ns) {
  check(ns >= 1 && ns <= h->max_ns, "ns must satisfy 1 <= ns <= max_ns");
  check((int64_t)ns <= h->nd, "ns must not exceed Nd");
}

void check_ws(chefsi_handle* h, int ns, void* ws, size_t ws_bytes, WsLayout& L) {
  L = layout(h, ns);
  if (ws == nullptr || ws_bytes < L.total)
    throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_workspace_bytes(ns)"};
  check(((uintptr_t)ws & 255) == 0, "workspace must be 256-byte aligned");
}

void check_bounds(double lo, double cut, double hi) {
  check(std::isfinite(lo) && std::isfinite(cut) && std::isfinite(hi), "spectral bounds must be finite");
  check(lo <= cut && cut < hi, "bounds must satisfy lam_lo <= lam_cut < lam_hi");
}

// ---- kernel wrappers -------------------------------------------------------
template <typename TI, typename TC, typename TO>
HxArgs<TI, TC, TO> hx_args(const chefsi_handle* h, const TI* x, const TO* prev, TO* out, const TC* veff,
                           const TC* alpha, bool records) {
  HxArgs<TI, TC, TO> a{};
  a.x = x;
  a.prev = prev;
  a.out = out;
  a.veff = veff;
  a.rec_ptr = records && h->n_hxrec > 0 ? h->hx_rec_ptr : nullptr;
  if constexpr (sizeof(TC) == 8)
    a.rec = h->hx_rec64;
  else
    a.rec = h->hx_rec32;
  a.alpha = alpha;
  a.np_tot = h->np_tot;
  a.nx = h->n[0];
  a.ny = h->n[1];
  a.nz = h->n[2];
  a.nd = h->nd;
  a.per_x = h->bc[0] == 0;
  a.per_y = h->bc[1] == 0;
  a.per_z = h->bc[2] == 0;
  double sumh = 0.0;
  for (int d = 0; d < 3; ++d) sumh += 1.0 / (h->h[d] * h->h[d]);
  a.c0 = TC(-0.5 * h->w[0] * sumh);
  for (int p = 0; p <= kMaxRadius; ++p) {
    const double wp = p <= h->radius ? h->w[p] : 0.0;
    a.cx[p] = TC(-0.5 * wp / (h->h[0] * h->h[0]));
    a.cy[p] = TC(-0.5 * wp / (h->h[1] * h->h[1]));
    a.cz[p] = TC(-0.5 * wp / (h->h[2] * h->h[2]));
  }
  a.sa = TC(1);
  a.sc = TC(0);
  a.sb = TC(0);
  return a;
}

template <typename TI, typename TC>
NlArgs<TI, TC> nl_args(const chefsi_handle* h, const TI* y, int ns, const TC* chi, const TC* gdv, TC* alpha) {
  NlArgs<TI, TC> a{};
  a.y = y;
  a.nd = h->nd;
  a.ns = ns;
  a.n_atoms = h->n_atoms;
  a.supp_off = h->supp_off;
  a.supp_idx = h->supp_idx;
  a.chi_off = h->chi_off;
  a.nproj = h->nproj;
  a.poff = h->poff;
  a.chi = chi;
  a.gdv = gdv;
  a.alpha = alpha;
  a.np_tot = h->np_tot;
  return a;
}

// out = sa (H x - sc x) + sb prev, with the projector gather for x first.
// out = sa ((H x) - sc x) + sb prev: projector gather (alpha), the stencil + Veff +
// Chebyshev pass, then the projector scatter onto the support points.
// Where a call's slot partials go: its own workspace if that has room for them, else the
// handle's buffer.
struct BandScratch {
  void* p;
  size_t bytes;
};

template <typename Layout>
BandScratch band_scratch(const chefsi_handle* h, void* ws, const Layout& L) {
  if (L.band_bytes > 0) return {at<void>(ws, L.band), L.band_bytes};
  return {h->nb_partial, h->nb_partial_bytes};
}

// Band-pass arguments for block y (the handle's tables for compute type TC).
template <typename TY, typename TC>
NbArgs<TY, TC> band_args(const chefsi_handle* h, TY* y, int ns, const TC* alpha, double sa) {
  NbArgs<TY, TC> a{};
  a.y = y;
  a.nd = h->nd;
  a.ns = ns;
  a.nreg = h->nb_reg;
  a.reg_pt = h->nb_reg_pt;
  a.pt_idx = h->nb_pt_idx;
  a.pt_ent = h->nb_pt_ent;
  a.ent_ls = h->nb_ent_ls;
  a.slot_q = h->nb_slot_q;
  a.reg_slot = h->nb_reg_slot;
  a.slot_ent = h->nb_slot_ent;
  a.gent_loc = h->nb_gent_loc;
  if constexpr (sizeof(TC) == 8) {
    a.ent_chi = h->nb_ent_chi64;
    a.gent_chi = h->nb_gent_chi64;
  } else {
    a.ent_chi = h->nb_ent_chi32;
    a.gent_chi = h->nb_gent_chi32;
  }
  a.alpha = alpha;
  a.sa = TC(sa);
  return a;
}

// The band pass over block y, and with want_alpha the projector-major coefficients alpha of
// the finished block from its slot partials.  The partials of a run of orbitals are written
// and added up before the next run (their buffer is bounded, and a run's values are still in
// the memory-side cache when they are read).
template <typename TY, typename TC>
void band_alpha(chefsi_handle* h, TY* y, int ns, TC* alpha, const TC* gdv, bool scatter, double sa,
                bool want_alpha, hipStream_t s, BandScratch bs) {
  if (h->nb_q_slot_ptr == nullptr) throw Error{CHEFSI_ERR_HIP, "the handle has no band-pass tables"};
  ProfScope ps(h, P_NL, s);
  int run = ns;
  if (want_alpha)
    run = (int)std::min<size_t>(ns, std::max<size_t>(1, bs.bytes / (std::max(1, h->nb_slots) * sizeof(TC))));
  if (run < ns && run > kBandRunStep) run = run / kBandRunStep * kBandRunStep;
  for (int v0 = 0; v0 < ns; v0 += run) {
    const int n = std::min(run, ns - v0);
    NbArgs<TY, TC> a = band_args<TY, TC>(h, y + (int64_t)v0 * h->nd, n, alpha + v0, sa);
    a.lda = ns;
    a.partial = static_cast<TC*>(bs.p);
    HIP_TRY((launch_nl_band<TY, TC>(a, scatter, want_alpha, s)));
    if (want_alpha)
      HIP_TRY(launch_nl_band_reduce<TC>(a.partial, h->nb_q_slot_ptr, h->nb_q_slot, gdv,
                                        h->np_tot, n, ns, alpha + v0, s));
  }
  ps.done();
}

// out = sa ((H - sc) x) + sb prev.  The projector term takes one of two routes: stencil-pass
// records plus a scatter pass for the points in more than four entries (the gather nl_project
// first), or, on a handle switched to the band pass, nl_band after a bare stencil pass.  In
// the band route alpha holds projector-major coefficients: alpha_ready says they are already
// those of x (the previous application computed them), want_next asks for those of out.
// in_filter: an application of the filter (or the one that follows it), for which a handle as
// created has another limit (band_filter).
template <typename TI, typename TC, typename TO>
void apply_fused(chefsi_handle* h, const TI* x, const TO* prev, TO* out, int ns, double sa, double sc, double sb,
                 TC* alpha, hipStream_t s, BandScratch bs, bool alpha_ready = false, bool want_next = false,
                 bool in_filter = false) {
  const TC* veff;
  const TC* nlv;
  const TC* chi;
  const TC* gdv;
  if constexpr (sizeof(TC) == 8) {
    veff = h->veff64;
    nlv = h->ent_val64;
    chi = h->chi64;
    gdv = h->gdv64;
  } else {
    veff = h->veff32;
    nlv = h->ent_val32;
    chi = h->chi32;
    gdv = h->gdv32;
  }
  const bool band = h->np_tot > 0 && (h->rec_max == 0 || ns >= (in_filter ? h->band_filter : h->band_apply));
  if (band) {
    if (!alpha_ready) band_alpha<TI, TC>(h, const_cast<TI*>(x), ns, alpha, gdv, false, 0.0, true, s, bs);
  } else if (h->np_tot > 0) {
    ProfScope ps(h, P_NL, s);
    HIP_TRY((launch_nl_project<TI, TC>(nl_args<TI, TC>(h, x, ns, chi, gdv, alpha), s)));
    ps.done();
  }
  auto a = hx_args<TI, TC, TO>(h, x, prev, out, veff, alpha, !band);
  a.sa = TC(sa);
  a.sc = TC(sc);
  a.sb = TC(sb);
  {
    ProfScope ps(h, P_HX, s);
    const HxPlan p = plan_hx(h->n[0], h->n[1], h->n[2], ns, h->radius, (int)sizeof(TI), h->hx_plan.py, h->hx_plan.nyg);
    if (!p.ok || p.ty != h->hx_plan.ty)
      throw Error{CHEFSI_ERR_HIP, "stencil tiling differs from the one the projector records were built for"};
    HIP_TRY((launch_hx<TI, TC, TO>(a, p, h->radius, ns, s)));
    ps.done();
  }
  if (band) {
    band_alpha<TO, TC>(h, out, ns, alpha, gdv, true, sa, want_next, s, bs);
  } else if (h->n_pts > 0) {  // points in more than rec_max entries
    NsArgs<TC, TO> n{};
    n.out = out;
    n.nd = h->nd;
    n.ns = ns;
    n.rec = h->rec;
    n.n_pts = h->n_pts;
    n.col = h->ent_col;
    n.val = nlv;
    n.alpha = alpha;
    n.np_tot = h->np_tot;
    n.sa = TC(sa);
    ProfScope ps(h, P_NL, s);
    HIP_TRY((launch_nl_scatter<TC, TO>(n, s)));
    ps.done();
  }
}

// Scaled Chebyshev filter (Alg. 1, Filtering).  Y_0 = X in buffer A; Y_{k+1} overwrites Y_{k-1}.
// Returns the buffer that holds Y_m (A when m is even, B when odd).
// With carry_last, alpha ends as the band-pass coefficients of the returned block.
template <typename T>
T* run_filter(chefsi_handle* h, T* A, T* B, int ns, int m, double lo, double cut, double hi, T* alpha,
              hipStream_t s, BandScratch bs, bool carry_last = false) {
  const double c = 0.5 * (hi + cut);
  const double e = 0.5 * (hi - cut);
  const double s1 = e / (lo - c);
  double sig = s1;
  // Y_1 = (s1 / e)(H - c) Y_0
  apply_fused<T, T, T>(h, A, nullptr, B, ns, s1 / e, c, 0.0, alpha, s, bs, false, m > 1 || carry_last, true);
  T* cur = B;
  T* other = A;
  for (int k = 1; k < m; ++k) {
    const double sig_next = 1.0 / (2.0 / s1 - sig);
    apply_fused<T, T, T>(h, cur, other, other, ns, 2.0 * sig_next / e, c, -sig * sig_next, alpha, s, bs, true,
                         k + 1 < m || carry_last, true);
    std::swap(cur, other);
    sig = sig_next;
  }
  return cur;
}

// Arithmetic of the dense products: FP64 MFMA, or split bf16 (three bf16 MFMAs per
// product, FP32 accumulation) for the FP32 blocks of a mixed handle.
enum class Gemm { F64, BF16X3 };

template <typename TX, typename TY>
hipError_t gram_launch(Gemm g, const TX* X, const TY* Y, int64_t nd, int ns, const GramPlan& p, double* part,
                       hipStream_t s) {
  if constexpr (std::is_same<TX, float>::value && std::is_same<TY, float>::value) {
    if (g == Gemm::BF16X3) return launch_gram_bf16x3(X, Y, nd, ns, p, part, s);
  }
  return launch_gram_f64<TX, TY>(X, Y, nd, ns, p, part, s);
}

// C = X^T Y (upper triangle, mirrored) for FP64 blocks of an FP64 handle: rocBLAS's MFMA
// dgemm over K chunks (a plain GEMM: no fusion to gain), partials summed in a fixed order.
void blas_gram(chefsi_handle* h, const double* X, const double* Y, int ns, const WsLayout& L, void* ws, double* C,
               hipStream_t s) {
  double* part = at<double>(ws, L.partial);
  const BlasGram& b = L.bgram;
  const double one = 1.0, zero = 0.0;
  const rocblas_int ld = (rocblas_int)h->nd;
  {
    ProfScope ps(h, P_GRAM, s);
    BLAS_TRY(rocblas_set_stream(h->blas, s));
    BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
    for (int q = 0; q < b.nblk; ++q) {
      // block row q against columns [r0, ns): rows r0 .. r0 + m - 1 of every partial
      const int r0 = b.start[q], m = b.start[q + 1] - r0, n = ns - r0;
      const double* Xq = X + (size_t)r0 * h->nd;
      const double* Yq = Y + (size_t)r0 * h->nd;
      double* Pq = part + r0 + (size_t)r0 * ns;
      BLAS_TRY(rocblas_dgemm_strided_batched(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                                             (rocblas_int)b.kc, &one, Xq, ld, b.kc, Yq, ld, b.kc, &zero, Pq, ns,
                                             (rocblas_stride)ns * ns, b.splits));
      if (b.tail > 0) {
        const int64_t k0 = b.kc * b.splits;
        BLAS_TRY(rocblas_dgemm(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                               (rocblas_int)b.tail, &one, Xq + k0, ld, Yq + k0, ld, &zero,
                               Pq + (size_t)b.splits * ns * ns, ns));
      }
    }
    ps.done();
  }
  {
    ProfScope ps(h, P_REDUCE, s);
    HIP_TRY(launch_sum_partials(part, b.nparts, ns, C, s));
    ps.done();
  }
}

// Hs = X^T Y and Ms = X^T X with FP64 arithmetic for the FP32 block X of a mixed handle
// (Y = H X in FP64): each row panel of X is widened once and feeds both rocBLAS products.
// Every FP32 value is exact in FP64, so this is the FP64 product of the stored block.
void panel_gram(chefsi_handle* h, const float* X, const double* Y, int ns, const WsLayout& L, void* ws, double* Hs,
                double* Ms, hipStream_t s) {
  const PanelPlan& p = L.pan;
  double* W = at<double>(ws, L.panel);
  double* partH = at<double>(ws, L.partial);
  double* partM = partH + (size_t)p.splits * ns * ns;
  const double one = 1.0, zero = 0.0;
  const rocblas_int ldw = (rocblas_int)p.rows, ldy = (rocblas_int)h->nd;
  const rocblas_stride pst = (rocblas_stride)ns * ns;
  {
    ProfScope ps(h, P_GRAM, s);
    BLAS_TRY(rocblas_set_stream(h->blas, s));
    BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
    for (int64_t r0 = 0; r0 < h->nd; r0 += p.rows) {
      // the first panel is whole (rows <= nd) and sets every partial; later panels add
      const int64_t r = std::min(p.rows, h->nd - r0);
      const double* beta = r0 == 0 ? &zero : &one;
      HIP_TRY(launch_widen_rows(X + r0, h->nd, r, ns, W, p.rows, s));
      const int64_t nfull = r / p.kc, tail = r - nfull * p.kc;
      for (int q = 0; q < L.bgram.nblk; ++q) {
        // upper triangle only: block row q of the product against columns [c0, ns)
        const int c0 = L.bgram.start[q], m = L.bgram.start[q + 1] - c0, n = ns - c0;
        const double* Wq = W + (size_t)c0 * p.rows;
        const double* Yq = Y + r0 + (size_t)c0 * h->nd;
        const size_t co = c0 + (size_t)c0 * ns;
        if (nfull > 0) {
          BLAS_TRY(rocblas_dgemm_strided_batched(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                                                 (rocblas_int)p.kc, &one, Wq, ldw, p.kc, Yq, ldy, p.kc, beta,
                                                 partH + co, ns, pst, (rocblas_int)nfull));
          BLAS_TRY(rocblas_dgemm_strided_batched(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                                                 (rocblas_int)p.kc, &one, Wq, ldw, p.kc, Wq, ldw, p.kc, beta,
                                                 partM + co, ns, pst, (rocblas_int)nfull));
        }
        if (tail > 0) {  // only in a last, partial panel: nfull < splits and r0 > 0
          const int64_t k0 = nfull * p.kc;
          BLAS_TRY(rocblas_dgemm(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                                 (rocblas_int)tail, &one, Wq + k0, ldw, Yq + k0, ldy, &one,
                                 partH + co + nfull * pst, ns));
          BLAS_TRY(rocblas_dgemm(h->blas, rocblas_operation_transpose, rocblas_operation_none, m, n,
                                 (rocblas_int)tail, &one, Wq + k0, ldw, Wq + k0, ldw, &one,
                                 partM + co + nfull * pst, ns));
        }
      }
    }
    ps.done();
  }
  {
    ProfScope ps(h, P_REDUCE, s);
    HIP_TRY(launch_sum_partials(partH, p.splits, ns, Hs, s));
    HIP_TRY(launch_sum_partials(partM, p.splits, ns, Ms, s));
    ps.done();
  }
}

// O = X Z with FP64 arithmetic for the FP32 block X of a mixed handle, rounded once to
// FP32: per row panel, widen, rocBLAS dgemm into the FP64 result panel, narrow into O.
void panel_rotate(chefsi_handle* h, const float* X, const double* Z, float* O, int ns, const WsLayout& L, void* ws,
                  hipStream_t s) {
  ProfScope ps(h, P_ROT, s);
  const PanelPlan& p = L.pan;
  double* W = at<double>(ws, L.panel);
  double* P = at<double>(ws, L.panel_out);
  const double one = 1.0, zero = 0.0;
  BLAS_TRY(rocblas_set_stream(h->blas, s));
  BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
  for (int64_t r0 = 0; r0 < h->nd; r0 += p.rows) {
    const int64_t r = std::min(p.rows, h->nd - r0);
    HIP_TRY(launch_widen_rows(X + r0, h->nd, r, ns, W, p.rows, s));
    BLAS_TRY(rocblas_dgemm(h->blas, rocblas_operation_none, rocblas_operation_none, (rocblas_int)r, ns, ns, &one, W,
                           (rocblas_int)p.rows, Z, ns, &zero, P, (rocblas_int)p.rows));
    HIP_TRY(launch_narrow_rows(P, p.rows, r, ns, O + r0, h->nd, s));
  }
  ps.done();
}

// The 256 x (128 + 128) units of the split-bf16 products run one block per CU; where they
// leave more of the chip idle, or form more lower-triangle waste, than this allows, the
// 128 x 128 tiles (two blocks per CU) are taken.  Both products measured, tiles / units, by
// that share: 0.85 (60x60x180, Ns 1200) 11.95 / 6.83 ms; 0.68 (60^3, Ns 900) 2.30 / 1.73;
// 0.67 (72^3, Ns 600) 1.94 / 1.62, (64^3, Ns 520) 1.27 / 1.22; 0.666 (60^3, Ns 400) 0.66 / 0.71;
// 0.41 (60^3, Ns 257) 0.59 / 0.68; 0.09 (45^3, Ns 187) 0.21 / 0.58.  Many sizes lie close to the
// line (whole rounds of six or twelve units: 0.665 to 0.674), where the share does not order
// them; it is a safe side, not a fit: of 105 projections (45^3 to 90^3, Ns 200 to 800) the 44 above
// it take 0.675 to 1.006 of the tiles' time, 0.669 (72^3, Ns 500) 0.857.
constexpr double kPairMinFill = 0.668;

// Hs = X^T Y, Ms = X^T X (full symmetric, FP64), via split-K partial tiles.
template <typename TX, typename TY>
void gram_pair(chefsi_handle* h, const TX* X, const TY* Y, int ns, const WsLayout& L, void* ws, double* Hs,
               double* Ms, hipStream_t s, Gemm g) {
  if constexpr (std::is_same<TX, double>::value && std::is_same<TY, double>::value) {
    if (h->precision == CHEFSI_FP64) {
      if (blas_gram_faster(h->nd, ns)) {
        blas_gram(h, X, Y, ns, L, ws, Hs, s);
        blas_gram(h, X, X, ns, L, ws, Ms, s);
        return;
      }
      ProfScope ps(h, P_GRAM, s);
      HIP_TRY(launch_gram_both(X, Y, h->nd, ns, L.both, at<double>(ws, L.partial), Hs, Ms, s));
      ps.done();
      return;
    }
  }
  double* part = at<double>(ws, L.partial);
  if constexpr (std::is_same<TX, float>::value && std::is_same<TY, float>::value) {
    if (g == Gemm::BF16X3 && L.pair.fill >= kPairMinFill) {
      ProfScope ps(h, P_GRAM, s);
      HIP_TRY(launch_gram_pair_bf16x3(X, Y, h->nd, ns, L.pair, part, Hs, Ms, s));
      ps.done();
      return;
    }
  }
  {
    ProfScope ps(h, P_GRAM, s);
    HIP_TRY((gram_launch<TX, TY>(g, X, Y, h->nd, ns, L.gram, part, s)));
    ps.done();
  }
  {
    ProfScope ps(h, P_REDUCE, s);
    HIP_TRY(launch_gram_reduce(part, L.gram, ns, Hs, s));
    ps.done();
  }
  {
    ProfScope ps(h, P_GRAM, s);
    HIP_TRY((gram_launch<TX, TX>(g, X, X, h->nd, ns, L.gram, part, s)));
    ps.done();
  }
  {
    ProfScope ps(h, P_REDUCE, s);
    HIP_TRY(launch_gram_reduce(part, L.gram, ns, Ms, s));
    ps.done();
  }
}

// Hs Z = Ms Z D in FP64 on the device (Alg. 1, Diagonalization; Sec. 2.3), as the standard
// reduction of a symmetric-definite pencil after a diagonal scaling S (S_ii = Ms_ii^-1/2):
// S Ms S = U^T U (Cholesky), C = U^-T S Hs S U^-1, C = W D W^T (divide and conquer),
// Z = S U^-1 W.  Z overwrites Hs, U overwrites Ms.  info[0] receives the Cholesky
// status, info[1] the eigensolver status.
// First half: scaling and Cholesky (info[0]); second half: reduction, eigensolve,
// back substitution and back scaling (info[1]).
void dense_factor(chefsi_handle* h, double* Hs, double* Ms, int ns, const WsLayout& L, void* ws, hipStream_t s) {
  ProfScope ps(h, P_EIG, s);
  BLAS_TRY(rocblas_set_stream(h->blas, s));
  BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
  rocblas_int* info = at<rocblas_int>(ws, L.info);
  double* sc = at<double>(ws, L.sc);
  HIP_TRY(launch_pencil_scale(Hs, Ms, sc, ns, s));
  // (rocSOLVER and rocBLAS above the sizes whose right-hand sides fit in LDS)
  if (ns <= kCholMax)
    HIP_TRY(launch_cholesky(Ms, ns, at<void>(ws, L.chol), info, s));
  else
    BLAS_TRY(rocsolver_dpotrf(h->blas, rocblas_fill_upper, ns, Ms, ns, info));
  ps.done();
}

void dense_solve(chefsi_handle* h, double* Hs, double* Ms, double* D, int ns, const WsLayout& L, void* ws,
                 hipStream_t s) {
  ProfScope ps(h, P_EIG, s);
  const double one = 1.0;
  BLAS_TRY(rocblas_set_stream(h->blas, s));
  BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
  rocblas_int* info = at<rocblas_int>(ws, L.info);
  double* sc = at<double>(ws, L.sc);
  if (ns <= kCholMax) {
    // the partial products are dead here (at least ns^2 doubles)
    HIP_TRY(launch_reduce_pencil(Ms, at<void>(ws, L.chol), ns, Hs, at<double>(ws, L.partial), info, s));
  } else {
    BLAS_TRY(rocblas_dtrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_transpose,
                           rocblas_diagonal_non_unit, ns, ns, &one, Ms, ns, Hs, ns));
    BLAS_TRY(rocblas_dtrsm(h->blas, rocblas_side_right, rocblas_fill_upper, rocblas_operation_none,
                           rocblas_diagonal_non_unit, ns, ns, &one, Ms, ns, Hs, ns));
  }
  double* W = Hs;  // eigenvectors of the reduced matrix
  if (own_tridiag(h, ns)) {
    // the partial products and the projector coefficients are dead here: eigenvectors of the
    // tridiagonal matrix and reflector factors go there (at least ns^2 and ns doubles)
    W = at<double>(ws, L.partial);
    double* tau = at<double>(ws, L.alpha);
    double* E = at<double>(ws, L.e);
    HIP_TRY(launch_tridiag(Hs, ns, D, E, tau, at<void>(ws, L.msg), info + 2, s));
    BLAS_TRY(rocsolver_dstedc(h->blas, rocblas_evect_tridiagonal, ns, D, E, W, ns, info + 1));
    HIP_TRY(launch_backtransform(Hs, tau, ns, W, s));
  } else {
    BLAS_TRY(rocsolver_dsyevd(h->blas, rocblas_evect_original, rocblas_fill_upper, ns, Hs, ns, D,
                              at<double>(ws, L.e), info + 1));
  }
  if (ns <= kCholMax) {
    HIP_TRY(launch_back_substitute(Ms, at<void>(ws, L.chol), ns, W, Hs, sc, info, s));
  } else {
    BLAS_TRY(rocblas_dtrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_none,
                           rocblas_diagonal_non_unit, ns, ns, &one, Ms, ns, W, ns));
    HIP_TRY(launch_row_scale(W, Hs, sc, ns, s));
  }
  ps.done();
}

void dense_eig(chefsi_handle* h, double* Hs, double* Ms, double* D, int ns, const WsLayout& L, void* ws,
               hipStream_t s) {
  dense_factor(h, Hs, Ms, ns, L, ws, s);
  dense_solve(h, Hs, Ms, D, ns, L, ws, s);
}

// After dense_factor: true when the Cholesky failed or its smallest pivot U_ii^2 of the
// scaled overlap matrix is below kMixedMinPivot (host round trip; the diagonal of U goes
// through the eigensolver's scratch E, which is free until dense_solve).
bool factor_is_weak(chefsi_handle* h, const double* U, int ns, const WsLayout& L, void* ws, hipStream_t s) {
  double* diag = at<double>(ws, L.e);
  HIP_TRY(launch_copy_diag(U, diag, ns, s));
  double* d = h->pinned;
  rocblas_int* info = pinned_info(h);
  HIP_TRY(hipMemcpyAsync(d, diag, (size_t)ns * 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipMemcpyAsync(info, at<rocblas_int>(ws, L.info), sizeof(rocblas_int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (info[0] > 0) return true;
  double mn = 1.0;
  for (int i = 0; i < ns; ++i) mn = std::min(mn, d[i] * d[i]);
  return !(mn >= kMixedMinPivot);
}

// Map the two dense-stage status words to a status (the Cholesky failure is reported as
// ns + order of the failing leading minor, the convention of the LAPACK generalized solvers).
void raise_info(chefsi_handle* h, const rocblas_int* info, int ns) {
  if (info[0] > 0) {
    h->last_info = ns + info[0];
    throw Error{CHEFSI_ERR_NOT_POSDEF, "Cholesky of the overlap matrix failed (leading minor " +
                                           std::to_string(info[0]) + ")"};
  }
  if (info[1] > 0) {
    h->last_info = info[1];
    throw Error{CHEFSI_ERR_EIG, "dense eigensolver did not converge"};
  }
}

void check_info(chefsi_handle* h, void* ws, const WsLayout& L, int ns, hipStream_t s) {
  rocblas_int* info = pinned_info(h);
  HIP_TRY(hipMemcpyAsync(info, at<rocblas_int>(ws, L.info), 2 * sizeof(rocblas_int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  raise_info(h, info, ns);
}

template <typename T>
void copy_block(chefsi_handle* h, T* dst, const T* src, int ns, hipStream_t s) {
  ProfScope ps(h, P_COPY, s);
  HIP_TRY(hipMemcpyAsync(dst, src, (size_t)h->nd * ns * sizeof(T), hipMemcpyDeviceToDevice, s));
  ps.done();
}

template <typename T>
void rotate_into(chefsi_handle* h, const T* X, const double* Z, T* O, int ns, hipStream_t s, Gemm g, void* ws,
                 const WsLayout& L) {
  if constexpr (std::is_same<T, float>::value) {
    if (g == Gemm::F64) {
      panel_rotate(h, X, Z, O, ns, L, ws, s);
      return;
    }
  }
  ProfScope ps(h, P_ROT, s);
  if constexpr (std::is_same<T, float>::value) {
    if (g == Gemm::BF16X3) {
      HIP_TRY(launch_rotate_bf16x3(X, Z, at<void>(ws, L.zsplit), O, h->nd, ns, s));
      ps.done();
      return;
    }
  }
  if constexpr (std::is_same<T, double>::value) {
    // FP64 X Z is a plain GEMM (nd x ns times ns x ns, no fusion): rocBLAS's MFMA kernel for
    // it runs at a higher fraction of the FP64 peak than launch_rotate_f64.  Its 32-bit
    // dimensions bound it to blocks of fewer than 2^31 elements.
    if ((int64_t)h->nd * ns < ((int64_t)1 << 31)) {
      const double one = 1.0, zero = 0.0;
      BLAS_TRY(rocblas_set_stream(h->blas, s));
      BLAS_TRY(rocblas_set_workspace(h->blas, at<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
      BLAS_TRY(rocblas_dgemm(h->blas, rocblas_operation_none, rocblas_operation_none, (rocblas_int)h->nd, ns, ns,
                             &one, X, (rocblas_int)h->nd, Z, ns, &zero, O, (rocblas_int)h->nd));
      ps.done();
      return;
    }
  }
  HIP_TRY((launch_rotate_f64<T, T>(X, Z, O, h->nd, ns, s)));
  ps.done();
}

// The dense-product arithmetic of a handle's own steps.
Gemm step_gemm(const chefsi_handle* h) { return h->precision == CHEFSI_MIXED ? Gemm::BF16X3 : Gemm::F64; }

void ritz_to_host(chefsi_handle* h, const double* D, int ns, double* ritz_host, void* ws, const WsLayout& L,
                  hipStream_t s) {
  double* d = h->pinned;
  rocblas_int* info = pinned_info(h);
  HIP_TRY(hipMemcpyAsync(d, D, (size_t)ns * 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipMemcpyAsync(info, at<rocblas_int>(ws, L.info), 2 * sizeof(rocblas_int), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  raise_info(h, info, ns);
  for (int i = 0; i < ns; ++i)
    if (!std::isfinite(d[i])) throw Error{CHEFSI_ERR_NONFINITE, "non-finite Ritz value"};
  if (ritz_host) std::memcpy(ritz_host, d, (size_t)ns * 8);
}

// One CheFSI step (Alg. 1) for element type T (double: FP64 handle, float: mixed handle).
template <typename T>
void step_impl(chefsi_handle* h, T* X, int ns, int m, double lo, double cut, double hi, void* ws,
               const WsLayout& L, hipStream_t s, double* ritz_host) {
  T* A = X;
  T* B = at<T>(ws, L.bufB);
  T* alpha = at<T>(ws, L.alpha);
  double* Hs = at<double>(ws, L.hs);
  double* Ms = at<double>(ws, L.ms);
  double* D = at<double>(ws, L.d);
  const BandScratch bs = band_scratch(h, ws, L);
  T* Xf = run_filter<T>(h, A, B, ns, m, lo, cut, hi, alpha, s, bs, true);
  T* Yf = Xf == A ? B : A;
  apply_fused<T, T, T>(h, Xf, nullptr, Yf, ns, 1.0, 0.0, 0.0, alpha, s, bs, true, false, true);  // Y~ = H X~
  Gemm g = step_gemm(h);
  gram_pair<T, T>(h, Xf, Yf, ns, L, ws, Hs, Ms, s, g);
  dense_factor(h, Hs, Ms, ns, L, ws, s);
  if (g == Gemm::BF16X3 && factor_is_weak(h, Ms, ns, L, ws, s)) {
    // the filtered block is too ill-conditioned for split-bf16 products: FP64 this step
    g = Gemm::F64;
    h->prof_n[P_FALLBACK] += 1;
    gram_pair<T, T>(h, Xf, Yf, ns, L, ws, Hs, Ms, s, g);
    dense_factor(h, Hs, Ms, ns, L, ws, s);
  }
  dense_solve(h, Hs, Ms, D, ns, L, ws, s);
  rotate_into<T>(h, Xf, Hs, Yf, ns, s, g, ws, L);  // Y~ is dead: X = X~ Z~ goes there
  if (Yf != X) copy_block<T>(h, X, Yf, ns, s);
  ritz_to_host(h, D, ns, ritz_host, ws, L, s);
}

// Optional filter of degree m (storage precision), then a Rayleigh-Ritz pass with FP64
// arithmetic whatever the storage type: H X in FP64 from the stored block, FP64 Gram
// products, the FP64 dense stage and an FP64 rotation rounded once to the storage type.
template <typename T>
void refine_impl(chefsi_handle* h, T* X, int ns, int m, double lo, double cut, double hi, void* ws,
                 const WsLayout& L, hipStream_t s, double* ritz_host) {
  if (m > 0) {
    T* r = run_filter<T>(h, X, at<T>(ws, L.bufB), ns, m, lo, cut, hi, at<T>(ws, L.alpha), s,
                       band_scratch(h, ws, L));
    if (r != X) copy_block<T>(h, X, r, ns, s);
  }
  double* HX = at<double>(ws, L.bufB);  // Nd x ns FP64
  double* alpha = at<double>(ws, L.alpha);
  double* Hs = at<double>(ws, L.hs);
  double* Ms = at<double>(ws, L.ms);
  double* D = at<double>(ws, L.d);
  apply_fused<T, double, double>(h, X, nullptr, HX, ns, 1.0, 0.0, 0.0, alpha, s, band_scratch(h, ws, L));
  T* B = at<T>(ws, L.bufB);
  if constexpr (std::is_same<T, float>::value) {
    panel_gram(h, X, HX, ns, L, ws, Hs, Ms, s);
    dense_eig(h, Hs, Ms, D, ns, L, ws, s);
    panel_rotate(h, X, Hs, B, ns, L, ws, s);
  } else {
    gram_pair<T, double>(h, X, HX, ns, L, ws, Hs, Ms, s, Gemm::F64);
    dense_eig(h, Hs, Ms, D, ns, L, ws, s);
    rotate_into<T>(h, X, Hs, B, ns, s, Gemm::F64, ws, L);
  }
  copy_block<T>(h, X, B, ns, s);
  ritz_to_host(h, D, ns, ritz_host, ws, L, s);
}

int fail(chefsi_handle* h, const Error& e) {
  if (h) h->last_error = e.msg;
  return e.status;
}

template <typename F>
int guarded(chefsi_handle* h, F&& f) {
  if (h == nullptr) return CHEFSI_ERR_INVALID_ARG;
  try {
    h->last_error.clear();
    h->last_info = 0;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != h->device) HIP_TRY(hipSetDevice(h->device));
    f();
    return CHEFSI_OK;
  } catch (const Error& e) {
    return fail(h, e);
  } catch (const std::bad_alloc&) {
    return fail(h, Error{CHEFSI_ERR_OOM, "host allocation failed"});
  } catch (...) {
    return fail(h, Error{CHEFSI_ERR_HIP, "unexpected exception"});
  }
}

template <typename T>
T* upload(chefsi_handle* h, const T* src, size_t n) {
  T* d = nullptr;
  if (n == 0) return nullptr;
  if (no_memory(hipMalloc(&d, n * sizeof(T)))) throw Error{CHEFSI_ERR_OOM, "device allocation failed"};
  h->device_bytes += n * sizeof(T);
  hipError_t e = hipMemcpy(d, src, n * sizeof(T), hipMemcpyHostToDevice);
  if (no_memory(e)) {
    (void)hipFree(d);
    h->device_bytes -= n * sizeof(T);
    throw Error{CHEFSI_ERR_HIP, std::string("upload: ") + hipGetErrorString(e)};
  }
  return d;
}

// Stencil-pass projector records for tiling hp (points in one to four projector entries,
// grouped by (y tile, z plane); at most ty * nx per group <= PY * threads), replacing the
// handle's current ones.  The LDS budget (the alpha row and the partial-sum buffers
// beside the tile) is checked for the longest z chunk (zc = nz), which the planner picks
// for wide blocks; with no records (band route) the pass carries neither.
static bool hx_records_fit(const chefsi_handle* h, const HxPlan& hp) {
  HxPlan worst = hp;
  worst.zc = h->n[2];
  const int nx = h->n[0];
  const size_t lds_need = std::max(hx_lds_bytes(worst, nx, h->radius, h->precision == CHEFSI_FP64 ? 8 : 4,
                                                h->np_tot, 8),
                                   hx_lds_bytes(worst, nx, h->radius, 4, h->np_tot, 8));
  return lds_need <= kHxMaxLds;
}

void build_hx_records(chefsi_handle* h, const HxPlan& hp) {
  const int nx = h->n[0], ny = h->n[1], nz = h->n[2];
  const int64_t nd = h->nd;
  check(h->rec_max == 0 || hx_records_fit(h, hp),
        "too many projectors for the stencil pass (alpha row does not fit in LDS)");
  const bool f32 = h->precision == CHEFSI_MIXED;
  const int planes = h->rec_max > 0 ? nz : 0;  // the band pass takes every term: no records
  const int64_t nkeys = (int64_t)hp.nty * planes;
  const std::vector<int>& cnt = h->pt_cnt;
  std::vector<int> rptr(nkeys + 1, 0);
  for (int z = 0; z < planes; ++z)
    for (int y = 0; y < ny; ++y) {
      const int* c = cnt.data() + ((int64_t)z * ny + y) * nx;
      int& count = rptr[(int64_t)(y / hp.ty) * nz + z + 1];
      for (int x = 0; x < nx; ++x) {
        const int n = c[x + 1] - c[x];
        count += n >= 1 && n <= h->rec_max;
      }
    }
  for (int64_t k = 0; k < nkeys; ++k) rptr[k + 1] += rptr[k];
  const int nrec = rptr[nkeys];
  std::unique_ptr<HxRec<double>[]> r64(new HxRec<double>[std::max(nrec, 1)]);
  std::unique_ptr<HxRec<float>[]> r32(f32 ? new HxRec<float>[std::max(nrec, 1)] : nullptr);
  std::vector<int> rfill(rptr.begin(), rptr.end() - 1);
  for (int z = 0; z < planes; ++z)
    for (int y = 0; y < ny; ++y) {
      const int* c = cnt.data() + ((int64_t)z * ny + y) * nx;
      int& r = rfill[(int64_t)(y / hp.ty) * nz + z];
      for (int x = 0; x < nx; ++x) {
        const int b = c[x], n = c[x + 1] - b;
        if (n < 1 || n > h->rec_max) continue;
        HxRec<double> rec{};
        int col[4] = {0, 0, 0, 0};
        for (int k = 0; k < n; ++k) {
          col[k] = h->pt_col[b + k];
          rec.val[k] = h->pt_val[b + k];
        }
        rec.lidx = (y % hp.ty) * nx + x;
        rec.c01 = col[0] | (col[1] << 16);
        rec.c23 = col[2] | (col[3] << 16);
        r64[r] = rec;
        if (f32) {
          HxRec<float> half{};
          half.lidx = rec.lidx;
          half.c01 = rec.c01;
          half.c23 = rec.c23;
          for (int k = 0; k < n; ++k) half.val[k] = (float)rec.val[k];
          r32[r] = half;
        }
        ++r;
      }
    }
  int* nptr = nullptr;
  HxRec<double>* n64 = nullptr;
  HxRec<float>* n32 = nullptr;
  const size_t before = h->device_bytes;
  try {
    if (nrec > 0) {
      nptr = upload(h, rptr.data(), rptr.size());
      n64 = upload(h, r64.get(), nrec);
      if (f32) n32 = upload(h, r32.get(), nrec);
    }
  } catch (...) {
    for (void* q : {(void*)nptr, (void*)n64, (void*)n32})
      if (q) (void)hipFree(q);
    h->device_bytes = before;
    throw;
  }
  for (void* q : {(void*)h->hx_rec_ptr, (void*)h->hx_rec64, (void*)h->hx_rec32})
    if (q) (void)hipFree(q);
  h->device_bytes -= h->hx_rec_bytes;
  h->hx_rec_bytes = nrec > 0 ? rptr.size() * sizeof(int) +
                                   (size_t)nrec * (sizeof(HxRec<double>) + (f32 ? sizeof(HxRec<float>) : 0))
                             : 0;
  h->hx_rec_ptr = nptr;
  h->hx_rec64 = n64;
  h->hx_rec32 = n32;
  h->n_hxrec = nrec;
  h->hx_plan = hp;
}

void free_band(const BandDevice& b) {
  void* ptrs[] = {b.nb_reg_pt,   b.nb_pt_idx,     b.nb_pt_ent,     b.nb_ent_ls,   b.nb_ent_chi64,
                  b.nb_ent_chi32, b.nb_reg_slot,  b.nb_slot_ent,   b.nb_gent_loc, b.nb_gent_chi64,
                  b.nb_gent_chi32, b.nb_q_slot_ptr, b.nb_q_slot,   b.nb_partial, b.nb_slot_q};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
}

void free_band_tables(chefsi_handle* h) {
  free_band(*h);
  h->device_bytes -= h->nb_bytes;
  static_cast<BandDevice&>(*h) = BandDevice();
}

// Band-pass regions from a point-major projector table (cnt: nd + 1 entry offsets, col: the
// projector column of every entry): regions of consecutive touched points (grid index
// order), each closed before it would exceed max_pts points, kBandMaxSlots projectors or
// max_ent entries; each region lists its points with their entries, and its projector slots
// (projector order) with their entries (point order); each projector lists its slots (region
// order) for the reduction.  The scatter entries are the table's, in its order; gent_src names the
// table entry behind every gather entry, so the caller attaches values of its own type.
struct BandRegions {
  std::vector<int> reg_pt{0}, pt_idx, pt_ent{0}, ent_ls, reg_slot{0}, slot_q, slot_ent{0}, gent_loc, q_slot_ptr{0},
      q_slot, gent_src;
};

BandRegions band_regions(int64_t nd, const int* cnt, const int* col, int np_tot, int max_pts, int max_ent) {
  BandRegions R;
  const size_t nent = (size_t)cnt[nd];
  for (std::vector<int>* v : {&R.pt_idx, &R.pt_ent}) v->reserve(nent / 4 + 16);
  for (std::vector<int>* v : {&R.ent_ls, &R.gent_loc, &R.gent_src}) v->reserve(nent);
  std::vector<int> stamp(np_tot, -1), local(np_tot, 0);  // region that last counted a projector, its slot there
  std::vector<int> cols, fill;                           // the open region's projectors
  int64_t first_pt = 0;                                  // places of the open region's first point and entry
  int first_ent = 0;
  int nreg = 0;
  auto close_region = [&]() {
    std::sort(cols.begin(), cols.end());  // slots in projector order
    const int ns = (int)cols.size(), base = (int)R.gent_loc.size();
    for (int i = 0; i < ns; ++i) local[cols[i]] = i;
    fill.assign(ns + 1, 0);
    for (int e = first_ent; e < R.pt_ent.back(); ++e) {
      const int ls = local[col[e]];
      R.ent_ls.push_back(ls);
      ++fill[ls + 1];
    }
    for (int i = 0; i < ns; ++i) {
      fill[i + 1] += fill[i];
      R.slot_q.push_back(cols[i]);
      R.slot_ent.push_back(base + fill[i + 1]);
    }
    R.gent_loc.resize(R.pt_ent.back());
    R.gent_src.resize(R.pt_ent.back());
    for (int64_t p = first_pt; p < (int64_t)R.pt_idx.size(); ++p)  // each slot's entries in point order
      for (int e = R.pt_ent[p]; e < R.pt_ent[p + 1]; ++e) {
        const int g = base + fill[R.ent_ls[e]]++;
        R.gent_loc[g] = (int)(p - first_pt);
        R.gent_src[g] = e;
      }
    R.reg_pt.push_back((int)R.pt_idx.size());
    R.reg_slot.push_back((int)R.slot_q.size());
    cols.clear();
    first_pt = (int64_t)R.pt_idx.size();
    first_ent = R.pt_ent.back();
    ++nreg;
  };
  for (int64_t i = 0; i < nd; ++i) {
    const int n = cnt[i + 1] - cnt[i];
    if (n == 0) continue;
    check(n <= kBandMaxSlots && n <= max_ent, "a grid point lies in too many projector supports for the band pass");
    int fresh = 0;
    for (int e = cnt[i]; e < cnt[i + 1]; ++e) fresh += stamp[col[e]] != nreg;
    const int64_t open_pts = (int64_t)R.pt_idx.size() - first_pt;
    if (open_pts > 0 && (open_pts + 1 > max_pts || cnt[i] - first_ent + n > max_ent ||
                         (int)cols.size() + fresh > kBandMaxSlots))
      close_region();
    for (int e = cnt[i]; e < cnt[i + 1]; ++e) {
      if (stamp[col[e]] != nreg) {
        stamp[col[e]] = nreg;
        cols.push_back(col[e]);
      }
    }
    R.pt_idx.push_back((int)i);
    R.pt_ent.push_back(cnt[i + 1]);
  }
  if ((int64_t)R.pt_idx.size() > first_pt) close_region();
  // each projector's slots in region order
  R.q_slot_ptr.assign(np_tot + 1, 0);
  for (int q : R.slot_q) ++R.q_slot_ptr[q + 1];
  for (int q = 0; q < np_tot; ++q) R.q_slot_ptr[q + 1] += R.q_slot_ptr[q];
  R.q_slot.resize(R.slot_q.size());
  std::vector<int> at(R.q_slot_ptr.begin(), R.q_slot_ptr.end() - 1);
  for (size_t sl = 0; sl < R.slot_q.size(); ++sl) R.q_slot[at[R.slot_q[sl]]++] = (int)sl;
  return R;
}

// Band-pass tables of a real handle (host): the regions and the projector values of their gather
// entries (the scatter entries' are the table's), in FP32 for mixed handles and in FP64 unless the
// band pass runs only in the filter of a mixed handle.
struct BandTables {
  BandRegions r;
  bool f64 = false;
  std::vector<double> gent_chi;
  std::vector<float> ent_chi32, gent_chi32;
};

BandTables band_tables(const chefsi_handle* h, bool filter_only) {
  BandTables t;
  t.r = band_regions(h->nd, h->pt_cnt.data(), h->pt_col.data(), h->np_tot, kBandMaxPts, kBandMaxEnt);
  t.f64 = !filter_only;
  auto gather_values = [&](auto& v) {
    v.resize(t.r.gent_src.size());
    for (size_t e = 0; e < v.size(); ++e) v[e] = h->pt_val[t.r.gent_src[e]];
  };
  if (t.f64) gather_values(t.gent_chi);
  if (h->precision == CHEFSI_MIXED) {
    t.ent_chi32.assign(h->pt_val.begin(), h->pt_val.end());
    gather_values(t.gent_chi32);
  }
  return t;
}

// The handle's current tables are replaced, or kept where the new ones cannot be built.
void build_band_tables(chefsi_handle* h, const BandTables& t) {
  const BandRegions& R = t.r;
  const size_t before = h->device_bytes;
  const BandDevice old = *h;
  static_cast<BandDevice&>(*h) = BandDevice();
  try {
    h->nb_reg_pt = upload(h, R.reg_pt.data(), R.reg_pt.size());
    h->nb_pt_idx = upload(h, R.pt_idx.data(), R.pt_idx.size());
    h->nb_pt_ent = upload(h, R.pt_ent.data(), R.pt_ent.size());
    h->nb_ent_ls = upload(h, R.ent_ls.data(), R.ent_ls.size());
    h->nb_slot_q = upload(h, R.slot_q.data(), R.slot_q.size());
    h->nb_reg_slot = upload(h, R.reg_slot.data(), R.reg_slot.size());
    h->nb_slot_ent = upload(h, R.slot_ent.data(), R.slot_ent.size());
    h->nb_gent_loc = upload(h, R.gent_loc.data(), R.gent_loc.size());
    h->nb_q_slot_ptr = upload(h, R.q_slot_ptr.data(), R.q_slot_ptr.size());
    h->nb_q_slot = upload(h, R.q_slot.data(), R.q_slot.size());
    if (t.f64) h->nb_ent_chi64 = upload(h, h->pt_val.data(), h->pt_val.size());
    h->nb_gent_chi64 = upload(h, t.gent_chi.data(), t.gent_chi.size());
    h->nb_ent_chi32 = upload(h, t.ent_chi32.data(), t.ent_chi32.size());
    h->nb_gent_chi32 = upload(h, t.gent_chi32.data(), t.gent_chi32.size());
    const int own_ns = h->ws_band_slots > 0 ? std::min<int>(h->max_ns, kBandMinOrbitals) : h->max_ns;
    const size_t pbytes = band_partial_bytes(h, (int)R.slot_q.size(), own_ns);
    if (no_memory(hipMalloc(&h->nb_partial, pbytes))) {
      h->nb_partial = nullptr;
      throw Error{CHEFSI_ERR_OOM, "device allocation failed (band-pass partial sums)"};
    }
    h->nb_partial_bytes = pbytes;
    h->device_bytes += pbytes;
  } catch (...) {
    free_band(*h);
    static_cast<BandDevice&>(*h) = old;
    h->device_bytes = before;
    throw;
  }
  free_band(old);
  h->nb_bytes = h->device_bytes - before;
  h->device_bytes -= old.nb_bytes;
  h->nb_reg = (int)R.reg_pt.size() - 1;
  h->nb_pts = (int)R.pt_idx.size();
  h->nb_slots = (int)R.slot_q.size();
}

// From how many orbitals on a call takes the band pass (kNoBand: never): single applications of
// H, and filters, on a handle as created.
//
// The band pass costs launches and passes over the touched points; it leaves the stencil pass
// bare, spares the scatter pass over the points in more than four entries that the records leave
// where supports overlap, and in a filter the gather of the coefficients.  So it pays from a number
// of values (points x orbitals) on, sooner the more such points there are, and without any only
// where few points are touched.  Band pass / records, one H X (FP64) or a filter application:
//   512 and more such points: four orbitals 30x33x28 1.00, 45^3 slab 0.99, 64^3 1.07 (16: 0.78),
//     60x60x180 0.96; 120^3 8 orbitals 1.09, 16 1.04, 24 0.96; below eight orbitals and 2^18 values
//     in the widest call the tables are not built.  Mixed filters from any such point on: four
//     orbitals 0.76 to 1.05, eight 0.65 to 0.92.
//   fewer in FP64: 2^21 values 0.99 to 1.05, 2^22 0.80 to 1.0.
//   none, at most a fifth touched: 2^22 values 1.1 to 1.4, 2^23 0.94 to 1.07, 2^24 0.81 to 0.95;
//     mixed filters 1.02 to 1.1, 0.93 to 1.0, 0.87.
//   none, more touched: one H X 1.05 to 1.15 up to 600 orbitals (72^3, 31 %; on rows of 96 points
//     and more, where the records cost more, 0.9 with up to a third), FP64 filters 0.97 to 1.02
//     from 2^23 and 0.95 from 2^26 values on, mixed ones 1.0 to 1.1 up to 2^26 and 0.94 to 0.98 from
//     2^27 on.
// Grids of 2^14 to 2^15 points without 512 such points take it from 2^20 values of the widest call
// on although the records are faster there (27x30x26, one atom, 60 orbitals 1.4): the tests hold
// these handles to the bits of that route.
// A mixed handle keeps the records for single applications: they add the projector term before
// the result is rounded to FP32, where the band pass rounds the touched points a second time (in a
// filter, too; there the result is FP32 at every step, while chefsi_project forms FP64 matrices).
struct BandFrom {
  int apply, filter;
};

BandFrom band_from(const chefsi_handle* h) {
  const int64_t nd = h->nd, widest = nd * h->max_ns;
  const bool mixed = h->precision == CHEFSI_MIXED;
  int64_t touched = 0, scattered = 0;
  for (int64_t i = 0; i < nd; ++i) {
    const int n = h->pt_cnt[i + 1] - h->pt_cnt[i];
    touched += n > 0;
    scattered += n > 4;
  }
  auto from = [&](int64_t values) { return (int)std::min<int64_t>(kNoBand, std::max<int64_t>(8, (values + nd - 1) / nd)); };
  const int few = nd >= (int64_t)1 << 20 ? 16 : 4;
  BandFrom b{kNoBand, kNoBand};
  if (scattered >= 512 || (mixed && scattered > 0)) {
    if (mixed ? h->max_ns >= 4 : h->max_ns >= 8 && widest >= (int64_t)1 << 18) b = {few, few};
  } else if (nd >= (int64_t)1 << 14 && nd < (int64_t)1 << 15) {
    if (h->max_ns >= 8 && widest >= (int64_t)1 << 20) b = {few, few};
  } else if (scattered > 0) {
    b.apply = b.filter = from((int64_t)3 << 20);
  } else {
    const bool sparse = touched * (h->n[0] >= 96 ? 3 : 5) <= nd;
    if (sparse) b.apply = from((int64_t)1 << 23);
    b.filter = from((int64_t)1 << (sparse || (!mixed && 3 * touched <= nd) ? 23 : 27));
  }
  if (mixed) b.apply = kNoBand;
  return b;
}

// Scatter-pass records for the points in more than rec_max projector entries (all touched
// points when rec_max is 0): one record {point, first entry, entry count, 0} each, entries
// in atom order padded with zeros to a multiple of 4; replaces the handle's current ones.
void build_scatter_records(chefsi_handle* h) {
  std::vector<int4> recs;
  const bool band = h->rec_max == 0;  // the band pass takes every term: no scatter records
  std::vector<int> ecol;
  std::vector<double> evals;
  for (int64_t i = 0; i < h->nd; ++i) {
    const int b = h->pt_cnt[i], n = h->pt_cnt[i + 1] - b;
    if (band || n <= h->rec_max) continue;
    recs.push_back(make_int4((int)i, (int)ecol.size(), n, 0));
    for (int k = b; k < b + n; ++k) {
      ecol.push_back(h->pt_col[k]);
      evals.push_back(h->pt_val[k]);
    }
    while (ecol.size() % 4) {
      ecol.push_back(0);
      evals.push_back(0.0);
    }
  }
  check(ecol.size() < ((size_t)1 << 31), "too many projector entries");
  int4* rec = nullptr;
  int* col = nullptr;
  double* v64 = nullptr;
  float* v32 = nullptr;
  const size_t before = h->device_bytes;
  try {
    if (!recs.empty()) {
      rec = upload(h, recs.data(), recs.size());
      col = upload(h, ecol.data(), ecol.size());
      v64 = upload(h, evals.data(), evals.size());
      std::vector<float> ev32(evals.begin(), evals.end());
      v32 = upload(h, ev32.data(), ev32.size());
    }
  } catch (...) {
    for (void* q : {(void*)rec, (void*)col, (void*)v64, (void*)v32})
      if (q) (void)hipFree(q);
    h->device_bytes = before;
    throw;
  }
  for (void* q : {(void*)h->rec, (void*)h->ent_col, (void*)h->ent_val64, (void*)h->ent_val32})
    if (q) (void)hipFree(q);
  h->device_bytes -= h->scatter_bytes;
  h->scatter_bytes = recs.empty() ? 0
                                  : recs.size() * sizeof(int4) + ecol.size() * (sizeof(int) + sizeof(double) +
                                                                                sizeof(float));
  h->rec = rec;
  h->ent_col = col;
  h->ent_val64 = v64;
  h->ent_val32 = v32;
  h->n_pts = (int)recs.size();
}

// The box of every atom's support (first grid index and length in each direction; the shortest
// wrapped interval in a periodic one), or nothing when an atom's points or its box, longer by
// r at both ends of a direction, exceed what the force kernel keeps in registers and LDS.
std::vector<int> support_boxes(const chefsi_handle* h) {
  std::vector<int> box(6 * (size_t)h->n_atoms, 0);
  std::vector<char> seen[3];
  for (int J = 0; J < h->n_atoms; ++J) {
    const int64_t s0 = h->supp_ptr_h[J], s1 = h->supp_ptr_h[J + 1];
    if (s1 - s0 > kGradBoxPoints) return {};
    int* b = box.data() + 6 * (size_t)J;
    for (int d = 0; d < 3; ++d) seen[d].assign(h->n[d], 0);
    int64_t row = 0, row_end = 0;  // grid row of the last point (support indices increase)
    for (int64_t s = s0; s < s1; ++s) {
      const int64_t i = h->supp_idx_h[s];
      if (i >= row_end) {
        row = i / h->n[0];
        row_end = (row + 1) * h->n[0];
        seen[1][row % h->n[1]] = 1;
        seen[2][row / h->n[1]] = 1;
      }
      seen[0][i - row * h->n[0]] = 1;
    }
    for (int d = 0; d < 3; ++d) {
      const int n = h->n[d];
      int first = 0, last = n - 1;
      while (first < n && !seen[d][first]) ++first;
      if (first == n) {  // no points
        b[d] = 0;
        b[3 + d] = 1;
        continue;
      }
      while (!seen[d][last]) --last;
      b[d] = first;
      b[3 + d] = last - first + 1;
      if (h->bc[d] == 0) {  // the longest run of unseen points between two seen ones, if longer
        for (int i = first, gap = 0; i <= last; ++i) {
          gap = seen[d][i] ? 0 : gap + 1;
          if (gap > 0 && n - gap < b[3 + d]) {
            b[d] = i + 1;
            b[3 + d] = n - gap;
          }
        }
      }
    }
    for (int d = 0; d < 3; ++d) {
      int64_t v = 1;
      for (int e = 0; e < 3; ++e) v *= b[3 + e] + (e == d ? 2 * h->radius : 0);
      if (v > kGradBoxValues) return {};
    }
  }
  return box;
}

void release(chefsi_handle* h) {
  free_band_tables(h);
  void* ptrs[] = {h->veff64, h->veff32, h->supp_off, h->supp_idx, h->chi_off,  h->nproj,    h->poff,     h->supp_box,
                  h->chi64,  h->chi32,  h->gdv64,    h->gdv32,    h->rec,      h->ent_col,  h->hx_rec_ptr,
                  h->hx_rec64, h->hx_rec32,
                  h->ent_val64,
                  h->ent_val32};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  for (auto& p : h->ev_pending) {
    (void)hipEventDestroy(p.b);
    (void)hipEventDestroy(p.e);
  }
  for (auto ev : h->ev_pool) (void)hipEventDestroy(ev);
  if (h->pinned) (void)hipHostFree(h->pinned);
  if (h->blas) rocblas_destroy_handle(h->blas);
}

}  // namespace

extern "C" {

int chefsi_version(void) { return 100; }

const char* chefsi_strerror(int status) {
  switch (status) {
    case CHEFSI_OK: return "ok";
    case CHEFSI_ERR_INVALID_ARG: return "invalid argument";
    case CHEFSI_ERR_HIP: return "HIP runtime error";
    case CHEFSI_ERR_WORKSPACE: return "workspace too small";
    case CHEFSI_ERR_NOT_POSDEF: return "overlap matrix not positive definite";
    case CHEFSI_ERR_EIG: return "dense eigensolver did not converge";
    case CHEFSI_ERR_NONFINITE: return "non-finite Ritz value";
    case CHEFSI_ERR_SOLVER: return "rocBLAS/rocSOLVER error";
    case CHEFSI_ERR_OOM: return "out of memory";
    default: return "unknown status";
  }
}

const char* chefsi_last_error(const chefsi_handle_t* h) { return h ? h->last_error.c_str() : ""; }

int chefsi_last_info(const chefsi_handle_t* h) { return h ? h->last_info : 0; }

int chefsi_update_veff(chefsi_handle_t* h, const double* veff_host, void* stream) {
  return guarded(h, [&] {
    check(veff_host != nullptr, "veff_host is NULL");
    for (int64_t i = 0; i < h->nd; ++i) check(std::isfinite(veff_host[i]), "Veff must be finite");
    hipStream_t s = (hipStream_t)stream;
    h->veff_h.assign(veff_host, veff_host + h->nd);
    const std::vector<float> v32(h->veff_h.begin(), h->veff_h.end());
    HIP_TRY(hipMemcpyAsync(h->veff64, h->veff_h.data(), (size_t)h->nd * sizeof(double), hipMemcpyHostToDevice, s));
    HIP_TRY(hipMemcpyAsync(h->veff32, v32.data(), (size_t)h->nd * sizeof(float), hipMemcpyHostToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));  // v32 and the caller's array may go away after return
  });
}

int chefsi_create(const chefsi_grid_t* grid, const double* veff_host, const chefsi_nonlocal_t* nl,
                  int32_t precision, int32_t max_ns, chefsi_handle_t** out) {
  if (out == nullptr) return CHEFSI_ERR_INVALID_ARG;
  *out = nullptr;
  if (grid == nullptr || veff_host == nullptr) return CHEFSI_ERR_INVALID_ARG;
  chefsi_handle* h = nullptr;
  try {
    h = new chefsi_handle();
  } catch (...) {
    return CHEFSI_ERR_OOM;
  }
  try {
    check(precision == CHEFSI_FP64 || precision == CHEFSI_MIXED, "precision must be CHEFSI_FP64 or CHEFSI_MIXED");
    check(grid->fd_order >= 2 && grid->fd_order <= 12 && grid->fd_order % 2 == 0, "fd_order must be even, 2..12");
    h->precision = precision;
    h->order = grid->fd_order;
    h->radius = grid->fd_order / 2;
    int64_t nd = 1;
    for (int d = 0; d < 3; ++d) {
      check(grid->n[d] >= 1, "grid sizes must be >= 1");
      check(grid->bc[d] == 0 || grid->bc[d] == 1, "bc must be 0 (periodic) or 1 (Dirichlet)");
      check(std::isfinite(grid->h[d]) && grid->h[d] > 0.0, "grid spacing must be positive");
      if (grid->bc[d] == 0) check(grid->n[d] >= h->radius, "periodic direction needs n >= fd_order/2");
      h->n[d] = grid->n[d];
      h->h[d] = grid->h[d];
      h->bc[d] = grid->bc[d];
      nd *= grid->n[d];
    }
    check(nd < (int64_t)1 << 31, "Nd must be below 2^31");
    // the stencil pass addresses one orbital, Veff and the projector records (48 bytes per
    // point at most) through buffer resources of fewer than 2^31 bytes
    check(nd * 48 < (int64_t)1 << 31, "grids above 44 million points are not supported by the stencil pass");
    check(grid->n[0] <= kHxMaxThreads, "nx above 512 is not supported by the stencil tiling");
    check(max_ns >= 1 && (int64_t)max_ns <= nd, "max_ns must satisfy 1 <= max_ns <= Nd");
    for (int eb : {4, 8})
      check(plan_hx(grid->n[0], grid->n[1], grid->n[2], 1, grid->fd_order / 2, eb, 0, 0).ok,
            "grid too wide in x for the stencil tiling (the halo rows of a tile need at most four values per thread)");
    h->nd = nd;
    h->max_ns = max_ns;
    h->dv = grid->h[0] * grid->h[1] * grid->h[2];
    h->w = fd_weights(h->order);
    h->veff_h.assign(veff_host, veff_host + nd);
    for (double v : h->veff_h) check(std::isfinite(v), "Veff must be finite");

    // projectors
    if (nl != nullptr && nl->n_atoms > 0) {
      check(nl->supp_ptr && nl->supp_idx && nl->nproj && nl->chi && nl->gamma, "null projector array");
      const int na = nl->n_atoms;
      h->n_atoms = na;
      h->supp_ptr_h.assign(nl->supp_ptr, nl->supp_ptr + na + 1);
      check(h->supp_ptr_h[0] == 0, "supp_ptr[0] must be 0");
      for (int J = 0; J < na; ++J) check(h->supp_ptr_h[J + 1] >= h->supp_ptr_h[J], "supp_ptr must be non-decreasing");
      const int64_t nsupp = h->supp_ptr_h[na];
      check(nsupp < (int64_t)1 << 31, "too many support points");
      h->supp_idx_h.assign(nl->supp_idx, nl->supp_idx + nsupp);
      h->nproj_h.assign(nl->nproj, nl->nproj + na);
      int64_t nchi = 0, npt = 0;
      for (int J = 0; J < na; ++J) {
        check(h->nproj_h[J] >= 1, "nproj must be >= 1");
        const int64_t nj = h->supp_ptr_h[J + 1] - h->supp_ptr_h[J];
        for (int64_t s = 0; s < nj; ++s) {
          const int64_t i = h->supp_idx_h[h->supp_ptr_h[J] + s];
          check(i >= 0 && i < nd, "support index outside the grid");
          if (s > 0) check(i > h->supp_idx_h[h->supp_ptr_h[J] + s - 1], "support indices must increase");
        }
        nchi += nj * h->nproj_h[J];
        npt += h->nproj_h[J];
      }
      check(npt < (int64_t)1 << 30 && nchi < ((int64_t)1 << 40), "too many projectors");
      h->np_tot = (int)npt;
      h->chi_h.assign(nl->chi, nl->chi + nchi);
      h->gamma_h.assign(nl->gamma, nl->gamma + npt);
      for (double v : h->chi_h) check(std::isfinite(v), "chi must be finite");
      for (double v : h->gamma_h) check(std::isfinite(v), "gamma must be finite");
    }

    h->hx_plan = plan_hx(h->n[0], h->n[1], h->n[2], 1, h->radius, precision == CHEFSI_FP64 ? 8 : 4, 0, 0);
    check(h->hx_plan.ok, "no stencil tiling fits this grid");

    // point-major projector table, and the band pass's tables from it in a second thread
    const int na = h->n_atoms;
    std::vector<int> soff(na + 1), poff(na);
    std::vector<int64_t> coff(na);
    std::vector<double> gdv(h->np_tot);
    bool fits = true, both = false;
    BandFrom from{kNoBand, kNoBand};
    std::future<BandTables> tables;
    if (h->np_tot > 0) {
      int64_t c = 0;
      int p = 0;
      for (int J = 0; J < na; ++J) {
        soff[J] = (int)h->supp_ptr_h[J];
        coff[J] = c;
        poff[J] = p;
        c += (h->supp_ptr_h[J + 1] - h->supp_ptr_h[J]) * h->nproj_h[J];
        p += h->nproj_h[J];
      }
      soff[na] = (int)h->supp_ptr_h[na];
      for (int q = 0; q < h->np_tot; ++q) gdv[q] = h->gamma_h[q] * h->dv;
      // point i lists (projector column, chi value), atoms in order
      std::vector<int> cnt(nd + 1, 0);
      for (int J = 0; J < na; ++J)
        for (int64_t s = h->supp_ptr_h[J]; s < h->supp_ptr_h[J + 1]; ++s) cnt[h->supp_idx_h[s] + 1] += h->nproj_h[J];
      for (int64_t i = 0; i < nd; ++i) cnt[i + 1] += cnt[i];
      const int64_t nent = cnt[nd];
      check(nent < (int64_t)1 << 31, "too many projector entries");
      std::vector<int> fill(cnt.begin(), cnt.end() - 1), eproj(nent);
      std::vector<double> eval(nent);
      for (int J = 0; J < na; ++J) {
        const int64_t nj = h->supp_ptr_h[J + 1] - h->supp_ptr_h[J];
        for (int64_t s = 0; s < nj; ++s) {
          const int i = h->supp_idx_h[h->supp_ptr_h[J] + s];
          for (int a = 0; a < h->nproj_h[J]; ++a) {
            const int pos = fill[i]++;
            eproj[pos] = poff[J] + a;
            eval[pos] = h->chi_h[coff[J] + a * nj + s];
          }
        }
      }
      h->pt_cnt = std::move(cnt);
      h->pt_col = std::move(eproj);
      h->pt_val = std::move(eval);
      check(h->np_tot < 65536, "more than 65535 projectors");
      // The record route keeps the block's projector row and partial sums in LDS beside the tile: a
      // handle whose projectors overflow that for the default tile has the band pass alone.  Others
      // have the records, and the band pass beside them for the calls that it serves better.
      fits = hx_records_fit(h, h->hx_plan);
      from = band_from(h);
      both = fits && (from.apply <= max_ns || from.filter <= max_ns);
      if (both) tables = std::async([h] { return band_tables(h, h->precision == CHEFSI_MIXED); });
    }

    HIP_TRY(hipGetDevice(&h->device));
    HIP_TRY(hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, h->device));
    (void)scratch_address(h->device);  // the static scratch's device address, once per device
    BLAS_TRY(rocblas_create_handle(&h->blas));
    // the dense stage must give the same bits whatever else runs on the device (results of
    // a request alone and among others are compared bit for bit): no atomics in rocBLAS
    BLAS_TRY(rocblas_set_atomics_mode(h->blas, rocblas_atomics_not_allowed));
    const size_t pinned_doubles = std::max({(size_t)max_ns + 8, (size_t)h->n_atoms * 10, (size_t)kVecBlocks});
    if (no_memory(hipHostMalloc((void**)&h->pinned, pinned_doubles * sizeof(double), hipHostMallocDefault))) {
      h->pinned = nullptr;
      throw Error{CHEFSI_ERR_OOM, "pinned host allocation failed"};
    }
    h->veff64 = upload(h, h->veff_h.data(), nd);
    std::vector<float> v32(h->veff_h.begin(), h->veff_h.end());
    h->veff32 = upload(h, v32.data(), nd);

    if (h->np_tot > 0) {
      if (!fits) {
        try {
          const BandTables t = band_tables(h, false);
          h->ws_band_slots = std::max<int>(1, (int)t.r.slot_q.size());
          build_band_tables(h, t);
          h->rec_max = 0;
        } catch (const Error& e) {
          throw Error{e.status,
                      "too many projectors for the stencil pass (alpha row does not fit in LDS), and " + e.msg};
        }
      }
      build_hx_records(h, h->hx_plan);
      build_scatter_records(h);
      h->supp_off = upload(h, soff.data(), soff.size());
      h->supp_idx = upload(h, h->supp_idx_h.data(), h->supp_idx_h.size());
      h->chi_off = upload(h, coff.data(), coff.size());
      h->nproj = upload(h, h->nproj_h.data(), h->nproj_h.size());
      h->poff = upload(h, poff.data(), poff.size());
      const std::vector<int> box = support_boxes(h);
      if (!box.empty()) h->supp_box = upload(h, box.data(), box.size());
      h->chi64 = upload(h, h->chi_h.data(), h->chi_h.size());
      std::vector<float> chi32(h->chi_h.begin(), h->chi_h.end());
      h->chi32 = upload(h, chi32.data(), chi32.size());
      h->gdv64 = upload(h, gdv.data(), gdv.size());
      std::vector<float> gdv32(gdv.begin(), gdv.end());
      h->gdv32 = upload(h, gdv32.data(), gdv32.size());
      if (both) {
        try {
          const BandTables t = tables.get();
          h->ws_band_slots = std::max<int>(1, (int)t.r.slot_q.size());
          build_band_tables(h, t);
          h->band_apply = from.apply;
          h->band_filter = from.filter;
        } catch (...) {  // a point in too many supports, or no memory: the records serve
          h->ws_band_slots = 0;
        }
      }
    }
    *out = h;
    return CHEFSI_OK;
  } catch (const Error& e) {
    release(h);
    delete h;
    return e.status;
  } catch (const std::bad_alloc&) {
    release(h);
    delete h;
    return CHEFSI_ERR_OOM;
  } catch (...) {
    release(h);
    delete h;
    return CHEFSI_ERR_HIP;
  }
}

void chefsi_destroy(chefsi_handle_t* h) {
  if (!h) return;
  release(h);
  delete h;
}

int chefsi_workspace_bytes(const chefsi_handle_t* hc, int32_t ns, size_t* bytes) {
  chefsi_handle* h = const_cast<chefsi_handle*>(hc);
  return guarded(h, [&] {
    check(bytes != nullptr, "bytes is NULL");
    check_ns(h, ns);
    *bytes = layout(h, ns).total;
  });
}

int chefsi_spectral_bounds(const chefsi_handle_t* hc, double* lam_lo, double* lam_cut, double* lam_hi) {
  chefsi_handle* h = const_cast<chefsi_handle*>(hc);
  return guarded(h, [&] {
    double s = std::fabs(h->w[0]);
    for (int p = 1; p <= h->radius; ++p) s += 2.0 * std::fabs(h->w[p]);
    double kin = 0.0;
    for (int d = 0; d < 3; ++d) kin += 0.5 * s / (h->h[d] * h->h[d]);
    double vmax = -INFINITY, vmin = INFINITY;
    for (double v : h->veff_h) {
      vmax = std::max(vmax, v);
      vmin = std::min(vmin, v);
    }
    std::vector<double> row(h->nd, 0.0);
    bool negative = false;
    int64_t coff = 0;
    int q = 0;
    for (int J = 0; J < h->n_atoms; ++J) {
      const int64_t s0 = h->supp_ptr_h[J], nj = h->supp_ptr_h[J + 1] - s0;
      for (int a = 0; a < h->nproj_h[J]; ++a, ++q) {
        const double* c = h->chi_h.data() + coff + a * nj;
        double l1 = 0.0;
        for (int64_t t = 0; t < nj; ++t) l1 += std::fabs(c[t]);
        const double g = std::fabs(h->gamma_h[q]);
        if (h->gamma_h[q] < 0) negative = true;
        for (int64_t t = 0; t < nj; ++t) row[h->supp_idx_h[s0 + t]] += g * std::fabs(c[t]) * l1 * h->dv;
      }
      coff += nj * h->nproj_h[J];
    }
    double nlb = 0.0;
    for (double v : row) nlb = std::max(nlb, v);
    const double hi = kin + vmax + nlb;
    const double lo = vmin - (negative ? nlb : 0.0);
    if (lam_hi) *lam_hi = hi;
    if (lam_lo) *lam_lo = lo;
    if (lam_cut) *lam_cut = lo + 0.1 * (hi - lo);
  });
}

int chefsi_static_scratch_bytes(const chefsi_handle_t* h, int32_t ns, size_t* bytes) {
  if (h == nullptr || bytes == nullptr || ns < 1) return CHEFSI_ERR_INVALID_ARG;
  *bytes = (size_t)h->np_tot * (size_t)ns * (h->precision == CHEFSI_FP64 ? sizeof(double) : sizeof(float));
  return CHEFSI_OK;
}

int chefsi_apply_h_static(chefsi_handle_t* h, const void* X, void* Y, int32_t ns, void* stream) {
  return guarded(h, [&] {
    check(X != nullptr && Y != nullptr && X != Y, "X and Y must be distinct device blocks");
    check_ns(h, ns);
    size_t need = 0;
    (void)chefsi_static_scratch_bytes(h, ns, &need);
    if (need > (size_t)CHEFSI_STATIC_SCRATCH_BYTES)
      throw Error{CHEFSI_ERR_WORKSPACE, "np_tot x ns projector coefficients (" + std::to_string(need) +
                                            " bytes) exceed the static scratch of " +
                                            std::to_string((size_t)CHEFSI_STATIC_SCRATCH_BYTES) +
                                            " bytes: call on fewer orbitals at a time"};
    void* alpha = scratch_address(h->device);  // looked up at create; a table read here
    hipStream_t s = (hipStream_t)stream;
    // no event records either (profiling may create events): the call only enqueues kernels
    const bool prof = h->prof_on;
    h->prof_on = false;
    struct Restore {
      chefsi_handle* h;
      bool v;
      ~Restore() { h->prof_on = v; }
    } restore{h, prof};
    const BandScratch bs{h->nb_partial, h->nb_partial_bytes};
    if (h->precision == CHEFSI_FP64)
      apply_fused<double, double, double>(h, (const double*)X, nullptr, (double*)Y, ns, 1.0, 0.0, 0.0,
                                          (double*)alpha, s, bs);
    else
      apply_fused<float, float, float>(h, (const float*)X, nullptr, (float*)Y, ns, 1.0, 0.0, 0.0, (float*)alpha,
                                       s, bs);
  });
}

int chefsi_apply_h(chefsi_handle_t* h, const void* X, void* Y, int32_t ns, void* ws, size_t ws_bytes, void* stream) {
  return guarded(h, [&] {
    check(X != nullptr && Y != nullptr && X != Y, "X and Y must be distinct device blocks");
    check_ns(h, ns);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64)
      apply_fused<double, double, double>(h, (const double*)X, nullptr, (double*)Y, ns, 1.0, 0.0, 0.0,
                                          at<double>(ws, L.alpha), s, band_scratch(h, ws, L));
    else
      apply_fused<float, float, float>(h, (const float*)X, nullptr, (float*)Y, ns, 1.0, 0.0, 0.0,
                                       at<float>(ws, L.alpha), s, band_scratch(h, ws, L));
  });
}

int chefsi_filter(chefsi_handle_t* h, void* X, int32_t ns, int32_t degree, double lam_lo, double lam_cut,
                  double lam_hi, void* ws, size_t ws_bytes, void* stream) {
  return guarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check(degree >= 1, "degree must be >= 1");
    check_ns(h, ns);
    check_bounds(lam_lo, lam_cut, lam_hi);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64) {
      double* A = (double*)X;
      double* r = run_filter<double>(h, A, at<double>(ws, L.bufB), ns, degree, lam_lo, lam_cut, lam_hi,
                                     at<double>(ws, L.alpha), s, band_scratch(h, ws, L));
      if (r != A) copy_block<double>(h, A, r, ns, s);
    } else {
      float* A = (float*)X;
      float* r = run_filter<float>(h, A, at<float>(ws, L.bufB), ns, degree, lam_lo, lam_cut, lam_hi,
                                   at<float>(ws, L.alpha), s, band_scratch(h, ws, L));
      if (r != A) copy_block<float>(h, A, r, ns, s);
    }
  });
}

int chefsi_project(chefsi_handle_t* h, const void* X, int32_t ns, double* Hs, double* Ms, void* ws,
                   size_t ws_bytes, void* stream) {
  return guarded(h, [&] {
    check(X != nullptr && Hs != nullptr && Ms != nullptr, "null pointer");
    check_ns(h, ns);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64) {
      double* Y = at<double>(ws, L.bufB);
      apply_fused<double, double, double>(h, (const double*)X, nullptr, Y, ns, 1.0, 0.0, 0.0,
                                          at<double>(ws, L.alpha), s, band_scratch(h, ws, L));
      gram_pair<double, double>(h, (const double*)X, Y, ns, L, ws, Hs, Ms, s, Gemm::F64);
    } else {
      float* Y = at<float>(ws, L.bufB);
      apply_fused<float, float, float>(h, (const float*)X, nullptr, Y, ns, 1.0, 0.0, 0.0, at<float>(ws, L.alpha),
                                       s, band_scratch(h, ws, L));
      gram_pair<float, float>(h, (const float*)X, Y, ns, L, ws, Hs, Ms, s, Gemm::BF16X3);
    }
  });
}

int chefsi_eigh(chefsi_handle_t* h, double* Hs, double* Ms, double* D, int32_t ns, void* ws, size_t ws_bytes,
                void* stream) {
  return guarded(h, [&] {
    check(Hs != nullptr && Ms != nullptr && D != nullptr, "null pointer");
    check_ns(h, ns);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    dense_eig(h, Hs, Ms, D, ns, L, ws, s);
    check_info(h, ws, L, ns, s);
  });
}

int chefsi_rotate(chefsi_handle_t* h, void* X, const double* Z, int32_t ns, void* ws, size_t ws_bytes,
                  void* stream) {
  return guarded(h, [&] {
    check(X != nullptr && Z != nullptr, "null pointer");
    check_ns(h, ns);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64) {
      double* B = at<double>(ws, L.bufB);
      rotate_into<double>(h, (const double*)X, Z, B, ns, s, Gemm::F64, ws, L);
      copy_block<double>(h, (double*)X, B, ns, s);
    } else {
      float* B = at<float>(ws, L.bufB);
      rotate_into<float>(h, (const float*)X, Z, B, ns, s, Gemm::BF16X3, ws, L);
      copy_block<float>(h, (float*)X, B, ns, s);
    }
  });
}

int chefsi_step(chefsi_handle_t* h, void* X, int32_t ns, int32_t degree, double lam_lo, double lam_cut,
                double lam_hi, void* ws, size_t ws_bytes, void* stream, double* ritz_host) {
  return guarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check(degree >= 1, "degree must be >= 1");
    check_ns(h, ns);
    check_bounds(lam_lo, lam_cut, lam_hi);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64)
      step_impl<double>(h, (double*)X, ns, degree, lam_lo, lam_cut, lam_hi, ws, L, s, ritz_host);
    else
      step_impl<float>(h, (float*)X, ns, degree, lam_lo, lam_cut, lam_hi, ws, L, s, ritz_host);
  });
}

int chefsi_solve(chefsi_handle_t* h, void* X, int32_t ns, int32_t degree, int32_t n_iter, double lam_lo,
                 double lam_cut, double lam_hi, void* ws, size_t ws_bytes, void* stream, double* ritz_host,
                 double* lam_lo_out, double* lam_cut_out) {
  return guarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check(degree >= 1 && n_iter >= 1, "degree and n_iter must be >= 1");
    check_ns(h, ns);
    check_bounds(lam_lo, lam_cut, lam_hi);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    std::vector<double> d(ns);
    double lo = lam_lo, cut = lam_cut;
    for (int it = 0; it < n_iter; ++it) {
      check_bounds(lo, cut, lam_hi);
      if (h->precision == CHEFSI_FP64)
        step_impl<double>(h, (double*)X, ns, degree, lo, cut, lam_hi, ws, L, s, d.data());
      else
        step_impl<float>(h, (float*)X, ns, degree, lo, cut, lam_hi, ws, L, s, d.data());
      lo = d[0];
      cut = d[ns - 1];
    }
    if (ritz_host) std::memcpy(ritz_host, d.data(), (size_t)ns * 8);
    if (lam_lo_out) *lam_lo_out = lo;
    if (lam_cut_out) *lam_cut_out = cut;
  });
}

int chefsi_refine_fp64(chefsi_handle_t* h, void* X, int32_t ns, int32_t degree, double lam_lo, double lam_cut,
                       double lam_hi, void* ws, size_t ws_bytes, void* stream, double* ritz_host) {
  return guarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check(degree >= 0, "degree must be >= 0");
    check_ns(h, ns);
    if (degree > 0) check_bounds(lam_lo, lam_cut, lam_hi);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64)
      refine_impl<double>(h, (double*)X, ns, degree, lam_lo, lam_cut, lam_hi, ws, L, s, ritz_host);
    else
      refine_impl<float>(h, (float*)X, ns, degree, lam_lo, lam_cut, lam_hi, ws, L, s, ritz_host);
  });
}

}  // extern "C"

namespace {

// ---------------------------------------------------------------------------
// Lanczos estimate of lam_Nd (Alg. 1: the largest eigenvalue of H).
// Workspace: v_{j-1}, v_j (storage type), w (FP64), the projector coefficients of one
// vector (FP64), the block sums and two result words.
// ---------------------------------------------------------------------------
struct LzLayout {
  size_t v0 = 0, v1 = 0, w = 0, alpha = 0, partial = 0, out = 0, band = 0, band_bytes = 0, total = 0;
};

LzLayout lanczos_layout(const chefsi_handle* h) {
  LzLayout L;
  const size_t vb = (size_t)h->nd * elem_bytes(h);
  size_t off = 0;
  L.v0 = off;
  off += align256(vb);
  L.v1 = off;
  off += align256(vb);
  L.w = off;
  off += align256((size_t)h->nd * 8);
  L.alpha = off;
  off += align256((size_t)std::max(1, h->np_tot) * 8);
  L.partial = off;
  off += align256((size_t)kVecBlocks * 8);
  L.out = off;
  off += 256;
  L.band = off;
  if (h->ws_band_slots > 0) L.band_bytes = (size_t)h->ws_band_slots * 8;
  off += align256(L.band_bytes);
  L.total = off;
  return L;
}

// Largest eigenvalue theta of the symmetric tridiagonal T (diagonal a[0..k), off-diagonal
// b[0..k-1)) by Sturm-count bisection to full precision, and the last component of its
// unit eigenvector by two steps of inverse iteration (T - theta I with a tiny shift).
void tridiagonal_top(const std::vector<double>& a, const std::vector<double>& b, double* theta, double* s_last) {
  const int k = (int)a.size();
  double lo = a[0], hi = a[0];
  for (int i = 0; i < k; ++i) {
    const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(b[i]) : 0.0);
    lo = std::min(lo, a[i] - r);
    hi = std::max(hi, a[i] + r);
  }
  auto count_above = [&](double x) {  // eigenvalues > x (Sturm sequence of T - x I)
    int neg = 0;
    double d = 1.0;
    for (int i = 0; i < k; ++i) {
      const double bb = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
      d = (a[i] - x) - (i > 0 ? bb / d : 0.0);
      if (d == 0.0) d = -1e-300;
      if (d < 0.0) ++neg;
    }
    return k - neg;
  };
  for (int it = 0; it < 200 && hi - lo > 2e-16 * std::max(std::fabs(lo), std::fabs(hi)); ++it) {
    const double mid = 0.5 * (lo + hi);
    if (count_above(mid) >= 1) lo = mid; else hi = mid;
  }
  *theta = 0.5 * (lo + hi);
  if (k == 1) {
    *s_last = 1.0;
    return;
  }
  const double shift = *theta + 1e-13 * std::max(1.0, std::fabs(*theta));
  std::vector<double> x(k, 1.0), c(k), d(k), y(k);
  for (int rep = 0; rep < 3; ++rep) {  // solve (T - shift I) y = x (tridiagonal LU, no pivoting)
    for (int i = 0; i < k; ++i) {
      d[i] = a[i] - shift;
      y[i] = x[i];
    }
    for (int i = 1; i < k; ++i) {
      const double m = b[i - 1] / d[i - 1];
      d[i] -= m * b[i - 1];
      y[i] -= m * y[i - 1];
    }
    x[k - 1] = y[k - 1] / d[k - 1];
    for (int i = k - 2; i >= 0; --i) x[i] = (y[i] - b[i] * x[i + 1]) / d[i];
    double nrm = 0.0;
    for (double v : x) nrm += v * v;
    nrm = std::sqrt(nrm);
    for (double& v : x) v /= nrm;
  }
  *s_last = x[k - 1];
}

// The coefficients of up to kLzBatch steps are left on the device, behind the two sets of block
// sums, and read together: the host only waits for a batch.  After an early stop (beta = 0)
// the rest of a batch runs on non-finite vectors and is not looked at.
constexpr int kLzScalars = kVecBlocks - 2 * kLzBlocks + 32;  // partial's rest and the out region behind it
constexpr int kLzBatch = (kLzScalars - 1) / 2;

template <typename TV>
void lanczos_impl(chefsi_handle* h, const TV* v0, int steps, void* ws, const LzLayout& L, hipStream_t s,
                  std::vector<double>& a, std::vector<double>& b) {
  TV* vb[2] = {at<TV>(ws, L.v0), at<TV>(ws, L.v1)};
  double* w = at<double>(ws, L.w);
  double* dots = at<double>(ws, L.partial);
  double* squares = dots + kLzBlocks;
  double* scal = squares + kLzBlocks;  // |v0|, then alpha, beta of each step of the batch
  double host[kLzScalars];
  // v_1 = v0 / ||v0||
  HIP_TRY(launch_widen<TV>(v0, h->nd, w, s));
  HIP_TRY(launch_lanczos_norm<TV>(w, nullptr, nullptr, h->nd, squares, nullptr, s));
  HIP_TRY(launch_lanczos_scale<TV>(w, squares, h->nd, vb[0], scal, s));
  int cur = 0;
  const double* beta = nullptr;  // the previous step's, on the device
  for (int j0 = 0; j0 < steps; j0 += kLzBatch) {
    const int nb = std::min(kLzBatch, steps - j0);
    for (int i = 0; i < nb; ++i) {
      const TV* v = vb[cur];
      TV* vprev = vb[cur ^ 1];
      double* alpha = scal + 1 + 2 * i;
      apply_fused<TV, double, double>(h, v, nullptr, w, 1, 1.0, 0.0, 0.0, at<double>(ws, L.alpha), s,
                                      band_scratch(h, ws, L));
      HIP_TRY(launch_lanczos_dot<TV>(w, v, beta != nullptr ? vprev : nullptr, beta, h->nd, dots, s));
      HIP_TRY(launch_lanczos_norm<TV>(w, v, dots, h->nd, squares, alpha, s));
      HIP_TRY(launch_lanczos_scale<TV>(w, squares, h->nd, vprev, alpha + 1, s));  // v_{j+1} over v_{j-1}
      beta = alpha + 1;
      cur ^= 1;
    }
    HIP_TRY(hipMemcpyAsync(h->pinned, scal, (size_t)(1 + 2 * nb) * sizeof(double), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    std::memcpy(host, h->pinned, (size_t)(1 + 2 * nb) * sizeof(double));
    check(std::isfinite(host[0]) && host[0] > 0.0, "the start vector must be finite and nonzero");
    for (int i = 0; i < nb; ++i) {
      const double al = host[1 + 2 * i], be = host[2 + 2 * i];
      if (!std::isfinite(al) || !std::isfinite(be)) throw Error{CHEFSI_ERR_NONFINITE, "non-finite Lanczos coefficient"};
      a.push_back(al);
      b.push_back(be);
      if (be == 0.0) return;
    }
  }
}

// ---------------------------------------------------------------------------
// Nonlocal forces and stresses.  Workspace: the partial sums (over atoms and orbitals, or
// over the blocks of the kinetic stress), occupations, the per-atom or total sums, and the
// support-point displacements.  The sizes are those the calls have always asked for (an FP64
// Nd x ns block, two coefficient blocks, three copies of the projector values): the partial
// sums need less, unless the atoms outnumber a tenth of the grid points.
// ---------------------------------------------------------------------------
struct FoLayout {
  size_t part = 0, occ = 0, sums = 0, disp = 0, total = 0;
  int64_t part_doubles = 0;
};

FoLayout forces_layout(const chefsi_handle* h, int ns) {
  FoLayout L;
  const size_t np = (size_t)std::max(1, h->np_tot), na = (size_t)std::max(1, h->n_atoms);
  const size_t part = align256((size_t)h->nd * ns * 8) + 2 * align256(np * ns * 8) + align256(np * 8);
  size_t off = std::max(part, align256((size_t)h->n_atoms * ns * 10 * 8));
  L.part_doubles = (int64_t)(off / 8);
  L.occ = off;
  off += align256((size_t)ns * 8);
  off += align256(na * 3 * 8) + align256(((size_t)kVecBlocks * 6 + 8) * 8);
  L.disp = off;
  off += align256(std::max<size_t>(1, 3 * h->supp_idx_h.size()) * 8);
  off += align256(std::max<size_t>(1, 3 * h->chi_h.size()) * 8);
  L.sums = off;
  off += align256(na * 12 * 8);
  L.total = off;
  return L;
}

// Central first-derivative weights of order 2r: c_p = (-1)^(p+1) (r!)^2 / (p (r-p)! (r+p)!).
std::vector<double> first_derivative_weights(int r) {
  std::vector<double> c(r + 1, 0.0);
  auto fact = [](int k) {
    double f = 1.0;
    for (int i = 2; i <= k; ++i) f *= i;
    return f;
  };
  for (int p = 1; p <= r; ++p)
    c[p] = ((p % 2) ? 1.0 : -1.0) * fact(r) * fact(r) / (p * fact(r - p) * fact(r + p));
  return c;
}

// Arguments of the force and stress kernels shared by the three calls: the block, its
// occupations (copied to the workspace) and the FD first-derivative weights.
template <typename TA, typename TV>
void gradient_args(chefsi_handle* h, TA& a, const TV* X, int ns, const double* occ_host, void* ws, const FoLayout& L,
                   hipStream_t s) {
  HIP_TRY(hipMemcpyAsync(at<double>(ws, L.occ), occ_host, (size_t)ns * 8, hipMemcpyHostToDevice, s));
  a.x = X;
  a.occ = at<double>(ws, L.occ);
  a.nd = h->nd;
  a.ns = ns;
  a.nx = h->n[0];
  a.ny = h->n[1];
  a.nz = h->n[2];
  const std::vector<double> c = first_derivative_weights(h->radius);
  for (int d = 0; d < 3; ++d) {
    a.periodic[d] = h->bc[d] == 0 ? 1 : 0;
    for (int p = 1; p <= h->radius; ++p) a.c[d][p] = c[p] / h->h[d];
  }
}

// n doubles at device address d to the handle's pinned staging, after the stream's work.
const double* read_pinned(chefsi_handle* h, const double* d, size_t n, hipStream_t s) {
  HIP_TRY(hipMemcpyAsync(h->pinned, d, n * 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  return h->pinned;
}

// Per-atom sums of the nonlocal forces (3 values per atom, times -2) or, with the support
// displacements, of the nonlocal stress (10 values per atom: energy, then direction pairs).
template <typename TV>
const double* nonlocal_sums(chefsi_handle* h, const TV* X, int ns, const double* occ_host, const double* disp_host,
                            void* ws, const FoLayout& L, hipStream_t s) {
  NlGradArgs<TV> a{};
  gradient_args(h, a, X, ns, occ_host, ws, L, s);
  if (disp_host != nullptr) {
    HIP_TRY(hipMemcpyAsync(at<double>(ws, L.disp), disp_host, 3 * h->supp_idx_h.size() * 8, hipMemcpyHostToDevice, s));
    a.disp = at<double>(ws, L.disp);
  }
  a.n_atoms = h->n_atoms;
  a.supp_off = h->supp_off;
  a.supp_idx = h->supp_idx;
  a.chi_off = h->chi_off;
  a.nproj = h->nproj;
  a.poff = h->poff;
  a.chi = h->chi64;
  a.gdv = h->gdv64;
  a.dv = h->dv;
  a.box = h->supp_box;
  a.part = at<double>(ws, L.part);
  double* out = at<double>(ws, L.sums);
  HIP_TRY((launch_nl_grad<TV>(a, h->radius, out, disp_host != nullptr ? 1.0 : -2.0, s)));
  return read_pinned(h, out, (size_t)h->n_atoms * (disp_host != nullptr ? 10 : 3), s);
}

// Nonlocal stress (see chefsi.h): the per-atom sums of the energy and of the nine direction
// pairs, added on the host in atom order.
template <typename TV>
void nonlocal_stress_impl(chefsi_handle* h, const TV* X, int ns, const double* occ_host, const double* disp_host,
                          void* ws, const FoLayout& L, hipStream_t s, double* stress_host) {
  const double* sums = nonlocal_sums<TV>(h, X, ns, occ_host, disp_host, ws, L, s);
  const double omega = (double)h->nd * h->dv;
  double t[10] = {0.0};
  for (int J = 0; J < h->n_atoms; ++J)
    for (int k = 0; k < 10; ++k) t[k] += sums[(size_t)J * 10 + k];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) stress_host[a * 3 + b] = -((a == b ? t[0] : 0.0) + 2.0 * t[1 + 3 * a + b]) / omega;
}

template <typename TV>
void kinetic_stress_impl(chefsi_handle* h, const TV* X, int ns, const double* occ_host, void* ws, const FoLayout& L,
                         hipStream_t s, double* stress_host) {
  StressArgs<TV> a{};
  gradient_args(h, a, X, ns, occ_host, ws, L, s);
  a.partial = at<double>(ws, L.part);
  a.out = at<double>(ws, L.sums);
  HIP_TRY(launch_stress_sums<TV>(a, h->radius, L.part_doubles / 6, s));
  const double* sums = read_pinned(h, a.out, 6, s);
  // sigma_ab = -(dV / Omega) sum = -(1 / Nd) sum, Omega = Nd dV
  const int ia[6] = {0, 1, 2, 0, 0, 1}, ib[6] = {0, 1, 2, 1, 2, 2};
  for (int k = 0; k < 6; ++k) {
    const double v = -sums[k] / (double)h->nd;
    stress_host[ia[k] * 3 + ib[k]] = v;
    stress_host[ib[k] * 3 + ia[k]] = v;
  }
}

}  // namespace

extern "C" {

int chefsi_kinetic_stress(chefsi_handle_t* h, const void* X, int32_t ns, const double* occ_host, void* ws,
                          size_t ws_bytes, void* stream, double* stress_host) {
  return guarded(h, [&] {
    check(X != nullptr && occ_host != nullptr && stress_host != nullptr && ws != nullptr,
          "X, occ, stress and ws must not be NULL");
    check_ns(h, ns);
    for (int i = 0; i < ns; ++i) check(std::isfinite(occ_host[i]), "occupations must be finite");
    const FoLayout L = forces_layout(h, ns);
    if (ws_bytes < L.total) throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_forces_workspace_bytes"};
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64)
      kinetic_stress_impl<double>(h, (const double*)X, ns, occ_host, ws, L, s, stress_host);
    else
      kinetic_stress_impl<float>(h, (const float*)X, ns, occ_host, ws, L, s, stress_host);
  });
}

int chefsi_nonlocal_stress(chefsi_handle_t* h, const void* X, int32_t ns, const double* occ_host,
                           const double* disp_host, void* ws, size_t ws_bytes, void* stream, double* stress_host) {
  return guarded(h, [&] {
    check(X != nullptr && occ_host != nullptr && stress_host != nullptr, "X, occ and stress must not be NULL");
    check_ns(h, ns);
    for (int i = 0; i < ns; ++i) check(std::isfinite(occ_host[i]), "occupations must be finite");
    if (h->n_atoms == 0 || h->np_tot == 0) {
      std::fill(stress_host, stress_host + 9, 0.0);
      return;
    }
    check(disp_host != nullptr, "disp must not be NULL when there are projectors");
    const size_t nsupp = h->supp_idx_h.size();
    for (size_t i = 0; i < 3 * nsupp; ++i) check(std::isfinite(disp_host[i]), "displacements must be finite");
    check(ws != nullptr, "ws is NULL");
    const FoLayout L = forces_layout(h, ns);
    if (ws_bytes < L.total) throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_forces_workspace_bytes"};
    hipStream_t s = (hipStream_t)stream;
    if (h->precision == CHEFSI_FP64)
      nonlocal_stress_impl<double>(h, (const double*)X, ns, occ_host, disp_host, ws, L, s, stress_host);
    else
      nonlocal_stress_impl<float>(h, (const float*)X, ns, occ_host, disp_host, ws, L, s, stress_host);
  });
}

int chefsi_forces_workspace_bytes(const chefsi_handle_t* hc, int32_t ns, size_t* bytes) {
  chefsi_handle* h = const_cast<chefsi_handle*>(hc);
  return guarded(h, [&] {
    check(bytes != nullptr, "bytes is NULL");
    check_ns(h, ns);
    *bytes = forces_layout(h, ns).total;
  });
}

int chefsi_nonlocal_forces(chefsi_handle_t* h, const void* X, int32_t ns, const double* occ_host, void* ws,
                           size_t ws_bytes, void* stream, double* forces_host) {
  return guarded(h, [&] {
    check(X != nullptr && occ_host != nullptr && forces_host != nullptr, "X, occ and forces must not be NULL");
    check_ns(h, ns);
    for (int i = 0; i < ns; ++i) check(std::isfinite(occ_host[i]), "occupations must be finite");
    if (h->n_atoms == 0 || h->np_tot == 0) {
      std::fill(forces_host, forces_host + 3 * (size_t)h->n_atoms, 0.0);
      return;
    }
    check(ws != nullptr, "ws is NULL");
    const FoLayout L = forces_layout(h, ns);
    if (ws_bytes < L.total) throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_forces_workspace_bytes"};
    hipStream_t s = (hipStream_t)stream;
    const double* f;
    if (h->precision == CHEFSI_FP64)
      f = nonlocal_sums<double>(h, (const double*)X, ns, occ_host, nullptr, ws, L, s);
    else
      f = nonlocal_sums<float>(h, (const float*)X, ns, occ_host, nullptr, ws, L, s);
    std::memcpy(forces_host, f, (size_t)h->n_atoms * 3 * 8);
  });
}

int chefsi_lanczos_workspace_bytes(const chefsi_handle_t* hc, size_t* bytes) {
  chefsi_handle* h = const_cast<chefsi_handle*>(hc);
  return guarded(h, [&] {
    check(bytes != nullptr, "bytes is NULL");
    *bytes = lanczos_layout(h).total;
  });
}

int chefsi_lanczos_bound(chefsi_handle_t* h, const void* v0, int32_t steps, void* ws, size_t ws_bytes, void* stream,
                         double* lam_nd, double* theta, double* alpha_host, double* beta_host) {
  return guarded(h, [&] {
    check(v0 != nullptr && ws != nullptr, "v0 and ws must be device buffers");
    check(steps >= 1 && steps <= 1000, "steps must be in 1..1000");
    check(lam_nd != nullptr, "lam_nd is NULL");
    const LzLayout L = lanczos_layout(h);
    if (ws_bytes < L.total) throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_lanczos_workspace_bytes"};
    hipStream_t s = (hipStream_t)stream;
    std::vector<double> a, b;
    if (h->precision == CHEFSI_FP64)
      lanczos_impl<double>(h, (const double*)v0, steps, ws, L, s, a, b);
    else
      lanczos_impl<float>(h, (const float*)v0, steps, ws, L, s, a, b);
    double th = 0.0, sl = 0.0;
    tridiagonal_top(a, b, &th, &sl);
    *lam_nd = th + std::fabs(b.back() * sl);
    if (theta) *theta = th;
    for (size_t i = 0; i < a.size(); ++i) {
      if (alpha_host) alpha_host[i] = a[i];
      if (beta_host) beta_host[i] = b[i];
    }
    for (size_t i = a.size(); i < (size_t)steps; ++i) {  // stopped early (invariant subspace)
      if (alpha_host) alpha_host[i] = 0.0;
      if (beta_host) beta_host[i] = 0.0;
    }
  });
}

int chefsi_set_stencil_tiling(chefsi_handle_t* h, int32_t rows_per_thread, int32_t row_groups) {
  return guarded(h, [&] {
    check(rows_per_thread >= 0 && rows_per_thread <= 4 && row_groups >= 0, "tiling parameters out of range");
    check((rows_per_thread == 0) == (row_groups == 0), "give both tiling parameters, or neither");
    const int eb = h->precision == CHEFSI_FP64 ? 8 : 4;
    const HxPlan p = plan_hx(h->n[0], h->n[1], h->n[2], 1, h->radius, eb, rows_per_thread, row_groups);
    check(p.ok, "the requested stencil tiling does not fit this grid");
    if (h->np_tot > 0)
      build_hx_records(h, p);
    else
      h->hx_plan = p;
  });
}

// Average time of one filter-form launch sequence (projector gather, stencil pass with the
// three-term update, scatter pass) on the first ns columns of X, written into the workspace
// block (X is not modified).
extern "C++" {
template <typename T>
static float time_filter_launch(chefsi_handle* h, const T* X, T* B, int ns, T* alpha, hipStream_t s,
                                hipEvent_t e0, hipEvent_t e1, BandScratch bs, int warm, int runs) {
  for (int i = 0; i < warm; ++i) apply_fused<T, T, T>(h, X, B, B, ns, 0.5, 0.25, -0.5, alpha, s, bs, false, true);
  HIP_TRY(hipEventRecord(e0, s));
  for (int i = 0; i < runs; ++i) apply_fused<T, T, T>(h, X, B, B, ns, 0.5, 0.25, -0.5, alpha, s, bs, true, true);
  HIP_TRY(hipEventRecord(e1, s));
  HIP_TRY(hipEventSynchronize(e1));
  float ms = 0.f;
  HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
  return ms / runs;
}
}  // extern "C++"

// Leave the band pass that a handle as created has beside its records.
static void leave_band(chefsi_handle* h) {
  if (h->rec_max == 0) return;
  h->band_apply = h->band_filter = kNoBand;
  free_band_tables(h);
}

// Switch the projector route of a handle with projectors (mode 4: records in the stencil
// pass, 0: band pass).  A route that cannot be built (a point in more than kBandMaxSlots
// projector supports, records whose LDS does not fit the current tiling, no memory) throws and
// leaves the handle on its current route: the new tables are complete before the old ones go.
static void set_projector_route(chefsi_handle* h, int mode) {
  if (mode == 0) {
    build_band_tables(h, band_tables(h, false));
    h->band_apply = h->band_filter = kNoBand;
    h->rec_max = 0;
    build_hx_records(h, h->hx_plan);  // none: nothing is allocated
    build_scatter_records(h);
  } else {
    check(hx_records_fit(h, h->hx_plan), "too many projectors for the stencil pass (alpha row does not fit in LDS)");
    const int was = h->rec_max;
    h->rec_max = mode;
    try {
      build_hx_records(h, h->hx_plan);
      build_scatter_records(h);
    } catch (...) {
      h->rec_max = was;
      build_hx_records(h, h->hx_plan);  // none again
      throw;
    }
    h->band_apply = h->band_filter = kNoBand;
    free_band_tables(h);
  }
}

int chefsi_autotune(chefsi_handle_t* h, const void* X, int32_t ns, void* ws, size_t ws_bytes, void* stream,
                    int32_t* choice) {
  return guarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check_ns(h, ns);
    WsLayout L;
    check_ws(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    const int nt = std::min(ns, 1024);  // orbitals timed: the per-orbital work is the same for all
    const int eb = h->precision == CHEFSI_FP64 ? 8 : 4;
    const int nx = h->n[0], ny = h->n[1];
    // candidate tilings: every row count per thread and row-group count the planner accepts,
    // tall tiles only (at least r + 1 rows, or the whole y extent)
    std::vector<HxPlan> cands;
    for (int py = 1; py <= 4; ++py)
      for (int nyg = 1; nx * nyg <= hx_max_threads(py); ++nyg) {
        if (py * nyg < std::min(h->radius + 1, ny) || py * nyg > ny + 2 * h->radius) continue;
        const HxPlan p = plan_hx(nx, ny, h->n[2], 1, h->radius, eb, py, nyg);
        if (p.ok) cands.push_back(p);
      }
    check(!cands.empty(), "no stencil tiling fits this grid");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    struct Events {
      hipEvent_t a, b;
      ~Events() {
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
      }
    } ev{e0, e1};
    const bool prof = h->prof_on;
    h->prof_on = false;
    leave_band(h);
    float best = 1e30f;
    int best_mode = h->rec_max, best_c = 0;
    auto timed = [&](const HxPlan& p, int nt, int warm, int runs) {
      if (h->np_tot > 0)
        build_hx_records(h, p);
      else
        h->hx_plan = p;
      return h->precision == CHEFSI_FP64
                 ? time_filter_launch<double>(h, (const double*)X, at<double>(ws, L.bufB), nt, at<double>(ws, L.alpha),
                                              s, e0, e1, band_scratch(h, ws, L), warm, runs)
                 : time_filter_launch<float>(h, (const float*)X, at<float>(ws, L.bufB), nt, at<float>(ws, L.alpha), s,
                                             e0, e1, band_scratch(h, ws, L), warm, runs);
    };
    struct Timed {
      float ms;
      int mode, c;
    };
    std::vector<Timed> seen;
    const int modes[2] = {h->rec_max > 0 ? 4 : 0, h->rec_max > 0 ? 0 : 4};  // the current one first
    for (int mode : modes) {
      if (h->np_tot == 0 && mode == 0) continue;
      if (h->rec_max != mode) {
        if (mode > 0)  // switch on the first tiling whose records fit (any tiling serves the band route)
          for (const HxPlan& c : cands)
            if (hx_records_fit(h, c)) {
              h->hx_plan = c;
              break;
            }
        try {
          set_projector_route(h, mode);
        } catch (const Error& e) {
          if (e.status == CHEFSI_ERR_INVALID_ARG) continue;  // this route cannot serve this handle
          throw;
        }
      }
      for (size_t c = 0; c < cands.size(); ++c) {
        if (h->np_tot > 0 && mode > 0 && !hx_records_fit(h, cands[c])) continue;  // tile too tall for the records
        const float ms = timed(cands[c], nt, 1, 3);
        seen.push_back({ms, mode, (int)c});
        if (ms < best) {
          best = ms;
          best_mode = mode;
          best_c = (int)c;
        }
      }
    }
    if (best == 1e30f) h->prof_on = prof;
    check(best < 1e30f, "no stencil tiling fits the projector records of this handle");
    h->hx_plan = cands[best_c];  // a route switch builds its records for the chosen tiling
    if (h->rec_max != best_mode) set_projector_route(h, best_mode);
    // The chosen route's four best are timed again in turn, the first of three rounds left out:
    // the tables built on the host between two routes let the clocks recover, so what is timed
    // first after them runs up to 20 % faster, and 1024 orbitals may happen to fill whole waves
    // of blocks where ns does not (60x60x180, 1200 FP32 orbitals: 32-row tiles 1.93 against
    // 2.40 ms, so that they won over 12-row ones; 71.8 against 69.7 ms a filter).
    // One launch a round where it takes long enough to time (120^3, 1800 orbitals: 1.75 -> 1.10 s).
    constexpr int kFinal = 4;
    const int runs = best > 1.5f ? 1 : 3;
    const int nf = std::min(ns, 2048);
    auto less = [](const Timed& a, const Timed& b) { return a.ms < b.ms; };
    seen.erase(std::remove_if(seen.begin(), seen.end(), [&](const Timed& t) { return t.mode != best_mode; }),
               seen.end());
    std::stable_sort(seen.begin(), seen.end(), less);
    if (seen.size() > kFinal) seen.resize(kFinal);
    for (int round = 0; round < 3 && seen.size() > 1; ++round)
      for (Timed& t : seen) {
        const float ms = timed(cands[t.c], nf, runs > 1 || round == 0, runs);
        t.ms = round > 1 ? t.ms + ms : ms;
      }
    best_c = std::min_element(seen.begin(), seen.end(), less)->c;
    h->prof_on = prof;
    if (h->np_tot > 0)
      build_hx_records(h, cands[best_c]);
    else
      h->hx_plan = cands[best_c];
    if (choice) {
      choice[0] = cands[best_c].py;
      choice[1] = cands[best_c].nyg;
      choice[2] = best_mode > 0 ? 1 : 0;
    }
  });
}

int chefsi_set_projector_pass(chefsi_handle_t* h, int32_t in_stencil) {
  return guarded(h, [&] {
    check(in_stencil == 0 || in_stencil == 1, "in_stencil must be 0 or 1");
    const int want = in_stencil ? 4 : 0;
    if (h->np_tot == 0) {
      h->rec_max = want;
      return;
    }
    if (want == h->rec_max) {
      leave_band(h);  // the records everywhere
      return;
    }
    set_projector_route(h, want);
  });
}

int chefsi_get_stencil_tiling(const chefsi_handle_t* hc, int32_t* tiling) {
  chefsi_handle* h = const_cast<chefsi_handle*>(hc);
  return guarded(h, [&] {
    check(tiling != nullptr, "tiling is NULL");
    tiling[0] = h->hx_plan.py;
    tiling[1] = h->hx_plan.nyg;
    tiling[2] = h->hx_plan.ty;
    tiling[3] = h->hx_plan.kh;
  });
}

int chefsi_handle_bytes(const chefsi_handle_t* h, size_t* bytes) {
  if (h == nullptr || bytes == nullptr) return CHEFSI_ERR_INVALID_ARG;
  *bytes = h->device_bytes;
  return CHEFSI_OK;
}

int chefsi_profile_enable(chefsi_handle_t* h, int32_t on) {
  return guarded(h, [&] { h->prof_on = on != 0; });
}

int chefsi_profile_reset(chefsi_handle_t* h) {
  return guarded(h, [&] {
    prof_collect(h);
    for (int i = 0; i < kNumProf; ++i) {
      h->prof_ms[i] = 0.0;
      h->prof_n[i] = 0;
    }
  });
}

int chefsi_profile_read(chefsi_handle_t* h, int32_t kernel_id, double* total_ms, int64_t* launches) {
  return guarded(h, [&] {
    check(kernel_id >= 0 && kernel_id < kNumProf, "kernel_id out of range");
    prof_collect(h);
    if (total_ms) *total_ms = h->prof_ms[kernel_id];
    if (launches) *launches = h->prof_n[kernel_id];
  });
}

}  // extern "C"

// ---------------------------------------------------------------------------
// CheFSI at a Bloch wavevector (complex FP64; Sec. 2: every Brillouin-zone sample other
// than Gamma runs in complex double precision).  H_k = T_k + Veff + V_nl,k with
// Bloch-phased FD ghosts and Bloch-summed projectors; the step is Alg. 1 with conjugate
// transposes: Hs = X~^H H X~, Ms = X~^H X~ (rocBLAS zgemm), Ms = U^H U, C = U^-H Hs U^-1,
// C = W D W^H (rocSOLVER zheevd), Z = U^-1 W, X = X~ Z.
// ---------------------------------------------------------------------------
struct chefsi_kpoint {
  int device = 0;
  int n[3] = {0, 0, 0};
  double h[3] = {0, 0, 0};
  int bc[3] = {0, 0, 0};
  int radius = 6;
  int64_t nd = 0;
  int max_ns = 0;
  double kvec[3] = {0, 0, 0};
  std::vector<double> w;
  int n_atoms = 0, np_tot = 0, n_pts = 0;
  double* veff = nullptr;
  double* gdv = nullptr;
  // band-pass tables (regions of touched points, complex chi~; the gather table conjugated)
  int nreg = 0;
  int max_pts = 0, max_ent = 0, max_slots = 0;  // of the largest band-pass region
  int *reg_pt = nullptr, *pt_idx = nullptr, *pt_ent = nullptr, *ent_ls = nullptr, *reg_slot = nullptr,
      *slot_q = nullptr, *slot_ent = nullptr, *gent_loc = nullptr, *q_slot_ptr = nullptr, *q_slot = nullptr;
  double2 *ent_chi = nullptr, *gent_chi = nullptr, *partial = nullptr;
  double* pinned = nullptr;
  rocblas_handle blas = nullptr;
  std::map<int, size_t> solver_ws_cache;
  bool prof_on = false;
  std::vector<hipEvent_t> ev_pool;
  std::vector<EventPair> ev_pending;
  double prof_ms[kNumProf] = {0};
  int64_t prof_n[kNumProf] = {0};
  std::string last_error;
};

namespace {

struct ZLayout {
  size_t bufB = 0, alpha = 0, hs = 0, ms = 0, d = 0, e = 0, info = 0, partial = 0, solver = 0, total = 0,
         solver_bytes = 0;
  BlasGram kg;  // K chunks of the projection (same split rule as the real FP64 Gram)
};

size_t zsolver_workspace(chefsi_kpoint* h, int ns) {
  auto it = h->solver_ws_cache.find(ns);
  if (it != h->solver_ws_cache.end()) return it->second;
  const rocblas_double_complex one(1.0, 0.0);
  size_t best = 0, sz = 0;
  auto query = [&](auto&& call) {
    BLAS_TRY(rocblas_start_device_memory_size_query(h->blas));
    call();
    BLAS_TRY(rocblas_stop_device_memory_size_query(h->blas, &sz));
    best = std::max(best, sz);
  };
  const rocblas_int ld = (rocblas_int)h->nd;
  query([&] { rocsolver_zpotrf(h->blas, rocblas_fill_upper, ns, nullptr, ns, nullptr); });
  query([&] {
    rocblas_ztrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_conjugate_transpose,
                  rocblas_diagonal_non_unit, ns, ns, &one, nullptr, ns, nullptr, ns);
  });
  query([&] {
    rocblas_ztrsm(h->blas, rocblas_side_right, rocblas_fill_upper, rocblas_operation_none, rocblas_diagonal_non_unit,
                  ns, ns, &one, nullptr, ns, nullptr, ns);
  });
  query([&] {
    rocblas_ztrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_none, rocblas_diagonal_non_unit,
                  ns, ns, &one, nullptr, ns, nullptr, ns);
  });
  query([&] {
    rocsolver_zheevd(h->blas, rocblas_evect_original, rocblas_fill_upper, ns, nullptr, ns, nullptr, nullptr, nullptr);
  });
  const BlasGram kg = plan_blas_gram(h->nd, ns);
  for (int q = 0; q < kg.nblk; ++q) {
    const int m = kg.start[q + 1] - kg.start[q], n = ns - kg.start[q];
    query([&] {
      rocblas_zgemm_strided_batched(h->blas, rocblas_operation_conjugate_transpose, rocblas_operation_none, m, n,
                                    (rocblas_int)kg.kc, &one, nullptr, ld, kg.kc, nullptr, ld, kg.kc, &one, nullptr,
                                    ns, (rocblas_stride)ns * ns, kg.splits);
    });
    if (kg.tail > 0)
      query([&] {
        rocblas_zgemm(h->blas, rocblas_operation_conjugate_transpose, rocblas_operation_none, m, n,
                      (rocblas_int)kg.tail, &one, nullptr, ld, nullptr, ld, &one, nullptr, ns);
      });
  }
  const rocblas_int prow = (rocblas_int)std::max<int64_t>(1, std::min<int64_t>(h->nd, (((int64_t)1 << 31) - 1) / ns));
  query([&] {
    rocblas_zgemm(h->blas, rocblas_operation_none, rocblas_operation_none, prow, ns, ns, &one, nullptr, ld, nullptr,
                  ns, &one, nullptr, ld);
  });
  h->solver_ws_cache[ns] = best;
  return best;
}

ZLayout zlayout(chefsi_kpoint* h, int ns) {
  ZLayout L;
  size_t off = 0;
  L.bufB = off;
  off += align256((size_t)h->nd * ns * 16);
  L.alpha = off;
  off += align256((size_t)std::max(1, h->np_tot) * ns * 16);
  L.hs = off;
  off += align256((size_t)ns * ns * 16);
  L.ms = off;
  off += align256((size_t)ns * ns * 16);
  L.d = off;
  off += align256((size_t)ns * 8);
  L.e = off;
  off += align256((size_t)ns * 8);
  L.info = off;
  off += 256;
  L.kg = plan_blas_gram(h->nd, ns);
  L.partial = off;
  off += align256((size_t)L.kg.nparts * ns * ns * 16);
  L.solver = off;
  L.solver_bytes = zsolver_workspace(h, ns);
  off += align256(std::max<size_t>(L.solver_bytes, 256));
  L.total = off;
  return L;
}

template <typename T>
T* zat(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

template <typename T>
T* kupload(const T* src, size_t n) {
  T* d = nullptr;
  if (n == 0) return nullptr;
  if (no_memory(hipMalloc(&d, n * sizeof(T)))) throw Error{CHEFSI_ERR_OOM, "device allocation failed"};
  hipError_t e = hipMemcpy(d, src, n * sizeof(T), hipMemcpyHostToDevice);
  if (no_memory(e)) {
    (void)hipFree(d);
    throw Error{CHEFSI_ERR_HIP, std::string("upload: ") + hipGetErrorString(e)};
  }
  return d;
}

void krelease(chefsi_kpoint* h) {
  void* ptrs[] = {h->veff,     h->gdv,      h->reg_pt,   h->pt_idx,     h->pt_ent,   h->ent_ls, h->reg_slot,
                  h->slot_q,   h->slot_ent, h->gent_loc, h->q_slot_ptr, h->q_slot,   h->ent_chi, h->gent_chi,
                  h->partial};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  for (auto& p : h->ev_pending) {
    (void)hipEventDestroy(p.b);
    (void)hipEventDestroy(p.e);
  }
  for (auto ev : h->ev_pool) (void)hipEventDestroy(ev);
  if (h->pinned) (void)hipHostFree(h->pinned);
  if (h->blas) rocblas_destroy_handle(h->blas);
}

// k-point kernel classes timed by chefsi_kpoint_profile_*
enum KProfId { KP_ZHX = 0, KP_BAND = 1, KP_GRAM = 2, KP_EIG = 3, KP_ROT = 4 };
using KProfScope = ProfScopeT<chefsi_kpoint>;

ZNbArgs zband_args(const chefsi_kpoint* h, double2* y, int ns, const double2* alpha, double sa) {
  ZNbArgs b{};
  b.y = y;
  b.nd = h->nd;
  b.ns = ns;
  b.nreg = h->nreg;
  b.reg_pt = h->reg_pt;
  b.pt_idx = h->pt_idx;
  b.pt_ent = h->pt_ent;
  b.ent_ls = h->ent_ls;
  b.ent_chi = h->ent_chi;
  b.reg_slot = h->reg_slot;
  b.slot_q = h->slot_q;
  b.slot_ent = h->slot_ent;
  b.gent_loc = h->gent_loc;
  b.gent_chi = h->gent_chi;
  b.alpha = alpha;
  b.sa = sa;
  b.partial = h->partial;
  b.max_pts = h->max_pts;
  b.max_ent = h->max_ent;
  b.max_slots = h->max_slots;
  return b;
}

// out = sa ((H_k x) - sc x) + sb prev: stencil + Veff + recurrence, then the band pass adds
// sa V_nl x at the touched points (coefficients alpha of x: formed first by a gather-only
// pass unless alpha_ready) and, when want_next, leaves the coefficients of out in alpha.
void zapply(chefsi_kpoint* h, const double2* x, const double2* prev, double2* out, int ns, double sa, double sc,
            double sb, double2* alpha, hipStream_t s, bool alpha_ready = false, bool want_next = false) {
  if (h->np_tot > 0 && !alpha_ready) {
    KProfScope ps(h, KP_BAND, s);
    HIP_TRY(launch_zband(zband_args(h, const_cast<double2*>(x), ns, alpha, 0.0), false, true, s));
    HIP_TRY(launch_zband_reduce(h->partial, h->q_slot_ptr, h->q_slot, h->gdv, h->np_tot, ns, alpha, s));
    ps.done();
  }
  ZHxArgs a{};
  a.x = x;
  a.prev = prev;
  a.out = out;
  a.veff = h->veff;
  a.r = h->radius;
  a.nd = h->nd;
  double sumh = 0.0;
  for (int d = 0; d < 3; ++d) {
    a.n[d] = h->n[d];
    a.per[d] = h->bc[d] == 0;
    sumh += 1.0 / (h->h[d] * h->h[d]);
    const double th = h->bc[d] == 0 ? h->kvec[d] * h->n[d] * h->h[d] : 0.0;
    a.ph[d] = make_double2(std::cos(th), std::sin(th));
    for (int p = 0; p <= kMaxRadius; ++p) a.cw[d][p] = p <= h->radius ? -0.5 * h->w[p] / (h->h[d] * h->h[d]) : 0.0;
  }
  a.c0 = -0.5 * h->w[0] * sumh;
  a.sa = sa;
  a.sc = sc;
  a.sb = sb;
  {
    KProfScope ps(h, KP_ZHX, s);
    HIP_TRY(launch_zhx(a, ns, s));
    ps.done();
  }
  if (h->np_tot > 0) {
    KProfScope ps(h, KP_BAND, s);
    HIP_TRY(launch_zband(zband_args(h, out, ns, alpha, sa), true, want_next, s));
    if (want_next)
      HIP_TRY(launch_zband_reduce(h->partial, h->q_slot_ptr, h->q_slot, h->gdv, h->np_tot, ns, alpha, s));
    ps.done();
  }
}

template <typename F>
int kguarded(chefsi_kpoint* h, F&& f) {
  if (h == nullptr) return CHEFSI_ERR_INVALID_ARG;
  try {
    h->last_error.clear();
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != h->device) HIP_TRY(hipSetDevice(h->device));
    f();
    return CHEFSI_OK;
  } catch (const Error& e) {
    h->last_error = e.msg;
    return e.status;
  } catch (const std::bad_alloc&) {
    h->last_error = "host allocation failed";
    return CHEFSI_ERR_OOM;
  } catch (...) {
    h->last_error = "unexpected exception";
    return CHEFSI_ERR_HIP;
  }
}

void kcheck_call(chefsi_kpoint* h, int ns, void* ws, size_t ws_bytes, ZLayout& L) {
  check(ns >= 1 && ns <= h->max_ns, "ns must satisfy 1 <= ns <= max_ns");
  check((int64_t)ns <= h->nd, "ns must not exceed Nd");
  L = zlayout(h, ns);
  if (ws == nullptr || ws_bytes < L.total)
    throw Error{CHEFSI_ERR_WORKSPACE, "workspace smaller than chefsi_kpoint_workspace_bytes(ns)"};
  check(((uintptr_t)ws & 255) == 0, "workspace must be 256-byte aligned");
}

}  // namespace

extern "C" {

int chefsi_kpoint_create(const chefsi_grid_t* grid, const double* veff_host, const chefsi_nonlocal_t* nl,
                         const int32_t* supp_img, const double* kvec, int32_t max_ns, chefsi_kpoint_t** out) {
  if (out == nullptr) return CHEFSI_ERR_INVALID_ARG;
  *out = nullptr;
  if (grid == nullptr || veff_host == nullptr || kvec == nullptr) return CHEFSI_ERR_INVALID_ARG;
  chefsi_kpoint* h = nullptr;
  try {
    h = new chefsi_kpoint();
  } catch (...) {
    return CHEFSI_ERR_OOM;
  }
  try {
    check(grid->fd_order >= 2 && grid->fd_order <= 12 && grid->fd_order % 2 == 0, "fd_order must be even, 2..12");
    h->radius = grid->fd_order / 2;
    int64_t nd = 1;
    for (int d = 0; d < 3; ++d) {
      check(grid->n[d] >= 1, "grid sizes must be >= 1");
      check(grid->bc[d] == 0 || grid->bc[d] == 1, "bc must be 0 (periodic) or 1 (Dirichlet)");
      check(std::isfinite(grid->h[d]) && grid->h[d] > 0.0, "grid spacing must be positive");
      check(std::isfinite(kvec[d]), "k must be finite");
      if (grid->bc[d] == 0) check(grid->n[d] >= h->radius, "periodic direction needs n >= fd_order/2");
      h->n[d] = grid->n[d];
      h->h[d] = grid->h[d];
      h->bc[d] = grid->bc[d];
      h->kvec[d] = kvec[d];
      nd *= grid->n[d];
    }
    check(nd < (int64_t)1 << 31, "Nd must be below 2^31");
    check(max_ns >= 1 && (int64_t)max_ns <= nd && max_ns <= 65535, "max_ns must satisfy 1 <= max_ns <= min(Nd, 65535)");
    {
      const ZTiling zt = plan_zhx(grid->n[0], grid->n[1], grid->n[2], 1, grid->fd_order / 2);
      check(grid->n[0] <= kZMaxThreads && zt.kh <= 4 && zt.lds_bytes <= 96 * 1024,
            "grid too wide in x for the complex stencil tiling (halo values per thread above four)");
    }
    h->nd = nd;
    h->max_ns = max_ns;
    h->w = fd_weights(grid->fd_order);
    const double dv = grid->h[0] * grid->h[1] * grid->h[2];
    std::vector<double> veff(veff_host, veff_host + nd);
    for (double v : veff) check(std::isfinite(v), "Veff must be finite");

    std::vector<int> soff, sidx, nproj, poff, cnt, cols;
    std::vector<int64_t> coff;
    std::vector<double2> chi, vals;
    std::vector<double> gdv;
    if (nl != nullptr && nl->n_atoms > 0) {
      check(nl->supp_ptr && nl->supp_idx && nl->nproj && nl->chi && nl->gamma && supp_img, "null projector array");
      const int na = nl->n_atoms;
      const int64_t nsupp = nl->supp_ptr[na];
      check(nl->supp_ptr[0] == 0 && nsupp >= 0 && nsupp < (int64_t)1 << 31, "bad supp_ptr");
      double kl[3];
      for (int d = 0; d < 3; ++d) kl[d] = grid->bc[d] == 0 ? kvec[d] * grid->n[d] * grid->h[d] : 0.0;
      soff.resize(na + 1);
      coff.resize(na);
      poff.resize(na);
      nproj.assign(nl->nproj, nl->nproj + na);
      int64_t c = 0;
      int p = 0;
      for (int J = 0; J < na; ++J) {
        check(nl->supp_ptr[J + 1] >= nl->supp_ptr[J], "supp_ptr must be non-decreasing");
        check(nproj[J] >= 1, "nproj must be >= 1");
        soff[J] = (int)nl->supp_ptr[J];
        coff[J] = c;
        poff[J] = p;
        const int64_t nj = nl->supp_ptr[J + 1] - nl->supp_ptr[J];
        for (int64_t s = 0; s < nj; ++s) {
          const int64_t i = nl->supp_idx[nl->supp_ptr[J] + s];
          check(i >= 0 && i < nd, "support index outside the grid");
          if (s > 0) check(i > nl->supp_idx[nl->supp_ptr[J] + s - 1], "support indices must increase");
        }
        c += nj * nproj[J];
        p += nproj[J];
      }
      check(p < (1 << 30) && c < ((int64_t)1 << 31), "too many projectors");
      soff[na] = (int)nsupp;
      h->n_atoms = na;
      h->np_tot = p;
      sidx.assign(nl->supp_idx, nl->supp_idx + nsupp);
      // Bloch-phased projector values: chi~ = chi * exp(i k.(m L)), m the image of the point
      chi.resize(c);
      for (int J = 0; J < na; ++J) {
        const int64_t nj = nl->supp_ptr[J + 1] - nl->supp_ptr[J];
        for (int64_t s = 0; s < nj; ++s) {
          const int64_t g = nl->supp_ptr[J] + s;
          double th = 0.0;
          for (int d = 0; d < 3; ++d) th += kl[d] * supp_img[3 * g + d];
          const double cr = std::cos(th), ci = std::sin(th);
          for (int a = 0; a < nproj[J]; ++a) {
            const double v = nl->chi[coff[J] + a * nj + s];
            check(std::isfinite(v), "chi must be finite");
            chi[coff[J] + a * nj + s] = make_double2(v * cr, v * ci);
          }
        }
      }
      gdv.resize(p);
      for (int q = 0; q < p; ++q) {
        check(std::isfinite(nl->gamma[q]), "gamma must be finite");
        gdv[q] = nl->gamma[q] * dv;
      }
      // point-major entries: grid points in increasing order, atoms in order
      cnt.assign(nd + 1, 0);
      for (int J = 0; J < na; ++J)
        for (int64_t s = nl->supp_ptr[J]; s < nl->supp_ptr[J + 1]; ++s) cnt[sidx[s] + 1] += nproj[J];
      for (int64_t i = 0; i < nd; ++i) cnt[i + 1] += cnt[i];
      const int64_t nent = cnt[nd];
      std::vector<int> fill(cnt.begin(), cnt.end() - 1);
      cols.resize(nent);
      vals.resize(nent);
      for (int J = 0; J < na; ++J) {
        const int64_t nj = nl->supp_ptr[J + 1] - nl->supp_ptr[J];
        for (int64_t s = 0; s < nj; ++s) {
          const int i = sidx[nl->supp_ptr[J] + s];
          for (int a = 0; a < nproj[J]; ++a) {
            const int pos = fill[i]++;
            cols[pos] = poff[J] + a;
            vals[pos] = chi[coff[J] + a * nj + s];
          }
        }
      }
      check(nent < ((int64_t)1 << 31), "too many projector entries");
    }

    HIP_TRY(hipGetDevice(&h->device));
    BLAS_TRY(rocblas_create_handle(&h->blas));
    BLAS_TRY(rocblas_set_atomics_mode(h->blas, rocblas_atomics_not_allowed));
    if (no_memory(hipHostMalloc((void**)&h->pinned, (size_t)max_ns * sizeof(double) + 64, hipHostMallocDefault))) {
      h->pinned = nullptr;
      throw Error{CHEFSI_ERR_OOM, "pinned host allocation failed"};
    }
    h->veff = kupload(veff.data(), veff.size());
    if (h->np_tot > 0) {
      // band-pass regions of the touched points (the real path's tables with chi~ values)
      const BandRegions R = band_regions(nd, cnt.data(), cols.data(), h->np_tot, kZBandThreads, kZBandMaxEnt);
      std::vector<double2> gent_chi(R.gent_src.size());
      for (size_t e = 0; e < gent_chi.size(); ++e) {
        const double2 v = vals[R.gent_src[e]];
        gent_chi[e] = make_double2(v.x, -v.y);
      }
      h->nreg = (int)R.reg_pt.size() - 1;
      h->n_pts = (int)R.pt_idx.size();
      for (int i = 0; i < h->nreg; ++i) {
        const int p0 = R.reg_pt[i], p1 = R.reg_pt[i + 1];
        h->max_pts = std::max(h->max_pts, p1 - p0);
        h->max_ent = std::max(h->max_ent, R.pt_ent[p1] - R.pt_ent[p0]);
        h->max_slots = std::max(h->max_slots, R.reg_slot[i + 1] - R.reg_slot[i]);
      }
      h->gdv = kupload(gdv.data(), gdv.size());
      h->reg_pt = kupload(R.reg_pt.data(), R.reg_pt.size());
      h->pt_idx = kupload(R.pt_idx.data(), R.pt_idx.size());
      h->pt_ent = kupload(R.pt_ent.data(), R.pt_ent.size());
      h->ent_ls = kupload(R.ent_ls.data(), R.ent_ls.size());
      h->ent_chi = kupload(vals.data(), vals.size());
      h->reg_slot = kupload(R.reg_slot.data(), R.reg_slot.size());
      h->slot_q = kupload(R.slot_q.data(), R.slot_q.size());
      h->slot_ent = kupload(R.slot_ent.data(), R.slot_ent.size());
      h->gent_loc = kupload(R.gent_loc.data(), R.gent_loc.size());
      h->gent_chi = kupload(gent_chi.data(), gent_chi.size());
      h->q_slot_ptr = kupload(R.q_slot_ptr.data(), R.q_slot_ptr.size());
      h->q_slot = kupload(R.q_slot.data(), R.q_slot.size());
      if (no_memory(hipMalloc((void**)&h->partial,
                              std::max<size_t>(1, R.slot_q.size()) * (size_t)max_ns * sizeof(double2)))) {
        h->partial = nullptr;
        throw Error{CHEFSI_ERR_OOM, "device allocation failed (band-pass partial sums)"};
      }
    }
    *out = h;
    return CHEFSI_OK;
  } catch (const Error& e) {
    krelease(h);
    delete h;
    return e.status;
  } catch (...) {
    krelease(h);
    delete h;
    return CHEFSI_ERR_OOM;
  }
}

void chefsi_kpoint_destroy(chefsi_kpoint_t* h) {
  if (h == nullptr) return;
  (void)hipSetDevice(h->device);
  krelease(h);
  delete h;
}

const char* chefsi_kpoint_last_error(const chefsi_kpoint_t* h) { return h ? h->last_error.c_str() : ""; }

int chefsi_kpoint_profile_enable(chefsi_kpoint_t* h, int32_t on) {
  return kguarded(h, [&] { h->prof_on = on != 0; });
}

int chefsi_kpoint_profile_reset(chefsi_kpoint_t* h) {
  return kguarded(h, [&] {
    prof_collect(h);
    for (int i = 0; i < kNumProf; ++i) {
      h->prof_ms[i] = 0.0;
      h->prof_n[i] = 0;
    }
  });
}

int chefsi_kpoint_profile_read(chefsi_kpoint_t* h, int32_t kernel_id, double* total_ms, int64_t* launches) {
  return kguarded(h, [&] {
    check(kernel_id >= 0 && kernel_id <= KP_ROT, "kernel_id out of range");
    prof_collect(h);
    if (total_ms) *total_ms = h->prof_ms[kernel_id];
    if (launches) *launches = h->prof_n[kernel_id];
  });
}

int chefsi_kpoint_workspace_bytes(chefsi_kpoint_t* h, int32_t ns, size_t* bytes) {
  return kguarded(h, [&] {
    check(bytes != nullptr, "null pointer");
    check(ns >= 1 && ns <= h->max_ns, "ns must satisfy 1 <= ns <= max_ns");
    *bytes = zlayout(h, ns).total;
  });
}

int chefsi_kpoint_apply_h(chefsi_kpoint_t* h, const void* X, void* Y, int32_t ns, void* ws, size_t ws_bytes,
                          void* stream) {
  return kguarded(h, [&] {
    check(X != nullptr && Y != nullptr, "null pointer");
    check(X != Y, "X and Y must not alias");
    ZLayout L;
    kcheck_call(h, ns, ws, ws_bytes, L);
    zapply(h, (const double2*)X, nullptr, (double2*)Y, ns, 1.0, 0.0, 0.0, zat<double2>(ws, L.alpha),
           (hipStream_t)stream);
  });
}

int chefsi_kpoint_step(chefsi_kpoint_t* h, void* X, int32_t ns, int32_t degree, double lam_lo, double lam_cut,
                       double lam_hi, void* ws, size_t ws_bytes, void* stream, double* ritz_host) {
  return kguarded(h, [&] {
    check(X != nullptr, "X is NULL");
    check(degree >= 1, "degree must be >= 1");
    check_bounds(lam_lo, lam_cut, lam_hi);
    ZLayout L;
    kcheck_call(h, ns, ws, ws_bytes, L);
    hipStream_t s = (hipStream_t)stream;
    double2* A = (double2*)X;
    double2* B = zat<double2>(ws, L.bufB);
    double2* alpha = zat<double2>(ws, L.alpha);
    double2* Hs = zat<double2>(ws, L.hs);
    double2* Ms = zat<double2>(ws, L.ms);
    double* D = zat<double>(ws, L.d);
    rocblas_int* info = zat<rocblas_int>(ws, L.info);
    // scaled Chebyshev filter (Alg. 1, Filtering), the same scalars as the real path
    const double c = 0.5 * (lam_hi + lam_cut);
    const double e = 0.5 * (lam_hi - lam_cut);
    const double s1 = e / (lam_lo - c);
    double sig = s1;
    // the projector coefficients of each output are left by its band pass for the next
    // application
    zapply(h, A, nullptr, B, ns, s1 / e, c, 0.0, alpha, s, false, true);
    double2* cur = B;
    double2* other = A;
    for (int k = 1; k < degree; ++k) {
      const double sig_next = 1.0 / (2.0 / s1 - sig);
      zapply(h, cur, other, other, ns, 2.0 * sig_next / e, c, -sig * sig_next, alpha, s, true, true);
      std::swap(cur, other);
      sig = sig_next;
    }
    double2* Xf = cur;
    double2* Yf = other;
    zapply(h, Xf, nullptr, Yf, ns, 1.0, 0.0, 0.0, alpha, s, true, false);  // Y~ = H X~
    // projection (upper triangles made Hermitian)
    const rocblas_double_complex one(1.0, 0.0), zero(0.0, 0.0);
    const rocblas_int ld = (rocblas_int)h->nd;
    BLAS_TRY(rocblas_set_stream(h->blas, s));
    BLAS_TRY(rocblas_set_workspace(h->blas, zat<void>(ws, L.solver), std::max<size_t>(L.solver_bytes, 256)));
    auto zc = [](const double2* p) { return reinterpret_cast<const rocblas_double_complex*>(p); };
    auto zm = [](double2* p) { return reinterpret_cast<rocblas_double_complex*>(p); };
    // split-K: K chunks as one strided batch of products, partials summed in a fixed order
    double2* part = zat<double2>(ws, L.partial);
    const BlasGram& kg = L.kg;
    // upper triangle only, by the real path's column blocks: block row q of every partial
    // against columns [start_q, ns)
    auto gram = [&](const double2* A, const double2* Bm, double2* C) {
      for (int q = 0; q < kg.nblk; ++q) {
        const int r0 = kg.start[q], m = kg.start[q + 1] - r0, n = ns - r0;
        const double2* Aq = A + (size_t)r0 * h->nd;
        const double2* Bq = Bm + (size_t)r0 * h->nd;
        double2* Pq = part + r0 + (size_t)r0 * ns;
        BLAS_TRY(rocblas_zgemm_strided_batched(h->blas, rocblas_operation_conjugate_transpose,
                                               rocblas_operation_none, m, n, (rocblas_int)kg.kc, &one, zc(Aq), ld,
                                               kg.kc, zc(Bq), ld, kg.kc, &zero, zm(Pq), ns, (rocblas_stride)ns * ns,
                                               kg.splits));
        if (kg.tail > 0) {
          const int64_t k0 = kg.kc * kg.splits;
          BLAS_TRY(rocblas_zgemm(h->blas, rocblas_operation_conjugate_transpose, rocblas_operation_none, m, n,
                                 (rocblas_int)kg.tail, &one, zc(Aq + k0), ld, zc(Bq + k0), ld, &zero,
                                 zm(Pq + (size_t)kg.splits * ns * ns), ns));
        }
      }
      HIP_TRY(launch_zsum_partials(part, kg.nparts, ns, C, s));
    };
    {
      KProfScope ps(h, KP_GRAM, s);
      gram(Xf, Yf, Hs);
      gram(Xf, Xf, Ms);
      ps.done();
    }
    // Hermitian-definite eigenproblem (Alg. 1, Diagonalization)
    KProfScope pe(h, KP_EIG, s);
    BLAS_TRY(rocsolver_zpotrf(h->blas, rocblas_fill_upper, ns, zm(Ms), ns, info));
    BLAS_TRY(rocblas_ztrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_conjugate_transpose,
                           rocblas_diagonal_non_unit, ns, ns, &one, zc(Ms), ns, zm(Hs), ns));
    BLAS_TRY(rocblas_ztrsm(h->blas, rocblas_side_right, rocblas_fill_upper, rocblas_operation_none,
                           rocblas_diagonal_non_unit, ns, ns, &one, zc(Ms), ns, zm(Hs), ns));
    BLAS_TRY(rocsolver_zheevd(h->blas, rocblas_evect_original, rocblas_fill_upper, ns, zm(Hs), ns, D,
                              zat<double>(ws, L.e), info + 1));
    BLAS_TRY(rocblas_ztrsm(h->blas, rocblas_side_left, rocblas_fill_upper, rocblas_operation_none,
                           rocblas_diagonal_non_unit, ns, ns, &one, zc(Ms), ns, zm(Hs), ns));
    pe.done();
    KProfScope pr(h, KP_ROT, s);
    // rotation (Alg. 1, Rotation): X = X~ Z into the buffer Y~ held, in row panels of fewer
    // than 2^31 output elements each (blocks of any size)
    const int64_t prow = std::max<int64_t>(1, std::min<int64_t>(h->nd, (((int64_t)1 << 31) - 1) / ns));
    for (int64_t r0 = 0; r0 < h->nd; r0 += prow) {
      const rocblas_int m = (rocblas_int)std::min<int64_t>(prow, h->nd - r0);
      BLAS_TRY(rocblas_zgemm(h->blas, rocblas_operation_none, rocblas_operation_none, m, ns, ns, &one, zc(Xf + r0),
                             ld, zc(Hs), ns, &zero, zm(Yf + r0), ld));
    }
    if (Yf != A) HIP_TRY(hipMemcpyAsync(A, Yf, (size_t)h->nd * ns * 16, hipMemcpyDeviceToDevice, s));
    pr.done();
    double* d = h->pinned;
    rocblas_int* inf = reinterpret_cast<rocblas_int*>(h->pinned + h->max_ns);
    HIP_TRY(hipMemcpyAsync(d, D, (size_t)ns * 8, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(inf, info, 2 * sizeof(rocblas_int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (inf[0] > 0) throw Error{CHEFSI_ERR_NOT_POSDEF, "Cholesky of the overlap matrix failed"};
    if (inf[1] > 0) throw Error{CHEFSI_ERR_EIG, "dense eigensolver did not converge"};
    for (int i = 0; i < ns; ++i)
      if (!std::isfinite(d[i])) throw Error{CHEFSI_ERR_NONFINITE, "non-finite Ritz value"};
    if (ritz_host) std::memcpy(ritz_host, d, (size_t)ns * 8);
  });
}

}  // extern "C"
