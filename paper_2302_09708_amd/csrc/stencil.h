// Device helpers of the z-marching stencil kernels (hx_apply, kinetic stress): buffer
// resources and loads, plane and row offsets with periodic wrap or Dirichlet zeros, and the
// list of values a block stages per plane besides its own rows.
#pragma once

#include "common.h"

namespace chefsi {

constexpr unsigned kOOB = 0x80000000u;  // any buffer offset at or past the end reads as zero

__device__ __forceinline__ int wrap_index(int v, int n) {
  v %= n;
  return v < 0 ? v + n : v;
}

// Offset of row gy inside a plane (x added), or -1 for a Dirichlet zero row.
__device__ __forceinline__ int row_offset(int x, int gy, int nx, int ny, int per_y) {
  if (per_y) return x + nx * wrap_index(gy, ny);
  return (gy < 0 || gy >= ny) ? -1 : x + nx * gy;
}

// Offset of plane pz, or -1 for a Dirichlet zero plane.
__device__ __forceinline__ int plane_offset(int pz, int nplane, int nz, int per_z) {
  if (per_z) return nplane * wrap_index(pz, nz);
  return (pz < 0 || pz >= nz) ? -1 : nplane * pz;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Buffer loads take a per-lane byte offset (voff) and a wave-uniform one (soff, a scalar
// register): the per-thread part of an address is computed once, the per-plane part on
// the scalar unit, so a load costs no vector instructions.  A lane whose voff is kOOB
// reads zero (kOOB + soff stays at or past the end because every buffer is below 2^31
// bytes and so is soff).
template <typename T>
__device__ __forceinline__ unsigned lane_off(int a) {
  return a < 0 ? kOOB : (unsigned)a * (unsigned)sizeof(T);
}

template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff);
template <>
__device__ __forceinline__ double bload<double>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float bload<float>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// element at lane offset voff of plane po (element offset, uniform) of the nbytes-long
// array at p; po = -1 (a zero plane) selects a resource with no records: reads give zero
template <typename T>
__device__ __forceinline__ T pload(const T* p, int nbytes, unsigned voff, int po) {
  const __amdgpu_buffer_rsrc_t r = make_rsrc(p, po < 0 ? 0 : nbytes);
  return bload<T>(r, voff, po < 0 ? 0u : (unsigned)po * (unsigned)sizeof(T));
}

// Number of LDS slots a block stages per plane besides its own body elements: the r halo
// rows above and below the tile (nx + 2r columns when x is periodic, the nx interior
// columns when it is not) and, when x is periodic, the r wrapped copies on each side of
// every body row.  (Dirichlet x halo columns are zeros written once.)
__host__ __device__ inline int hx_halo_slots(int nx, int ty, int radius, int per_x) {
  return 2 * radius * (per_x ? nx + 2 * radius : nx) + (per_x ? ty * 2 * radius : 0);
}

// Slot e of a plane's staged set: LDS destination (row-major with the given pitch, element
// x of a row at column r + x) and source row offset inside the plane (x added; -1 for a
// zero value).
__device__ __forceinline__ void halo_slot(int e, int nx, int ny, int ty, int y0, int radius, int pitch, int per_x,
                                          int per_y, int& dst, int& src) {
  const int w = per_x ? nx + 2 * radius : nx;
  int yy, c;
  if (e < 2 * radius * w) {  // halo rows: local rows [0, r) and [r + ty, ty + 2r)
    const int hr = e / w;
    c = e % w + (per_x ? 0 : radius);
    yy = hr < radius ? hr : hr + ty;
  } else {  // periodic x copies of the body rows: columns [0, r) and [r + nx, nx + 2r)
    const int f = e - 2 * radius * w;
    const int cc = f % (2 * radius);
    c = cc < radius ? cc : nx + cc;
    yy = radius + f / (2 * radius);
  }
  int gx = c - radius;
  if (gx < 0) gx += nx;  // only reached with periodic x (nx >= r: one wrap)
  if (gx >= nx) gx -= nx;
  dst = yy * pitch + c;
  src = row_offset(gx, y0 - radius + yy, nx, ny, per_y);
}

}  // namespace chefsi
