// Trilinear sampling of a scalar image at p = x + T(x) with its analytic
// gradient: the image side of the SSD registration step.
//
// p is formed in FP32 (the precision that decides the cell); corners on voxel
// centres, p clamped to [0, n-1]; at an exact integer p the cell [p, p+1] is
// used; a coordinate on or beyond the border (p <= 0 or p >= n-1) gets zero
// gradient.
#pragma once

#include "bsi_device.h"

namespace bsi {

struct Axis {
  int i0, i1;
  float f;
  float in;  // 1 where p is strictly inside (0, n-1), else 0
};

__device__ __forceinline__ Axis sample_axis(float p, int n) {
  Axis a;
  const float top = (float)(n - 1), last = (float)max(n - 2, 0);
  a.in = (p > 0.f && p < top) ? 1.f : 0.f;
  const float pc = __builtin_amdgcn_fmed3f(p, 0.f, top);  // NaN -> 0
  const float fl = fminf(floorf(pc), last);               // (n <= 2^20: exact)
  a.i0 = (int)fl;
  a.i1 = min(a.i0 + 1, n - 1);
  a.f = pc - fl;
  return a;
}

// Two consecutive floats, 4-byte aligned.
struct __attribute__((packed, aligned(4))) F2 {
  float x, y;
};
__device__ __forceinline__ F2 ldf2(const float* p) { return *reinterpret_cast<const F2*>(p); }

struct Sample {
  float w;            // interpolated value
  float gx, gy, gz;   // dW/dp, masked at the border
};

// The sample in two halves, so that a caller can issue the loads of one
// sample before it finishes the previous one: trilinear_load forms the cell
// and loads its 8 corners, trilinear_finish interpolates.
struct SampleIn {
  float c000, c001, c010, c011, c100, c101, c110, c111;  // corners, x fastest
  float fx, fy, fz;                                      // offsets in the cell
  float inx, iny, inz;                                   // 1 strictly inside, else 0
};

// Pairs: 1 when the caller guarantees nx >= 2 (x-neighbours as one 8-byte load), 0 when
// nx == 1.
template <int Pairs>
__device__ __forceinline__ SampleIn trilinear_load(const float* __restrict__ img, int nx, int ny, int nz, float px,
                                                   float py, float pz) {
  const Axis ax = sample_axis(px, nx), ay = sample_axis(py, ny), az = sample_axis(pz, nz);
  const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
  const float* p00 = img + az.i0 * sz + ay.i0 * sy;
  const float* p01 = img + az.i0 * sz + ay.i1 * sy;
  const float* p10 = img + az.i1 * sz + ay.i0 * sy;
  const float* p11 = img + az.i1 * sz + ay.i1 * sy;
  SampleIn s;
  if constexpr (Pairs == 1) {
    // i1 = i0 + 1: each pair of x-neighbours is one 8-byte load
    const F2 q00 = ldf2(p00 + ax.i0), q01 = ldf2(p01 + ax.i0);
    const F2 q10 = ldf2(p10 + ax.i0), q11 = ldf2(p11 + ax.i0);
    s.c000 = q00.x, s.c001 = q00.y, s.c010 = q01.x, s.c011 = q01.y;
    s.c100 = q10.x, s.c101 = q10.y, s.c110 = q11.x, s.c111 = q11.y;
  } else {
    s.c000 = s.c001 = p00[0];
    s.c010 = s.c011 = p01[0];
    s.c100 = s.c101 = p10[0];
    s.c110 = s.c111 = p11[0];
  }
  s.fx = ax.f, s.fy = ay.f, s.fz = az.f;
  s.inx = ax.in, s.iny = ay.in, s.inz = az.in;
  return s;
}

__device__ __forceinline__ Sample trilinear_finish(const SampleIn& c) {
  const float fx = c.fx, fy = c.fy, fz = c.fz;
  // interpolate along x, then y, then z
  const float x00 = fmaf(fx, c.c001 - c.c000, c.c000), x01 = fmaf(fx, c.c011 - c.c010, c.c010);
  const float x10 = fmaf(fx, c.c101 - c.c100, c.c100), x11 = fmaf(fx, c.c111 - c.c110, c.c110);
  const float y0 = fmaf(fy, x01 - x00, x00), y1 = fmaf(fy, x11 - x10, x10);
  Sample s;
  s.w = fmaf(fz, y1 - y0, y0);
  // analytic derivatives of the trilinear form
  const float dx00 = c.c001 - c.c000, dx01 = c.c011 - c.c010, dx10 = c.c101 - c.c100, dx11 = c.c111 - c.c110;
  const float dx0 = fmaf(fy, dx01 - dx00, dx00), dx1 = fmaf(fy, dx11 - dx10, dx10);
  s.gx = fmaf(fz, dx1 - dx0, dx0) * c.inx;
  s.gy = fmaf(fz, (x11 - x10) - (x01 - x00), x01 - x00) * c.iny;
  s.gz = (y1 - y0) * c.inz;
  return s;
}

// trilinear_load for an image below 4 GiB: one 32-bit lane offset, and the cell's
// other rows from base addresses at the uniform distances sy and sz (bytes to the
// next row and plane; 0 along an axis of one voxel, whose corners coincide).  Global
// loads: through a buffer resource the same gathers, which seldom start on 8 bytes,
// took longer (warp of 303 x 167 x 212 72 us against 62; fused step of 256 x 256 x 160 at
// rough displacements 72 against 67).  The same operations on the same values as
// trilinear_load.  Pairs as there.
template <int Pairs>
__device__ __forceinline__ SampleIn trilinear_load_small(const float* __restrict__ img, int nx, int ny, int nz,
                                                         uint32_t sy, uint32_t sz, float px, float py, float pz) {
  const Axis ax = sample_axis(px, nx), ay = sample_axis(py, ny), az = sample_axis(pz, nz);
  const uint32_t o = (((uint32_t)az.i0 * (uint32_t)ny + (uint32_t)ay.i0) * (uint32_t)nx + (uint32_t)ax.i0) * 4u;
  const char* p00 = reinterpret_cast<const char*>(img);
  const char *p01 = p00 + sy, *p10 = p00 + sz, *p11 = p10 + sy;
  SampleIn s;
  if constexpr (Pairs == 1) {
    const F2 q00 = *reinterpret_cast<const F2*>(p00 + o), q01 = *reinterpret_cast<const F2*>(p01 + o);
    const F2 q10 = *reinterpret_cast<const F2*>(p10 + o), q11 = *reinterpret_cast<const F2*>(p11 + o);
    s.c000 = q00.x, s.c001 = q00.y, s.c010 = q01.x, s.c011 = q01.y;
    s.c100 = q10.x, s.c101 = q10.y, s.c110 = q11.x, s.c111 = q11.y;
  } else {
    s.c000 = s.c001 = *reinterpret_cast<const float*>(p00 + o);
    s.c010 = s.c011 = *reinterpret_cast<const float*>(p01 + o);
    s.c100 = s.c101 = *reinterpret_cast<const float*>(p10 + o);
    s.c110 = s.c111 = *reinterpret_cast<const float*>(p11 + o);
  }
  s.fx = ax.f, s.fy = ay.f, s.fz = az.f;
  s.inx = ax.in, s.iny = ay.in, s.inz = az.in;
  return s;
}

// A volume sampled voxel by voxel: thread t of workgroup item (pb, zb) owns the
// voxel column p = pb kColThreads + t of the plane, p = y nx + x, and takes it
// through the planes [zb zchunk, (zb + 1) zchunk).  Columns run on over the ends
// of the rows, so that every lane is used at any width, the position in the row is
// found once per column, and the two image planes of a voxel's cell are the next
// voxel's too.
constexpr int kColThreads = 256;
struct ColLaunch {
  int npb, nzb, zchunk;  // column blocks, z-chunks, planes per chunk
};
// kColPlanes planes per column: short workgroups in the order of the planes, so
// that what is read and written at any moment is one compact range of addresses
// (SSD at 512 x 400 x 220: 332 us, against 358 with planes for 2048 workgroups).
constexpr int kColPlanes = 4;
inline ColLaunch make_col_launch(const VolGeom& g) {
  const int64_t columns = (int64_t)g.nx * g.ny;
  ColLaunch c;
  c.npb = (int)((columns + kColThreads - 1) / kColThreads);
  c.zchunk = kColPlanes;
  c.nzb = (g.nz + kColPlanes - 1) / kColPlanes;
  return c;
}

}  // namespace bsi
