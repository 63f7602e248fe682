// Real-spacing grid: the exact window-start decision shared by host and
// device, and the geometry of the adjoint's bricks (used by the kernels in
// general.hip and by the host index checker).
#pragma once

#include <cmath>

#include "adjoint_device.h"
#include "bsi_internal.h"

namespace bsi {

// a + b = s + e exactly (Knuth's two-sum; round to nearest, no overflow).
__host__ __device__ inline void two_sum(float a, float b, float& s, float& e) {
  s = a + b;
  const float bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// Exact sign of D(i) = (x - o) - i s for integers 0 <= x, |i| < 2^24, and the
// FP32 value of D rounded from its exact expansion.  x - o = A + a and i s =
// P + p are error-free; growing the nonoverlapping expansion (a, A) by -p and
// then by -P (Shewchuk's grow-expansion) gives four nonoverlapping components
// whose largest nonzero one carries the sign of the exact sum.
__host__ __device__ inline int gen_residual(float X, float o, float s, int i, float& D) {
  float A, a;
  two_sum(X, -o, A, a);
  const float I = (float)i;
  const float P = I * s;
  const float p = fmaf(I, s, -P);
  float Q, h0, h1, k0, k1, k2;
  two_sum(-p, a, Q, h0);
  two_sum(Q, A, Q, h1);
  const float h2 = Q;
  two_sum(-P, h0, Q, k0);
  two_sum(Q, h1, Q, k1);
  two_sum(Q, h2, Q, k2);
  const float k3 = Q;
  D = k3 + k2;
  const float top = k3 != 0.f ? k3 : k2 != 0.f ? k2 : k1 != 0.f ? k1 : k0;
  return top > 0.f ? 1 : top < 0.f ? -1 : 0;
}

// Window start i = floor((v - o)/s) of voxel v (exact) and u = (v - o)/s - i
// in FP32.  The FP32 quotient is within 1/8 of the exact one for v < 2^21, so
// the floor is its floor, one below or one above; the exact residual decides.
__host__ __device__ inline int gen_locate(const GenAxis& a, int v, float& u) {
  const float X = (float)v;
  int i = (int)floorf((X - a.o) / a.s);
  float D;
  if (gen_residual(X, a.o, a.s, i, D) < 0) {
    --i;
    (void)gen_residual(X, a.o, a.s, i, D);
  } else {
    float D1;
    if (gen_residual(X, a.o, a.s, i + 1, D1) >= 0) {
      ++i;
      D = D1;
    }
  }
  u = D / a.s;
  return i;
}

__host__ __device__ inline int gen_tile(const GenAxis& a, int v) {
  float u;
  return gen_locate(a, v, u);
}


constexpr int kGenMaxZ = 256;  // the forward's voxel planes per workgroup (z table in LDS)

// ---------------------------------------------------------------------------
// The adjoint over the aligned adjoint's cells and bricks (adjoint_device.h), with
// per-axis tables in place of equal tiles.
// i(v) of every voxel (tile), B_0 .. B_3 at u(v) (w), and min{v : i(v) >= k} (first).
struct GenTiles {
  const int *tx, *ty;
  __host__ __device__ int x(int v) const { return tx[v]; }
  __host__ __device__ int y(int v) const { return ty[v]; }
};

// Brick id: whole z-tiles [bz k, (bz + 1) k) of the g - 3 that hold voxels.
__host__ __device__ inline AdjBrick gen_brick(const AdjGeom& a, const GenTiles& t, const int* first_z, int id) {
  const VolGeom& g = a.g;
  AdjBrick b;
  const int bx = id % a.x.nb, r = id / a.x.nb, by = r % a.y.nb, bz = r / a.y.nb;
  b.x0 = adj_brick_begin(a.x, g.nx, bx);
  b.xe = adj_brick_begin(a.x, g.nx, bx + 1);
  b.y0 = adj_brick_begin(a.y, g.ny, by);
  b.ye = adj_brick_begin(a.y, g.ny, by + 1);
  b.cz0 = bz * a.z.k;
  b.z0 = first_z[b.cz0];
  b.ze = first_z[imin(b.cz0 + a.z.k, g.gz - 3)];
  b.cx0 = t.x(b.x0);
  b.cy0 = t.y(b.y0);
  b.Cx = t.x(b.xe - 1) - b.cx0 + 4;
  b.Cy = t.y(b.ye - 1) - b.cy0 + 4;
  return b;
}
// Its control planes: every tile holds a voxel (s >= 1).
__host__ __device__ inline int gen_brick_cz(const AdjGeom& a, const AdjBrick& b) {
  return imin(a.z.k, a.g.gz - 3 - b.cz0) + 3;
}

// Largest control window of w consecutive voxels: their starts span at most
// ceil((w - 1) / s) tiles (exact in FP64: s has 24 bits).
inline int gen_window(const GenAxis& x, int w) { return imin((int)std::ceil((w - 1) / (double)x.s) + 4, x.g); }

// Cells of up to 32 voxels in x, as many as a window of 16 control points takes (s
// >= 2.59: 32), evenly wide where narrower.  A pure function of the geometry.
inline AdjGeom make_gen_adj(const GenGeom& q, const VolGeom& vol) {
  AdjGeom a;
  a.g = vol;
  a.g.dx = (int)std::ceil(q.x.s);  // bounds, for adj_gather_lx; the z axis counts tiles
  a.g.dy = (int)std::ceil(q.y.s);
  a.g.dz = 1;
  a.cell = imin(kAdjCellX, (int)(12. * q.x.s) + 1);
  if (a.cell < kAdjCellX) {
    const int nb = (q.x.n + kAdjCellsX * a.cell - 1) / (kAdjCellsX * a.cell);
    a.cell = (q.x.n + nb * kAdjCellsX - 1) / (nb * kAdjCellsX);
  }
  a.cw = (gen_window(q.x, imin(a.cell, q.x.n)) + 3) / 4 * 4;
  a.ch = gen_window(q.y, imin(kAdjCellY, q.y.n));
  auto axis = [](int units, int u, int k, int cm) {
    AdjAxis x;
    x.u = u;
    x.U = units;
    x.k = imin(k, units);
    x.nb = (units + x.k - 1) / x.k;
    x.w = x.k * u;
    x.md = 0;
    x.mw = (int64_t)units * u * x.w < ((int64_t)1 << 32) ? adj_magic(x.w) : 0;
    x.cm = cm;
    return x;
  };
  a.x = axis(q.x.n, 1, kAdjCellsX * a.cell, gen_window(q.x, imin(kAdjCellsX * a.cell, q.x.n)));
  a.y = axis(q.y.n, 1, kAdjCellsY * kAdjCellY, gen_window(q.y, imin(kAdjCellsY * kAdjCellY, q.y.n)));
  const int tiles = q.z.g - 3;  // z-tiles holding voxels
  const AdjDepth depth = adj_depth(a, tiles, q.z.s);
  auto set_depth = [&](int k) {
    a.z = axis(tiles, 1, k, imin(k, tiles) + 3);  // in tiles
    a.slots = a.z.cm <= depth.fit + 3 ? a.z.cm : 2;
  };
  set_depth(depth.best);
  if (a.z.k < depth.most && adj_workspace_bytes(a) > kAdjShallowBytes) set_depth(depth.most);
  a.part_bytes = adj_workspace_bytes(a) <= kAdjGatherSmall ? (uint32_t)adj_workspace_bytes(a) : 0;
  a.lx = adj_gather_lx(a);
  return a;
}

// The voxel whose table entries lane (q, m) reads for voxel v of a cell's n from v0 on an
// axis of `size` voxels; a cell past the volume (n = 0) reads the last one's.
__host__ __device__ inline int gen_weight_voxel(int v0, int n, int v, int size) {
  return imin(v0 + imax(0, imin(v, n - 1)), size - 1);
}

// Pass 2: the bricks whose voxels meet the support [first(c - 3), first(c + 1)) of
// control index c, along z those of tiles c - 3 .. c that hold voxels.
struct GenMap {
  const AdjGeom& a;
  const int *tx, *ty, *fx, *fy;
  __host__ __device__ AdjSpan span(const AdjAxis& x, const int* first, int c) const {
    return AdjSpan{adj_brick_of_voxel(x, first[c >= 3 ? c - 3 : 0]), adj_brick_of_voxel(x, first[c + 1] - 1)};
  }
  __host__ __device__ AdjSpan span_x(int c) const { return span(a.x, fx, c); }
  __host__ __device__ AdjSpan span_y(int c) const { return span(a.y, fy, c); }
  __host__ __device__ AdjSpan span_z(int c) const {
    return AdjSpan{adj_brick_of_voxel(a.z, imax(0, c - 3)), adj_brick_of_voxel(a.z, imin(c, a.g.gz - 4))};
  }
  // (a brick past the axis, whose term is not used, reads the last voxel's tile)
  __host__ __device__ size_t part_x(int b, int c) const {
    return b * adj_brick_stride(a) + (c - tx[imin(b * a.x.w, a.g.nx - 1)]) * 3;
  }
  __host__ __device__ size_t part_y(int b, int c) const {
    return b * (a.x.nb * adj_brick_stride(a)) + (c - ty[imin(b * a.y.w, a.g.ny - 1)]) * a.x.cm * 3;
  }
  __host__ __device__ size_t part_z(int b, int c) const {
    return b * ((size_t)a.y.nb * a.x.nb * adj_brick_stride(a)) + (c - b * a.z.k) * (a.y.cm * a.x.cm * 3);
  }
};

}  // namespace bsi
