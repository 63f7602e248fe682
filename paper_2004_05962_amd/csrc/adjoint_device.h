// Adjoint of Eq. 1 (its transpose), as a deterministic two-pass gather.
//
// Pass 1, z-first.  A brick is 2 x 2 cells in x and y by a run of whole
// z-tiles; a cell is 32 x 8 voxel columns (13 or 16 x 8 at x spacings 1 and 2, adj_cell,
// with other lanes, kAdjSteps) and belongs to one wave.  Lane (h, v) = (lane / 32, lane % 32) of
// the wave owns voxel v of the cell's rows h, 2 + h, 4 + h, 6 + h and marches z:
// per voxel plane it loads its 4 voxels (a load instruction reads 2 row segments
// of 384 bytes, three whole 128-byte lines each when rows are aligned; 16 x 16
// columns, whose segments of 192 bytes split lines between waves, read 20%
// slower) and accumulates the z-contraction in registers,
//   A[n] += Bz_n(w) * dfield[z][y][x]        (n = cz - tz, 4 planes),
// the only per-voxel work.  When a z-tile ends, control plane A[0] is finished
// for the cell's columns and is contracted over y, then x, as two chained
// matrix products on the matrix cores, straight from the accumulators, for each
// half of 16 voxels:
//   D[x][cy]  = sum_row  A[x][row] By[row][cy]      (2 steps of 4 rows)
//   E[cx][cy] += sum_x   Bx[cx][x] D[x][cy]         (4 steps of 4 voxels, 4 sums)
// (v_mfma_f32_16x16x4_f32, FP32 in and out: two row swaps between lanes turn
// the accumulator registers into the first product's A operand, its result
// registers are the second one's B operand, and the weight matrices of the
// brick are 2 + 8 registers per lane).  A cell's window is at most 16 x 16
// control points.  E goes to the wave's own slab in LDS; no wave waits for
// another while it marches.  After the brick's last plane one barrier, and the
// slabs of the brick's cells are summed in wave order into the brick's partials.
// Where the slabs would leave a brick fewer than kAdjMinStaged tiles, they hold two
// planes, and each plane is summed and stored when it is finished, after one
// barrier per z-tile.
//
// What bounds it: reading dfield once (12 bytes per voxel).  The z-accumulation
// is 12 FMAs per voxel (about 20 us of every SIMD at 512 x 512 x 256), the
// contractions are 20 matrix instructions of 32 cycles per 256 columns and
// z-tile where a window has at most 5 rows, 28 up to 8 (about 20 us at spacing 5), both
// under the 120 us that the read takes.  512 x 512 x 256, spacing 5: 148 us, with the
// contractions as vector moments on tile lanes, two barriers a tile, 156; 267 x 169
// x 237, spacing 16: 31 against 52.
//
// Pass 2 (a lane or a wave per control point) sums, in a fixed order, the
// partials of the bricks whose voxels meet the point's support.  No atomics
// anywhere: the bits depend on the inputs only.
#pragma once

#include "bsi_device.h"

namespace bsi {

// Waves per SIMD the pass-1 kernels are compiled for (a register bound of 512 /
// this): 3, because at 4 the march and the contraction together spill, which cost
// 12% at 512 x 512 x 256, spacing 5 (168 against 150 us).
#ifndef BSI_ADJ_WPE
#define BSI_ADJ_WPE 3
#endif
// Narrow cells (adj_narrow) hold half of that: 6 (300 x 256 x 200, spacing 1: 212 us, 230 at 4
// and 5; what spills at 6 lies in adj_cell_sparse).
constexpr int kAdjWpeNarrow = 6;
__host__ __device__ constexpr int adj_wpe(bool narrow) { return narrow ? kAdjWpeNarrow : BSI_ADJ_WPE; }
constexpr int kAdjCellsX = 2, kAdjCellsY = 2;      // cells of a brick, one per wave
constexpr int kAdjWaves = kAdjCellsX * kAdjCellsY;
constexpr int kAdjThreads = kAdjWaves * kWave;
constexpr int kAdjTile = 16;                       // points per axis of a matrix tile
constexpr int kAdjCellX = 32, kAdjCellY = 8;       // voxel columns of a cell
// A lane's voxels.  Cells of up to 32 columns: row s is 2 s + h, h = lane / 32.  Narrow: cells
// of up to 16 (spacings 1 and 2, adj_narrow), 16 lanes a row: row s is adj_step_row(s, lane / 16),
// which is the first product's operand as it stands, half the accumulators and loads, and no
// second half of products.  Pass 1 of 300 x 256 x 200 at spacing 1: 212 us, with 32 lanes a
// row, 13 of them at work, 272; of 118 x 357 x 486 286 and 353 (then 183 and 254 by
// adj_combine_slabs).
template <bool Narrow>
constexpr int kAdjSteps = Narrow ? 2 : 4;
// The brick depth rule (make_adj_geom), measured on pass 1 alone:
// - the number of z-bricks: a CU reads at most about 28 bytes per ns, whatever
//   it holds (a plane of a brick in 0.44 us), and all CUs together 22 each (0.54), so
//   a launch takes (planes per brick + kAdjBrickCost) x the larger of kAdjCuCost x
//   the bricks of the fullest CU and the bricks per CU on average, where
//   kAdjBrickCost is what a brick's start and last four planes cost.  256 x 256 x 160,
//   spacing 5: 29.4 us with 256 or 512 bricks, 32.6 with 384; 294 x 130 x 208,
//   spacing 6: 27.5 with 405, 31.3 with 540, 33.6 with 270.
// - depth bound where a brick's slabs hold all of its planes: 96 voxels
//   (spacing 8 at 511 x 509 x 250: 140 us against 148 at 48).
// - LDS of those slabs: three workgroups per CU, or, for the wide windows of
//   spacing 3, two (512 x 228 x 385, spacing 3: 129 us; with two-plane
//   slabs 138 to 147, before the cells 145 to 152).
// - depth with two-plane slabs (spacing 1, or 1 along z): 20 voxels (both passes at
//   spacing 1: 300 x 256 x 200 279 us, 285 at 30, 280 at 16; 512 x 512 x 100 440, 462 and 464;
//   128^3 67, 74 and 60; 200^3 141, 135 and 138).
// - whole slabs of fewer than kAdjMinStagedDeep planes (spacings 4 to 7 x 1 x 1), whose
//   partials are 4/3 of their voxels' points, only where bricks of that depth would not
//   fill the CUs four times: 300 x 260 x 400 at 4 x 1 x 1 256 us with them, 224 without; 200^3
//   at 6 x 1 x 1 86 and 89.
constexpr int kAdjCus = 256;
constexpr double kAdjCuCost = 0.9, kAdjBrickCost = 4;
constexpr int kAdjDepthStaged = 96, kAdjDepthTwo = 20, kAdjDepthMost = 48;
constexpr int kAdjMinStaged = 8, kAdjMinStagedDeep = 10;             // tiles and planes, of a brick with whole slabs
constexpr int kAdjSlabFloats3 = 13312, kAdjSlabFloats2 = 20000;      // slabs of 3 and of 2 workgroups per CU
// Shallower bricks than the depth bounds are used up to this workspace size,
// and deeper ones, of kAdjDepthMost planes or all of them, where the partials of a
// geometry that bsi_adjoint_noalloc takes would be above 9/8 of its limit.
constexpr size_t kAdjShallowBytes = (size_t)32 << 20;

// Voxels of a cell along x at spacing d: the most, up to 32, whose window is at
// most 16 control points ((31 + 2) / 3 + 4 = 15 at spacing 3; w + 3 at spacing 1), but 16 at
// spacing 2, where 24 would fit: 16 lanes a row all at work, 24 of 32 otherwise
// (300 x 300 x 200: the adjoint 95 us against 112, the fused step 207 against 265).  Along y a
// cell of 8 rows meets at most 11.
__host__ __device__ constexpr int adj_cell(int d) { return d == 1 ? 13 : d == 2 ? 16 : kAdjCellX; }

__host__ __device__ constexpr int adj_gcd(int a, int b) { return b == 0 ? a : adj_gcd(b, a % b); }
// Largest control window of runs of w voxels that start at multiples of w, at
// spacing d: the start's offset in its tile is at most d - gcd(w, d).
__host__ __device__ constexpr int adj_window(int w, int d) { return (d - adj_gcd(w, d) + w - 1) / d + 4; }

// v / d for 0 <= v and v d < 2^32, by m = adj_magic(d): the product is above v / d
// by at most v / 2^32 < 1 / d.
__host__ __device__ inline uint32_t adj_magic(int d) { return (uint32_t)(((uint64_t)1 << 32) / (uint32_t)d + (d > 1)); }
__host__ __device__ inline int adj_div(int v, int d, uint32_t m) {
  return d == 1 ? v : (int)(((uint64_t)(uint32_t)v * m) >> 32);
}

// The brick of voxel v.
__host__ __device__ inline int adj_brick_of_voxel(const AdjAxis& a, int v) {
  return a.mw ? adj_div(v, a.w, a.mw) : v / a.w;
}

struct AdjBrick {
  int x0, y0, z0, xe, ye, ze;  // voxel range [x0, xe) etc.
  int cx0, cy0, cz0;           // first control index of the window
  int Cx, Cy;                  // window extent in x, y
};

__host__ __device__ inline AdjBrick adj_brick_geom(const AdjGeom& a, int brick) {
  const VolGeom& g = a.g;
  AdjBrick b;
  const int bx = brick % a.x.nb;
  const int t = brick / a.x.nb;
  const int by = t % a.y.nb;
  const int bz = t / a.y.nb;
  b.x0 = adj_brick_begin(a.x, g.nx, bx);
  b.y0 = adj_brick_begin(a.y, g.ny, by);
  b.z0 = adj_brick_begin(a.z, g.nz, bz);
  b.xe = adj_brick_begin(a.x, g.nx, bx + 1);
  b.ye = adj_brick_begin(a.y, g.ny, by + 1);
  b.ze = adj_brick_begin(a.z, g.nz, bz + 1);
  b.cx0 = adj_div(b.x0, g.dx, a.x.md);
  b.cy0 = adj_div(b.y0, g.dy, a.y.md);
  b.cz0 = bz * a.z.k;  // whole tiles
  b.Cx = adj_div(b.xe - 1, g.dx, a.x.md) - b.cx0 + 4;
  b.Cy = adj_div(b.ye - 1, g.dy, a.y.md) - b.cy0 + 4;
  return b;
}

// Control planes of a brick's window: the z-tiles of its voxels plus 3.
__host__ __device__ inline int adj_brick_cz(const AdjGeom& a, const AdjBrick& b) {
  return adj_div(b.ze - 1, a.g.dz, a.z.md) - b.cz0 + 4;
}

// Floats per brick in the workspace, and the offset of window point
// (czl, cyl, cxl) within its brick's partials.
__host__ __device__ inline size_t adj_brick_stride(const AdjGeom& a) {
  return (size_t)a.z.cm * a.y.cm * a.x.cm * 3;
}
__host__ __device__ inline size_t adj_part_offset(const AdjGeom& a, int czl, int cyl, int cxl) {
  return ((size_t)(czl * a.y.cm + cyl) * a.x.cm + cxl) * 3;
}

// Cell w of a brick, (w mod 2, w / 2) in x and y: its voxels [x0, x0 + nx) x
// [y0, y0 + ny) and its window of Cx x Cy control points from (cx0, cy0).  A
// cell past the volume has no voxels and no window.
struct AdjCell {
  int x0, nx, cx0, Cx;
  int y0, ny, cy0, Cy;
};
// The tile (first control index) of a voxel on the x and y axes; the real-spacing
// grid reads its own from tables (GenTiles).
struct AdjTiles {
  const AdjGeom& a;
  __host__ __device__ int x(int v) const { return adj_div(v, a.g.dx, a.x.md); }
  __host__ __device__ int y(int v) const { return adj_div(v, a.g.dy, a.y.md); }
};
template <class Tiles>
__host__ __device__ inline AdjCell adj_cell_of(const AdjGeom& a, const Tiles& t, const AdjBrick& b, int w) {
  AdjCell c;
  c.x0 = b.x0 + w % kAdjCellsX * a.cell;
  c.y0 = b.y0 + w / kAdjCellsX * kAdjCellY;
  c.nx = imax(0, imin(a.cell, b.xe - c.x0));
  c.ny = imax(0, imin(kAdjCellY, b.ye - c.y0));
  const bool any = c.nx > 0 && c.ny > 0;
  c.cx0 = any ? t.x(c.x0) : b.cx0;
  c.cy0 = any ? t.y(c.y0) : b.cy0;
  c.Cx = any ? t.x(c.x0 + c.nx - 1) - c.cx0 + 4 : 0;
  c.Cy = any ? t.y(c.y0 + c.ny - 1) - c.cy0 + 4 : 0;
  return c;
}
__host__ __device__ inline AdjCell adj_cell_geom(const AdjGeom& a, const AdjBrick& b, int w) {
  return adj_cell_of(a, AdjTiles{a}, b, w);
}

// LDS slabs: wave w's plane in slot s begins at float (s * kAdjWaves + w) *
// slab; component c of point (cyl, cxl) of the cell's window is at
// adj_slab_point.  Rows hold a multiple of 4 points: a lane's 4 columns of E are
// one 16-byte store.
__host__ __device__ inline int adj_slab(const AdjGeom& a) { return 3 * a.ch * a.cw; }
__host__ __device__ inline int adj_slab_at(const AdjGeom& a, int slot, int w) { return (slot * kAdjWaves + w) * adj_slab(a); }
__host__ __device__ inline int adj_slab_point(const AdjGeom& a, int c, int cyl, int cxl) {
  return (c * a.ch + cyl) * a.cw + cxl;
}
// Cells of one matrix tile's width (kAdjSteps).
__host__ __device__ inline bool adj_narrow(const AdjGeom& a) { return a.cell <= kAdjTile; }
// Slots: every plane of the brick, or two in turn.
__host__ __device__ inline bool adj_staged(const AdjGeom& a) { return a.slots >= a.z.cm; }
__host__ __device__ inline size_t adj_lds_bytes(const AdjGeom& a) {
  return (size_t)a.slots * kAdjWaves * adj_slab(a) * sizeof(float);
}

// The row that lanes 16 k .. 16 k + 15 hold in step t of the first product,
// after the row swaps of adj_cell_emit.
__host__ __device__ constexpr int adj_step_row(int t, int k) { return 4 * t + 2 * (k & 1) + (k >> 1); }
// This lane's voxels within the plane: their column in the cell and rows, and their byte
// offsets from the cell's first voxel, clamped into the cell so that every lane loads from
// a valid address without a branch (a clamped voxel's weights are zero).  8 rows
// of at most 2^20 voxels: below 2^32 bytes.
template <bool Narrow>
__host__ __device__ constexpr int adj_lane_col(int lane) { return lane % (Narrow ? kAdjTile : kAdjCellX); }
template <bool Narrow>
__host__ __device__ constexpr int adj_lane_row(int lane, int s) {
  return Narrow ? adj_step_row(s, lane / kAdjTile) : 2 * s + lane / kAdjCellX;
}
template <bool Narrow>
__host__ __device__ inline void adj_cell_offsets(int nx, int cnx, int cny, int lane,
                                                 uint32_t (&off)[kAdjSteps<Narrow>]) {
  const int v = imin(adj_lane_col<Narrow>(lane), cnx - 1);
#pragma unroll
  for (int s = 0; s < kAdjSteps<Narrow>; ++s)
    off[s] = ((uint32_t)imin(adj_lane_row<Narrow>(lane, s), cny - 1) * (uint32_t)nx + (uint32_t)v) * 12u;
}

// Load of three floats through a buffer resource (uniform base, 32-bit lane offset:
// no address arithmetic per load).  Stream: non-temporal, for the voxels of
// dfield, since every one is read once; the read stream then
// does not leave the caches full of dfield lines that the next kernel's writes
// have to displace.
template <bool Stream>
__device__ __forceinline__ F3 adj_load3(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  // the whole vector is converted: a bit cast of single elements reads element 0 for all three
  const fwd_f3 v = __builtin_bit_cast(fwd_f3, __builtin_amdgcn_raw_buffer_load_b96(rs, (int)off, 0, Stream ? kCpolNT : 0));
  return F3{v.x, v.y, v.z};
}
// Bytes of that part: the cell's rows, up to its last voxel.
__host__ __device__ inline uint32_t adj_cell_bytes(int nx, int cnx, int cny) {
  return ((uint32_t)(cny - 1) * (uint32_t)nx + (uint32_t)cnx) * 12u;
}

// Weight matrices of a cell, the entries of lane (q, m) = (lane / 16, lane % 16).
// y[t] = By of row adj_step_row(t, q) at control row cy0 + m (the first
// product's B operand); x[g][i] = Bx of voxel 16 g + 4 q + i at control column
// cx0 + m (the second product's A operand).  Zero outside a voxel's window and
// for voxels outside the cell.  A weight inside its window that is zero (B3 at
// offset 0) is kept as -0: the same in every sum, but its bits tell the two kinds
// apart (adj_cell_sparse).
struct AdjWeights {
  float x[2][4], y[2];
};
// Weight of voxel o0 + v (o0: the offset in its tile of the cell's first voxel, `in`: v lies in the cell)
// at the cell's control index c; rows: the weight rows of this spacing.  Every
// lane loads, from a row and entry within the table.
__device__ __forceinline__ float adj_weight(const float* __restrict__ rows, int d, uint32_t magic, int o0, int v, int c,
                                            bool in) {
  const int t = adj_div(o0 + v, d, magic), l = c - t;
  const float w = rows[4 * (o0 + v - t * d) + (l & 3)];
  return in && (uint32_t)l < 4u ? (w == 0.f ? -0.f : w) : 0.f;
}
__device__ __forceinline__ AdjWeights adj_cell_weights(const AdjGeom& a, const AdjCell& c, const float* __restrict__ lut,
                                                       int lane) {
  const int m = lane % kAdjTile, q = lane / kAdjTile;
  const float *rx = lut_row(lut, a.g.dx, 0), *ry = lut_row(lut, a.g.dy, 0);
  const int ox = c.x0 - c.cx0 * a.g.dx, oy = c.y0 - c.cy0 * a.g.dy;
  AdjWeights w;
#pragma unroll
  for (int g = 0; g < 2; ++g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = kAdjTile * g + 4 * q + i;
      w.x[g][i] = adj_weight(rx, a.g.dx, a.x.md, ox, v, m, v < c.nx);
    }
    const int row = adj_step_row(g, q);
    w.y[g] = adj_weight(ry, a.g.dy, a.y.md, oy, row, m, row < c.ny);
  }
  return w;
}

typedef float adj_f4 __attribute__((ext_vector_type(4)));

// Swap the odd rows of 16 lanes of a with the even rows of b: from a = row pair
// (2 s, 2 s + 1) and b = row pair (2 s + 2, 2 s + 3) of 32 voxels each, a becomes
// the first 16 voxels of the rows 2 s, 2 s + 2, 2 s + 1, 2 s + 3 and b the last 16.
__device__ __forceinline__ void adj_swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                  false, false);
  const uint32_t ra = r[0], rb = r[1];
  a = __builtin_bit_cast(float, ra);
  b = __builtin_bit_cast(float, rb);
}

// The value of lane (q, (m - N) mod 16) of this lane's row of 16 (DPP row_ror).
template <int N>
__device__ __forceinline__ float adj_row_ror(float v) {
  if constexpr (N == 0) return v;
  else
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, true));
}

// E of a plane that holds an infinity or a NaN, whose product with a zero
// weight would reach the whole window: the same sums over each point's own
// support only.  f[g][t]: the first product's operands of half g, of G halves.
// Lane (q, m) forms columns 4 q + j, row m.
template <int G>
__device__ __forceinline__ adj_f4 adj_cell_sparse(const float (&f)[2][2], const AdjWeights& w, int lane) {
  const int m = lane % kAdjTile, q = lane / kAdjTile;
  adj_f4 e{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {  // the row that lanes 16 k .. hold in step t
      const float wy = __shfl(w.y[t], kAdjTile * k + m);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll 1
          for (int v4 = 0; v4 < 4; ++v4) {  // voxel 16 g + 4 v4 + i
            const float val = __shfl(f[g][t], kAdjTile * k + 4 * v4 + i);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float wx = __shfl(w.x[g][i], kAdjTile * v4 + 4 * q + j);
              if (__builtin_bit_cast(uint32_t, wx) != 0 && __builtin_bit_cast(uint32_t, wy) != 0)
                e[j] = fmaf(wx, wy * val, e[j]);
            }
          }
    }
  return e;
}

// Components [C0, C0 + N) of a finished plane, together in one set of products:
// component C0 + c takes rows c S .. of the first product's result, so that the
// second product's 16 columns hold N windows of at most S rows.
template <int C0, int N, int S, int A = 4, int G = 2>
__device__ __forceinline__ void adj_contract(const float (&f)[3][2][2], const AdjWeights& w, adj_f4& E) {
  static_assert(N * S <= kAdjTile || N == 1, "the windows fit a tile");
  adj_f4 D[2];
#pragma unroll
  for (int g = 0; g < G; ++g) D[g] = adj_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      D[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[C0][g][t], w.y[t], D[g], 0, 0, 0);
      if constexpr (N > 1)
        D[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[C0 + 1][g][t], adj_row_ror<S % 16>(w.y[t]), D[g], 0, 0, 0);
      if constexpr (N > 2)
        D[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[C0 + 2][g][t], adj_row_ror<2 * S % 16>(w.y[t]), D[g], 0, 0, 0);
    }
  // The second in A sums of every A-th step: a window of 4 d columns in one chain
  // rounds more often than per tile (256 x 256 x 96, spacing 5, error against 64
  // bits: 1.31e-7 in one chain, 1.22e-7 in four; the time is the same).
  adj_f4 X[A];
#pragma unroll
  for (int i = 0; i < A; ++i) X[i] = adj_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) X[i % A] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x[g][i], D[g][i], X[i % A], 0, 0, 0);
  E = X[0] + X[1];
  if constexpr (A == 4) E += X[2] + X[3];
}

// Contract a finished plane of a cell (f3[s]: this lane's voxel of its row s) and store its window to `dst`, the wave's slab slot: all of a slab's
// rows and columns (those past the cell's window are zeros).  cw, ch: of the
// geometry; ch decides how many components share the products (a uniform
// branch, the same bits: the other components only add zeros).  28 matrix
// instructions for windows of up to 8 rows, 20 for up to 5 (spacings 4 and 6 and
// up) and 36 for more; narrow cells have no second half: 18 for more than 8 rows (spacing 1).
// Every lane of the wave takes part.
template <bool Narrow>
__device__ __forceinline__ void adj_cell_emit(const F3 (&f3)[kAdjSteps<Narrow>], const AdjWeights& w,
                                              float* __restrict__ dst, int cw, int ch, int lane) {
  constexpr int G = Narrow ? 1 : 2;
  const int m = lane % kAdjTile, q = lane / kAdjTile;
  float f[3][2][2];  // [component][half][step]
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if constexpr (Narrow) {
      f[0][0][t] = f3[t].x, f[1][0][t] = f3[t].y, f[2][0][t] = f3[t].z;
    } else {
      f[0][0][t] = f3[2 * t].x, f[1][0][t] = f3[2 * t].y, f[2][0][t] = f3[2 * t].z;
      f[0][1][t] = f3[2 * t + 1].x, f[1][1][t] = f3[2 * t + 1].y, f[2][1][t] = f3[2 * t + 1].z;
#pragma unroll
      for (int c = 0; c < 3; ++c) adj_swap_rows(f[c][0][t], f[c][1][t]);
    }
  }
  // an infinity or NaN anywhere in the plane makes every entry of its E
  // non-finite (0 * inf = NaN), so any one entry per set of products tells
  float probe;
  // E's columns 4 q .. of row `row` of component `comp`
  auto store = [&](const adj_f4& E, int row, int comp) {
    if (row < ch && comp < 3 && 4 * q < cw)
      *reinterpret_cast<adj_f4*>(dst + (comp * ch + row) * cw + 4 * q) = E;
  };
  if (ch <= 5) {
    adj_f4 E;
    adj_contract<0, 3, 5, 4, G>(f, w, E);
    const int c = (m >= 5) + (m >= 10) + (m >= 15);
    store(E, m - 5 * c, c);
    probe = E[0];
  } else if (ch <= 8) {
    adj_f4 E, E2;
    adj_contract<0, 2, 8, 4, G>(f, w, E);
    adj_contract<2, 1, 16, 4, G>(f, w, E2);
    store(E, m & 7, m >> 3);
    store(E2, m, 2);
    probe = E[0] + E2[0];
  } else {
    adj_f4 E, E1, E2;
    adj_contract<0, 1, 16, 2, G>(f, w, E);
    store(E, m, 0);
    adj_contract<1, 1, 16, 2, G>(f, w, E1);
    store(E1, m, 1);
    adj_contract<2, 1, 16, 2, G>(f, w, E2);
    store(E2, m, 2);
    probe = E[0] + E1[0] + E2[0];
  }
  if (__builtin_expect(__any(!(fabsf(probe) < __builtin_inff())), 0)) {
#pragma unroll
    for (int c = 0; c < 3; ++c) store(adj_cell_sparse<G>(f[c], w, lane), m, c);
  }
}

// The cells' windows within their brick's (first point, and extent), and the reciprocals of
// the brick's points per plane and per row.
struct AdjWindows {
  int fx[kAdjWaves], fy[kAdjWaves], nx[kAdjWaves], ny[kAdjWaves];
  uint32_t mp, mc;
};
template <class Tiles>
__host__ __device__ inline AdjWindows adj_windows(const AdjGeom& a, const Tiles& tiles, const AdjBrick& b) {
  AdjWindows v;
  v.mp = adj_magic(b.Cy * b.Cx);
  v.mc = adj_magic(b.Cx);
#pragma unroll
  for (int w = 0; w < kAdjWaves; ++w) {
    const AdjCell c = adj_cell_of(a, tiles, b, w);
    v.fx[w] = c.cx0 - b.cx0;
    v.fy[w] = c.cy0 - b.cy0;
    v.nx[w] = c.Cx;
    v.ny[w] = c.Cy;
  }
  return v;
}

// Sum the slabs of planes czl0 .. czl0 + np - 1 (slots slot0 ..) over the
// brick's cells, in wave order, into the brick's partials.  Collective over
// `threads` threads, after a barrier.  Without branches: a point outside a cell's window
// reads the slab's first and leaves it, and the windows are the caller's: with two-plane slabs
// this runs at every plane (a branch per cell took 300 instructions per point, the
// windows 181 per wave; pass 1 of 300 x 256 x 200 at spacing 1: 183 us against 212).
__device__ __forceinline__ void adj_combine_slabs(const AdjGeom& a, const AdjWindows& win, const AdjBrick& b,
                                                  const float* __restrict__ slabs, float* __restrict__ pbase, int czl0,
                                                  int np, int slot0, int tid, int threads) {
  // items: (plane, point), a wave's lanes consecutive; plane and row of an item
  // by reciprocal (at most 2^11 points, and 2^16 items: exact)
  const int slab = adj_slab(a), comp = a.ch * a.cw;
  const int points = b.Cy * b.Cx, n = np * points;
  for (int i = tid; i < n; i += threads) {
    const int p = np == 1 ? 0 : adj_div(i, points, win.mp), j = i - p * points;
    const int cyl = adj_div(j, b.Cx, win.mc), cxl = j - cyl * b.Cx;
    const float* slot = slabs + (slot0 + p) * kAdjWaves * slab;
    F3 h[2]{};  // per cell row
#pragma unroll
    for (int w = 0; w < kAdjWaves; ++w) {
      const int y = cyl - win.fy[w], x = cxl - win.fx[w];
      const bool in = ((uint32_t)y < (uint32_t)win.ny[w]) & ((uint32_t)x < (uint32_t)win.nx[w]);
      const float* v = slot + w * slab + (in ? y * a.cw + x : 0);
      const F3 e{v[0], v[comp], v[2 * comp]};
      h[w / kAdjCellsX] = h[w / kAdjCellsX] + F3{in ? e.x : 0.f, in ? e.y : 0.f, in ? e.z : 0.f};
    }
    const F3 s = h[0] + h[1];
    stf3(pbase + adj_part_offset(a, czl0 + p, cyl, cxl), s);
  }
}

// Where a wave is along z while it marches a brick of the aligned grid: the
// plane's offset in its z-tile, for its weights.  Bricks start on a tile.
struct AdjZ {
  const float* row;  // weight rows of this z spacing
  int dz, oz;
  __device__ __forceinline__ AdjZ(const float* lut, int dz_) : row(lut_row(lut, dz_, 0)), dz(dz_), oz(0) {}
  __device__ __forceinline__ const float* weights() const { return row + 4 * oz; }
  // step to the next plane; true when this one was its tile's last
  __device__ __forceinline__ bool step() {
    oz = oz + 1 == dz ? 0 : oz + 1;
    return oz == 0;
  }
};

// a0 .. a3 <- a1, a2, a3, 0, in place.  Written as instructions on four fixed
// registers: as assignments, the compiler gives the shifted values registers of
// their own and copies all 48 accumulators at every plane (96 moves per plane).
__device__ __forceinline__ void adj_shift(float& a0, float& a1, float& a2, float& a3) {
  asm volatile("v_mov_b32 %0, %1\n\tv_mov_b32 %1, %2\n\tv_mov_b32 %2, %3\n\tv_mov_b32 %3, 0"
               : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3));
}

// March np voxel planes of a cell: the lane's voxel s of plane z is at
// base + z * zs + off[s] (bytes; `bytes`: adj_cell_bytes).  emit(f, czl) is called for each finished
// control plane, czl = 0, 1, ... in order, the last three of them after the
// last plane; setup() once, after the first loads are issued.  acc[n] is the z-accumulation of control plane tile + n; the
// accumulators move down when a tile ends (48 moves, against 48 FMAs per plane).
//
// Two register sets, each holding one plane's loads.  The loop is unrolled over
// them and its loads are unconditional (past the end, from the last plane
// again), so each set keeps fixed registers, and waiting for one set's loads
// leaves the other set's in flight.
template <bool Stream, int S, class Z, class Setup, class Emit>
__device__ __forceinline__ void adj_march(const char* base, size_t zs, uint32_t bytes, const uint32_t (&off)[S],
                                          int np, Z zp, Setup&& setup, Emit&& emit) {
  F3 acc[4][S];
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int s = 0; s < S; ++s) acc[n][s] = F3{0.f, 0.f, 0.f};
  const char* ahead = base;  // the plane to be loaded next, at most the last
  int left = np - 1;         // planes after it
  int czl = 0;
  auto load = [&](F3(&d)[S]) {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(ahead), 0, (int)bytes, kBufferFlags);
#pragma unroll
    for (int s = 0; s < S; ++s) d[s] = adj_load3<Stream>(rs, off[s]);
    ahead += left > 0 ? zs : 0;
    --left;
  };
  auto add = [&](const F3(&d)[S]) {
    const float* ws = zp.weights();  // uniform: one scalar load
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const float w = ws[n];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        acc[n][s].x = fmaf(w, d[s].x, acc[n][s].x);
        acc[n][s].y = fmaf(w, d[s].y, acc[n][s].y);
        acc[n][s].z = fmaf(w, d[s].z, acc[n][s].z);
      }
    }
  };
  auto finish = [&]() {
    emit(acc[0], czl++);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      adj_shift(acc[0][s].x, acc[1][s].x, acc[2][s].x, acc[3][s].x);
      adj_shift(acc[0][s].y, acc[1][s].y, acc[2][s].y, acc[3][s].y);
      adj_shift(acc[0][s].z, acc[1][s].z, acc[2][s].z, acc[3][s].z);
    }
    asm volatile("s_nop 4");  // the moves above are done before a lane swap may read their results
  };
  F3 d0[S], d1[S];
  load(d0);
  __builtin_amdgcn_sched_barrier(0);  // d0's loads are issued first: waiting for them leaves d1's in flight
  load(d1);
  __builtin_amdgcn_sched_barrier(0);
  setup();  // what the emission needs, while the first loads are on their way
  // pairs of planes, with one way in and one way back, so that both sets'
  // loads are in flight on either
#pragma unroll 1
  for (int pairs = np >> 1; pairs > 0; --pairs) {
    add(d0);
    load(d0);
    if (zp.step()) finish();
    add(d1);
    load(d1);
    if (zp.step() && (pairs > 1 || (np & 1))) finish();
  }
  if (np & 1) add(d0);
  // after the last plane, the four control planes in hand, in order
#pragma unroll 1
  for (int k = 0; k < 4; ++k) finish();
}

// Pass 1 for one brick.  Collective over the workgroup (kAdjThreads threads).
// Stream: dfield is read with non-temporal loads.  Staged: adj_staged(a), Narrow:
// adj_narrow(a).  cz: the brick's control planes; z: its march along z; weights(c): cell c's
// matrices.
template <bool Stream, bool Staged, bool Narrow, class Tiles, class Z, class Weights>
__device__ __forceinline__ void adj_brick_of(const float* __restrict__ dfield, float* __restrict__ part,
                                             const AdjGeom& a, const Tiles& tiles, const AdjBrick& b, int brick, int cz,
                                             const Z& z, Weights&& weights, float* __restrict__ slabs, int tid) {
  const VolGeom& g = a.g;
  float* pbase = part + (size_t)brick * adj_brick_stride(a);
  const int lane = tid & (kWave - 1), wave = uniform(tid / kWave);
  const AdjCell c = adj_cell_of(a, tiles, b, wave);
  const bool any = c.nx > 0 && c.ny > 0;
  __syncthreads();  // a previous brick of this workgroup may still read the slabs
  // A cell past the volume has nothing to add; with two slots it marches all
  // the same (the brick's first voxels, nothing stored), for the barriers.
  if (!Staged || any) {
    AdjWeights w;
    const int cnx = any ? c.nx : 1, cny = any ? c.ny : 1;
    uint32_t off[kAdjSteps<Narrow>];
    adj_cell_offsets<Narrow>(g.nx, cnx, cny, lane, off);
    const uint32_t bytes = adj_cell_bytes(g.nx, cnx, cny);
    const size_t zs = (size_t)g.ny * g.nx * 12;
    const char* base = reinterpret_cast<const char*>(dfield) + (size_t)b.z0 * zs +
                       ((size_t)(any ? c.y0 : b.y0) * g.nx + (any ? c.x0 : b.x0)) * 12;
    AdjWindows win;
    const auto setup = [&] {
      w = weights(c);
      if constexpr (!Staged) win = adj_windows(a, tiles, b);
    };
    adj_march<Stream>(base, zs, bytes, off, b.ze - b.z0, z, setup, [&](const F3(&f)[kAdjSteps<Narrow>], int czl) {
      const int slot = Staged ? czl : czl & 1;
      adj_cell_emit<Narrow>(f, w, slabs + adj_slab_at(a, slot, wave), a.cw, a.ch, lane);
      if constexpr (!Staged) {
        // the barrier of plane czl + 1 orders this sum before the slot's next store
        __syncthreads();
        adj_combine_slabs(a, win, b, slabs, pbase, czl, 1, slot, tid, kAdjThreads);
      }
    });
  }
  if constexpr (Staged) {
    __syncthreads();
    adj_combine_slabs(a, adj_windows(a, tiles, b), b, slabs, pbase, 0, cz, 0, tid, kAdjThreads);
  }
}

// The aligned grid's.
template <bool Stream, bool Staged, bool Narrow>
__device__ __forceinline__ void adj_brick(const float* __restrict__ dfield, float* __restrict__ part,
                                          const AdjGeom& a, const float* __restrict__ lut, int brick,
                                          float* __restrict__ slabs, int tid) {
  const AdjBrick b = adj_brick_geom(a, brick);
  adj_brick_of<Stream, Staged, Narrow>(dfield, part, a, AdjTiles{a}, b, brick, adj_brick_cz(a, b), AdjZ(lut, a.g.dz),
                               [&](const AdjCell& c) { return adj_cell_weights(a, c, lut, tid & (kWave - 1)); }, slabs, tid);
}

// Pass 2: the fixed-order sum, per control point, of the partials of the bricks
// whose voxels meet its support [(c-3)d, (c+1)d) on each axis.
struct AdjSpan {
  int lo, hi;  // brick range
};

// First control index of brick b's window (b < nb): its first voxel's tile,
// b * k when the units are whole tiles.
__host__ __device__ inline int adj_brick_c0(const AdjAxis& ax, int b, int d) {
  return ax.u == d ? b * ax.k : adj_div(b * ax.w, d, ax.md);
}

__host__ __device__ inline AdjSpan adj_span(const AdjAxis& ax, int c, int d, int n) {
  return AdjSpan{adj_brick_of_voxel(ax, imax(0, (c - 3) * d)), adj_brick_of_voxel(ax, imin(n, (c + 1) * d) - 1)};
}

// Workspace offset (floats) of control point (cx, cy, cz) in brick (bx, by, bz)'s
// partials: the sum of one term per axis.
__host__ __device__ inline size_t adj_part_x(const AdjGeom& a, int bx, int cx) {
  return bx * adj_brick_stride(a) + (cx - adj_brick_c0(a.x, bx, a.g.dx)) * 3;
}
__host__ __device__ inline size_t adj_part_y(const AdjGeom& a, int by, int cy) {
  return by * (a.x.nb * adj_brick_stride(a)) + (cy - adj_brick_c0(a.y, by, a.g.dy)) * a.x.cm * 3;
}
__host__ __device__ inline size_t adj_part_z(const AdjGeom& a, int bz, int cz) {
  return bz * ((size_t)a.y.nb * a.x.nb * adj_brick_stride(a)) + (cz - adj_brick_c0(a.z, bz, a.g.dz)) * (a.y.cm * a.x.cm * 3);
}
__host__ __device__ inline size_t adj_part_addr(const AdjGeom& a, int bx, int by, int bz, int cx, int cy, int cz) {
  return adj_part_x(a, bx, cx) + adj_part_y(a, by, cy) + adj_part_z(a, bz, cz);
}

// The aligned grid's spans and terms; the real-spacing grid has its own (GenMap).
struct AdjMap {
  const AdjGeom& a;
  __device__ AdjSpan span_x(int c) const { return adj_span(a.x, c, a.g.dx, a.g.nx); }
  __device__ AdjSpan span_y(int c) const { return adj_span(a.y, c, a.g.dy, a.g.ny); }
  __device__ AdjSpan span_z(int c) const { return adj_span(a.z, c, a.g.dz, a.g.nz); }
  __device__ size_t part_x(int b, int c) const { return adj_part_x(a, b, c); }
  __device__ size_t part_y(int b, int c) const { return adj_part_y(a, b, c); }
  __device__ size_t part_z(int b, int c) const { return adj_part_z(a, b, c); }
};

// The partials of one point, of the bricks lo, lo + step, lo + 2 step .. of each span:
// two by two by two, 8 loads in flight, summed pairwise.  Bound by the latency of
// that one round, and at many points by the partials' bytes; so the instructions
// before it are few and 8 waves per SIMD wait at once.  Small: at most kAdjGatherSmall
// bytes of partials, read by buffer loads with 32-bit offsets; a brick past its span
// adds kAdjGatherSmall to the offset, which is then past the buffer (three of them
// and the largest offset stay below 2^32) and reads as zero without an access to
// memory.  Otherwise 64-bit addresses, a branch per load, four of them in flight.
// Pass 2 at 512 x 512 x 256, spacing 5: 9.0 us (of which 6.5 for its bytes at a copy's rate),
// 17.2 with divisions, clamped duplicate loads and 3 bricks on an axis in a loop;
// 512 x 228 x 385, spacing 3: 13.9 against 32.4.
constexpr uint32_t kAdjGatherSmall = 1u << 30;
template <bool Small, class Map>
__device__ __forceinline__ F3 adj_gather_point(const float* __restrict__ part, const AdjGeom& a, const Map& map, int cx,
                                               int cy, int cz, AdjSpan sx, AdjSpan sy, AdjSpan sz, int step) {
  F3 s{0.f, 0.f, 0.f};
  if constexpr (Small) {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(part), 0, (int)a.part_bytes, kBufferFlags);
    for (int bz = sz.lo; bz <= sz.hi; bz += 2 * step)
      for (int by = sy.lo; by <= sy.hi; by += 2 * step)
        for (int bx = sx.lo; bx <= sx.hi; bx += 2 * step) {
          uint32_t ox[2], oy[2], oz[2];
          F3 v[2][2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            ox[i] = (uint32_t)map.part_x(bx + i * step, cx) * 4;
            oy[i] = (uint32_t)map.part_y(by + i * step, cy) * 4;
            oz[i] = (uint32_t)map.part_z(bz + i * step, cz) * 4;
          }
          if (bx + step > sx.hi) ox[1] = kAdjGatherSmall;
          if (by + step > sy.hi) oy[1] = kAdjGatherSmall;
          if (bz + step > sz.hi) oz[1] = kAdjGatherSmall;
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const uint32_t oxy = ox[i] + oy[j];
#pragma unroll
              for (int k = 0; k < 2; ++k) v[k][j][i] = adj_load3<false>(rs, oxy + oz[k]);
            }
          s = s + (((v[0][0][0] + v[0][0][1]) + (v[0][1][0] + v[0][1][1])) +
                   ((v[1][0][0] + v[1][0][1]) + (v[1][1][0] + v[1][1][1])));
        }
  } else {
    for (int bz = sz.lo; bz <= sz.hi; bz += step)
      for (int by = sy.lo; by <= sy.hi; by += 2 * step)
        for (int bx = sx.lo; bx <= sx.hi; bx += 2 * step) {
          F3 v[2][2];
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int x = bx + i * step, y = by + j * step;
              v[j][i] = F3{0.f, 0.f, 0.f};
              if (x <= sx.hi && y <= sy.hi) v[j][i] = ldf3(part + map.part_x(x, cx) + map.part_y(y, cy) + map.part_z(bz, cz));
            }
          s = s + ((v[0][0] + v[0][1]) + (v[1][0] + v[1][1]));
        }
  }
  return s;
}

// Pass 2's workgroups.  One lane per control point, 2^lx points along x by 256 >> lx
// rows of one control plane; or one wave per point (lx < 0), whose lanes take every
// 4th brick of each axis (make_adj_geom's rule).
constexpr int kGatherThreads = 256;
constexpr int kGatherLanes = 4;  // lanes per axis of a point's wave

__host__ __device__ inline int64_t adj_gather_blocks(const AdjGeom& a) {
  const VolGeom& g = a.g;
  if (a.lx < 0) return ((int64_t)g.gx * g.gy * g.gz + kGatherThreads / kWave - 1) / (kGatherThreads / kWave);
  const int nxb = (g.gx + (1 << a.lx) - 1) >> a.lx, rows = kGatherThreads >> a.lx;
  return (int64_t)nxb * ((g.gy + rows - 1) / rows) * g.gz;
}

// Control point of thread tid of pass-2 workgroup blk (blk < adj_gather_blocks <
// 2^31); false for a thread past the grid.
__host__ __device__ inline bool adj_gather_index(const AdjGeom& a, int blk, int tid, int& cx, int& cy, int& cz) {
  const VolGeom& g = a.g;
  if (a.lx < 0) {
    const int i = blk * (kGatherThreads / kWave) + tid / kWave, row = i / g.gx;  // below 2^20
    cx = i - row * g.gx;
    cz = row / g.gy;
    cy = row - cz * g.gy;
    return cz < g.gz;
  }
  const int nxb = (g.gx + (1 << a.lx) - 1) >> a.lx, rows = kGatherThreads >> a.lx, nyb = (g.gy + rows - 1) / rows;
  const int xb = blk % nxb;
  blk /= nxb;
  cx = (xb << a.lx) + (tid & ((1 << a.lx) - 1));
  cy = blk % nyb * rows + (tid >> a.lx);
  cz = blk / nyb;
  return cy < g.gy && cx < g.gx;
}

// Workgroup blk of pass 2, thread tid: put(i, v) for each control point i, by one thread.
template <bool Small, class Map, class Put>
__device__ __forceinline__ void adj_gather_block(const float* __restrict__ part, const AdjGeom& a, const Map& map, int blk,
                                                 int tid, Put&& put) {
  int cx, cy, cz;
  const VolGeom& g = a.g;
  const bool wave = a.lx < 0;  // uniform: a function of the geometry
  const int lane = tid % kWave;
  if (!adj_gather_index(a, blk, wave ? uniform(tid / kWave) * kWave : tid, cx, cy, cz)) return;
  AdjSpan sx = map.span_x(cx), sy = map.span_y(cy), sz = map.span_z(cz);
  if (wave) {
    sx.lo += lane % kGatherLanes;
    sy.lo += lane / kGatherLanes % kGatherLanes;
    sz.lo += lane / (kGatherLanes * kGatherLanes);
  }
  F3 s = adj_gather_point<Small>(part, a, map, cx, cy, cz, sx, sy, sz, wave ? kGatherLanes : 1);
  if (wave) {
#pragma unroll
    for (int h = 1; h < kWave; h *= 2) s = s + F3{__shfl_xor(s.x, h), __shfl_xor(s.y, h), __shfl_xor(s.z, h)};
    if (lane != 0) return;
  }
  put(((size_t)cz * g.gy + cy) * g.gx + cx, s);
}

}  // namespace bsi
