// Adjoint BSI kernels for one volume: pass 1 (bricks -> partials) and pass 2
// (fixed-order gather per control point).  See adjoint_device.h.
#include <cmath>

#include "adjoint_device.h"
#include "bsi_internal.h"

namespace bsi {

template <bool Staged, bool Narrow>
__global__ __launch_bounds__(kAdjThreads) __attribute__((amdgpu_waves_per_eu(adj_wpe(Narrow)))) void adj_pass1_kernel(
    const float* __restrict__ dfield, float* __restrict__ part, AdjGeom a, const float* __restrict__ lut) {
  extern __shared__ float adj_slabs[];
  const int nbricks = a.x.nb * a.y.nb * a.z.nb;
  const int brick = xcd_remap(blockIdx.x, gridDim.x);
  if (brick >= nbricks) return;  // uniform over the workgroup
  adj_brick<true, Staged, Narrow>(dfield, part, a, lut, brick, adj_slabs, threadIdx.x);
}

template <bool Small>
__global__ __launch_bounds__(kGatherThreads) __attribute__((amdgpu_waves_per_eu(8))) void adj_pass2_kernel(
    const float* __restrict__ part, float* __restrict__ grad, AdjGeom a) {
  adj_gather_block<Small>(part, a, AdjMap{a}, xcd_remap(blockIdx.x, gridDim.x), threadIdx.x,
                          [&](size_t i, const F3& v) { stf3(grad + i * 3, v); });
}

namespace {
// k units of u voxels per brick.
AdjAxis make_axis(int n, int d, int u, int k) {
  AdjAxis a;
  a.u = u;
  a.U = (n + u - 1) / u;
  a.k = k < a.U ? k : a.U;
  a.nb = (a.U + a.k - 1) / a.k;
  a.w = a.k * u;
  a.md = adj_magic(d);
  a.mw = (int64_t)n * a.w < ((int64_t)1 << 32) ? adj_magic(a.w) : 0;
  a.cm = a.nb == 1 ? (n - 1) / d + 4 : adj_window(a.w, d);
  return a;
}
}  // namespace

// The most bricks of an axis that meet the support of one control point.
static int adj_most_bricks(const AdjAxis& x, int d) { return imin(x.nb, (4 * d + x.w - 2) / x.w + 1); }

// Pass 2's workgroups.  One point per lane, in rows of 64, 32 or 16 points, whichever
// leaves the fewest lanes idle (303 x 167 x 212, spacing 4, 79 points a row: 4.1 us
// in rows of 16 against 5.2 of 64).  Where a point's bricks take many rounds of 8
// loads and the points are few, a wave each: 512 x 512 x 256, spacing 64 (847
// points, 54 rounds) 4.2 us against 14.8, 150 x 130 x 100, spacing 20 (880, 8) 3.8
// against 6.9, but 512 x 512 x 256, spacing 24 (8750, 8) 6.8 against 5.8.
int adj_gather_lx(const AdjGeom& a) {
  const VolGeom& g = a.g;
  auto pairs = [](int n) { return (n + 1) / 2; };
  const int rounds = pairs(adj_most_bricks(a.x, g.dx)) * pairs(adj_most_bricks(a.y, g.dy)) *
                     pairs(adj_most_bricks(a.z, g.dz));
  if (rounds > 1 && a.part_bytes != 0 && (int64_t)g.gx * g.gy * g.gz <= 512 * (int64_t)imin(rounds, 2048)) return -1;
  int lx = 6;
  for (int l = 5; l >= 4; --l)
    if (((g.gx + (1 << l) - 1) >> l << l) < ((g.gx + (1 << lx) - 1) >> lx << lx)) lx = l;
  return lx;
}

// Brick depths in z-tiles of dz voxels, by the rule stated with its constants
// (adjoint_device.h).
AdjDepth adj_depth(const AdjGeom& a, int tiles, double dz) {
  AdjDepth d;
  const int plane = kAdjWaves * adj_slab(a);  // slab floats of one control plane
  const int fit3 = kAdjSlabFloats3 / plane - 3, fit2 = kAdjSlabFloats2 / plane - 3;
  // (fewer planes than that with the slabs of three workgroups per CU: of two)
  auto deep = [&](int fit) { return fit * dz >= kAdjMinStagedDeep; };
  d.fit = fit3 >= kAdjMinStaged && deep(fit3) ? fit3 : fit2;
  const long base = (long)a.x.nb * a.y.nb;
  const bool many = base * (tiles * dz / kAdjDepthTwo) >= 4 * kAdjCus;
  const bool staged = d.fit >= kAdjMinStaged && (deep(d.fit) || !many);
  d.most = imin(tiles, imax(1, (int)((staged ? kAdjDepthStaged : kAdjDepthTwo) / dz)));
  if (staged) d.most = imin(d.most, d.fit);
  // z-bricks: the fewest of those with the least modelled time (kAdjCuCost)
  const int most = (tiles + d.most - 1) / d.most;
  int nbz = most;
  double best = 0.;
  for (int n = most; n <= tiles && n <= 64 * most; ++n) {
    const int k = (tiles + n - 1) / n;
    const double per_cu = (double)(base * ((tiles + k - 1) / k)) / kAdjCus;
    const double cost = (k * dz + kAdjBrickCost) * fmax(ceil(per_cu) * kAdjCuCost, per_cu);
    if (n == most || cost < best) {
      best = cost;
      nbz = n;
    }
    if (per_cu >= 4) break;
  }
  d.best = (tiles + nbz - 1) / nbz;
  return d;
}

// Bricks of pass 1: 2 x 2 cells in x and y by whole z-tiles; the depth by the
// rule stated with its constants (adjoint_device.h).  A pure function of the
// geometry.
AdjGeom make_adj_geom(const VolGeom& g) {
  AdjGeom a;
  a.g = g;
  a.cell = adj_cell(g.dx);
  if (g.dx <= 2) {  // narrow cells: evenly wide, so that the last brick's window is not kept for a few voxels
    const int nb = (g.nx + kAdjCellsX * a.cell - 1) / (kAdjCellsX * a.cell);
    a.cell = ((g.nx + nb * kAdjCellsX - 1) / (nb * kAdjCellsX) + g.dx - 1) / g.dx * g.dx;
  }
  a.cw = (imin(adj_window(a.cell, g.dx), (g.nx - 1) / g.dx + 4) + 3) / 4 * 4;
  a.ch = imin(adj_window(kAdjCellY, g.dy), (g.ny - 1) / g.dy + 4);
  a.x = make_axis(g.nx, g.dx, 1, kAdjCellsX * a.cell);
  a.y = make_axis(g.ny, g.dy, 1, kAdjCellsY * kAdjCellY);
  const int tiles = (g.nz + g.dz - 1) / g.dz;
  const AdjDepth depth = adj_depth(a, tiles, g.dz);
  auto set_depth = [&](int k) {
    a.z = make_axis(g.nz, g.dz, g.dz, k);
    a.slots = a.z.cm <= depth.fit + 3 ? a.z.cm : 2;
  };
  set_depth(depth.best);
  if (a.z.k < depth.most && adj_workspace_bytes(a) > kAdjShallowBytes) set_depth(depth.most);
  if (adj_limit_bytes(g) <= BSI_ADJOINT_NOALLOC_MAX_BYTES)
    for (int deeper : {imax(1, kAdjDepthMost / g.dz), tiles}) {
      if (adj_workspace_bytes(a) <= BSI_ADJOINT_NOALLOC_MAX_BYTES / 8 * 9) break;
      set_depth(imin(tiles, deeper));
    }
  a.part_bytes = adj_workspace_bytes(a) <= kAdjGatherSmall ? (uint32_t)adj_workspace_bytes(a) : 0;
  a.lx = adj_gather_lx(a);
  return a;
}

size_t adj_workspace_bytes(const AdjGeom& a) {
  return (size_t)a.x.nb * a.y.nb * a.z.nb * a.x.cm * a.y.cm * a.z.cm * 3 * sizeof(float);
}

// The size that bsi_adjoint_noalloc's limit is stated for: the partials of bricks
// of 64 x 16 voxel columns, about 48 planes deep (fewer, down to half, where a
// brick's window then holds at most 6144 floats), with the window strides
// (w - 1) / d + 5.  The limit is a property of the geometry alone and does not
// move with the bricks that the kernels use.
size_t adj_limit_bytes(const VolGeom& g) {
  auto axis = [](int n, int d, int k, size_t* bricks, size_t* window) {
    const int w = n < k ? n : k;
    *bricks = (size_t)(n + w - 1) / w;
    *window = (size_t)(d == 1 ? w + 3 : (w - 1) / d + 5);
  };
  size_t bx, by, wx, wy;
  axis(g.nx, g.dx, 64, &bx, &wx);
  axis(g.ny, g.dy, 16, &by, &wy);
  int kz = imax(1, 48 / g.dz);
  const int kfit = 6144 / (int)(wy * wx * 3) - 3;
  if (kfit < kz && 2 * kfit >= kz) kz = kfit;
  const int tiles = (g.nz + g.dz - 1) / g.dz;
  kz = imin(kz, tiles);
  const size_t bz = (size_t)(tiles + kz - 1) / kz;
  return bx * by * bz * wx * wy * (size_t)(kz + 3) * 3 * sizeof(float);
}

hipError_t launch_adjoint_partials(const float* dfield, const AdjGeom& a, const float* lut, float* part,
                                  hipStream_t s) {
  const long nbricks = (long)a.x.nb * a.y.nb * a.z.nb;
  const dim3 grid((unsigned)nbricks), block(kAdjThreads);
  const auto kernel = adj_narrow(a) ? (adj_staged(a) ? &adj_pass1_kernel<true, true> : &adj_pass1_kernel<false, true>)
                                    : (adj_staged(a) ? &adj_pass1_kernel<true, false> : &adj_pass1_kernel<false, false>);
  hipLaunchKernelGGL(kernel, grid, block, adj_lds_bytes(a), s, dfield, part, a, lut);
  return hipGetLastError();
}

hipError_t launch_adjoint_reduce(const float* part, float* grad, const AdjGeom& a, hipStream_t s) {
  const int64_t nblk = adj_gather_blocks(a);
  if (nblk > kMaxLaunchThreads / kGatherThreads) return hipErrorInvalidConfiguration;  // 2^32 control points
  if (a.part_bytes != 0)
    hipLaunchKernelGGL(adj_pass2_kernel<true>, dim3((unsigned)nblk), dim3(kGatherThreads), 0, s, part, grad, a);
  else
    hipLaunchKernelGGL(adj_pass2_kernel<false>, dim3((unsigned)nblk), dim3(kGatherThreads), 0, s, part, grad, a);
  return hipGetLastError();
}

hipError_t launch_adjoint(const float* dfield, float* grad, const AdjGeom& a, const float* lut,
                          float* part, hipStream_t s) {
  hipError_t e = launch_adjoint_partials(dfield, a, lut, part, s);
  if (e != hipSuccess) return e;
  return launch_adjoint_reduce(part, grad, a, s);
}

}  // namespace bsi
