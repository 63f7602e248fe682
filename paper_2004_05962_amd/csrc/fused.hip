// Fused SSD gradient: BSI (Eq. 1) -> trilinear warp -> SSD -> adjoint of Eq. 1
// in one pass over the voxels, so neither the displacement field nor its
// gradient is ever written to memory.  Merging the other FFD steps into BSI is
// the direction the paper's conclusion (Sec. 8) names for further speed-up.
//
//   T(x)      = sum_{l,m,n} Bx_l By_m Bz_n phi                 (Eq. 1)
//   W(x)      = moving(x + T(x))        trilinear, see warp_device.h
//   L         = sum_x (W(x) - fixed(x))^2
//   dL/dphi   = B^T [ 2 (W - fixed) dW/dp ]                    (the adjoint)
//
// Pass 1 is the adjoint's z-first pass 1 (adjoint_device.h: the same bricks,
// lanes, z-accumulation and emission) with dfield replaced by the voxel's
// SSD gradient, computed on the spot.  T is evaluated as the forward kernel
// does (fwd_block): per control plane, Q = sum_m By_m sum_l Bx_l phi from the
// plane's window staged in LDS, kept for the 4 planes of the current z-tile,
// and T = sum_n Bz_n Q per voxel plane, with the same operations in the same
// order; the sampling and gradient are the SSD kernel's.  So the field, the
// per-voxel gradient and the adjoint's accumulation are bit-identical to the
// separate forward, SSD and adjoint kernels, and so is the control-grid
// gradient; only the loss is summed in another order.
//
// Each workgroup sums its voxels' squared residuals in a fixed order into one
// loss partial; pass 2 is the adjoint's fixed-order gather, and the
// loss is the fixed-order sum of the partials.  No atomics.
#include "bsi_internal.h"
#include "fused_device.h"
#include "warp_device.h"

namespace bsi {

namespace {

// The fused pass uses the adjoint's bricks with one voxel column per lane: 16
// waves of one row each, lane = x (8 waves for bricks of x spacings 1 and 2,
// FusedShape), so each lane keeps the forward's 4 contracted
// planes and the adjoint's 4 accumulators of a single column.  When a z-tile
// ends, the rows of the finished control plane meet in LDS (F, two in turn, one
// barrier per tile), and the first kAdjWaves waves contract one cell each with
// the adjoint's matrix products (adj_cell_emit: the same operations on the same
// values, so the same bits) while the others go on with the next tile.
// Bounds: per voxel about 105 vector instructions and 4 gathers of 8 bytes, and at
// each tile's border a barrier, the contraction and the first gathers of the next
// tile, which nothing hides: 1.4 us per plane of a workgroup at 256 x 256 x 160,
// spacing 5, half of it instructions.  61 to 70 us there, by how rough the
// displacements are (73 to 84 with the adjoint's brick depth, 64-bit addresses per
// corner and moments on tile lanes), 22 at 64 x 64 x 40 (62).  Starting the next tile's gathers before the border, its control plane a
// tile earlier, took more registers than 128: 68 us against 63.

// Loads of control plane cz's window into registers, and their store into a slot.
template <int L>
__device__ __forceinline__ void fused_fetch(const float* __restrict__ grid, const VolGeom& g, const FusedStage<L>& m,
                                            int cz, float (&r)[L]) {
  const float* plane = grid + (size_t)cz * g.gy * g.gx * 3;
#pragma unroll
  for (int k = 0; k < L; ++k) r[k] = m.src[k] >= 0 ? plane[m.src[k]] : 0.f;
}

template <int L>
__device__ __forceinline__ void fused_stage(float* __restrict__ slot, const FusedStage<L>& m, const float (&r)[L]) {
#pragma unroll
  for (int k = 0; k < L; ++k)
    if (m.src[k] >= 0) slot[m.dst[k]] = r[k];
}

// Q = sum_m By_m (sum_l Bx_l phi[row + m][col + l]) from a staged plane: the
// operations of the forward kernel's contraction (fwd_contract), in its order.
__device__ __forceinline__ F3 fused_contract(const float* __restrict__ slot, int base, int pitch, const float (&bx)[4],
                                             const float (&by)[4]) {
  float q[3];
  {
    const float* p = slot + base;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      q[c] = by[0] * fmaf(bx[3], p[9 + c], fmaf(bx[2], p[6 + c], fmaf(bx[1], p[3 + c], bx[0] * p[c])));
  }
#pragma unroll 1
  for (int m = 1; m < 4; ++m) {
    const float* p = slot + base + m * pitch;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float r = fmaf(bx[3], p[9 + c], fmaf(bx[2], p[6 + c], fmaf(bx[1], p[3 + c], bx[0] * p[c])));
      q[c] = fmaf(by[m], r, q[c]);
    }
  }
  return F3{q[0], q[1], q[2]};
}

// Pairs: the sampler's x-neighbour loads (trilinear_load): 1 for nx >= 2, 0 for nx == 1.
// L: staged floats per thread.  Small: the images are below 4 GiB.
// Cols: fused_cols(a).
template <int L, bool Staged, int Pairs, bool Small, int Cols>
__global__ __launch_bounds__(FusedShape<Cols>::threads) __attribute__((amdgpu_waves_per_eu(4))) void fused_pass1_kernel(const float* __restrict__ grid,
                                                                  const float* __restrict__ moving,
                                                                  const float* __restrict__ fixed,
                                                                  float* __restrict__ part,
                                                                  float* __restrict__ lpart, AdjGeom a, FusedSplit fs,
                                                                  const float* __restrict__ lut) {
  using Shape = FusedShape<Cols>;
  static_assert(!(Shape::narrow && Staged));
  constexpr int kThreads = Shape::threads;
  extern __shared__ float fused_smem[];
  const FusedLds lds = fused_lds<Cols>(a);
  float* ring = fused_smem + lds.ring;
  float* red = fused_smem + lds.red;
  float* slabs = fused_smem + lds.slabs;
  const VolGeom& g = a.g;
  const int tid = threadIdx.x;
  const int item = xcd_remap(blockIdx.x, gridDim.x);
  const int nxy = a.x.nb * a.y.nb;
  const int bz0 = item / nxy * fs.deep, bz1 = imin(bz0 + fs.deep, a.z.nb);
  const int bxy = item % nxy;
  AdjBrick b = adj_brick_geom(a, bz0 * nxy + bxy);
  int bz = bz0;
  const int zend = adj_brick_begin(a.z, g.nz, bz1);  // the workgroup's last plane + 1
  const int lane = tid & (kWave - 1), wave = uniform(tid / kWave);

  // this lane's voxel column (x, y): forward weights and window base
  const int row = Cols == kWave ? wave : tid / Cols, col = Cols == kWave ? lane : tid - row * Cols;
  const int x = b.x0 + col, y = b.y0 + row;
  const int xc = imin(x, b.xe - 1), yc = imin(y, b.ye - 1);
  const bool act = x < b.xe && y < b.ye;
  const int tx = xc / g.dx, ty = yc / g.dy;
  float bx[4], by[4];
  {
    const float* wx = lut_row(lut, g.dx, xc - tx * g.dx);
    const float* wy = lut_row(lut, g.dy, yc - ty * g.dy);
#pragma unroll
    for (int l = 0; l < 4; ++l) bx[l] = wx[l], by[l] = wy[l];
  }
  const int pitch = a.x.cm * 3;
  const int base = (ty - b.cy0) * pitch + (tx - b.cx0) * 3;
  const FusedStage<L> map = fused_stage_map<L, kThreads>(a, b, tid);
  // the cell whose planes this wave contracts: waves 0 .. kAdjWaves - 1 at the end of
  // a z-tile, three times as many at the end of a brick
  const AdjCell cell = adj_cell_geom(a, b, wave % kAdjWaves);
  const bool any = cell.nx > 0 && cell.ny > 0;
  const AdjWeights cw = adj_cell_weights(a, cell, lut, lane);

  // Q: the 4 contracted control planes of the z-tile
  F3 Q[4];
  float st[L], s1[L], s2[L], s3[L];
  auto slot = [&](int cz) { return ring + (cz & 1) * lds.slot; };
  const auto ring_ops = fused_ring(
      [&](int cz) {
        fused_fetch<L>(grid, g, map, cz, st);
        fused_fetch<L>(grid, g, map, cz + 1, s1);
        fused_fetch<L>(grid, g, map, cz + 2, s2);
        fused_fetch<L>(grid, g, map, cz + 3, s3);
      },
      [&](int k, int cz) { fused_stage<L>(slot(cz), map, k == 0 ? st : k == 1 ? s1 : k == 2 ? s2 : s3); },
      [&](int cz) { fused_fetch<L>(grid, g, map, cz, st); },
      [&](int n, int cz) { Q[n] = fused_contract(slot(cz), base, pitch, bx, by); }, [] { __syncthreads(); });
  fused_start(g, b.cz0, zend, ring_ops);

  F3 acc[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) acc[n] = F3{0.f, 0.f, 0.f};
  // squared residuals of the z-brick, and of the bricks before it: no chain of sums grows
  // with the volume (2 x 4096 x 2000, equal residuals: relative error 2.5e-5 in one chain)
  float l2 = 0.f, loss = 0.f;
  // This lane's value of a finished plane to F[n], and the contraction of F[n] by this
  // wave's cell into the slabs, a barrier apart.
  auto put = [&](int n, const F3& v) {
    stf3(fused_smem + lds.F + (n * kFusedRows + row) * Shape::f_row + col * 3, v);
  };
  auto contract = [&](int n, int czl) {
    const float* F = fused_smem + lds.F + n * kFusedRows * Shape::f_row;
    F3 f[kAdjSteps<Shape::narrow>];
#pragma unroll
    for (int s = 0; s < kAdjSteps<Shape::narrow>; ++s) f[s] = ldf3(F + fused_f_at<Cols>(b, cell, lane, s));
    adj_cell_emit<Shape::narrow>(f, cw, slabs + adj_slab_at(a, Staged ? czl : czl & 1, wave % kAdjWaves), a.cw, a.ch, lane);
  };
  // Per voxel plane, in two stages: (a) T from the 4 contracted planes, the
  // sample's cell and the loads of its corners and of `fixed`; (b) the
  // residual, the gradient and the z-accumulation.  Within a z-tile, (a) of
  // the next plane is issued before (b) of the current one, so a wave keeps
  // one plane's loads in flight while it finishes the previous plane.  Every
  // lane loads (a lane outside the brick from its clamped column and row, and
  // a clamped sample position), so that no load is conditional and waiting
  // for one plane's loads leaves the next plane's in flight; (b) ignores the
  // values of such lanes.
  struct Pending {
    SampleIn s;
    float fx;
    float w[4];  // Bz_0..3 of the plane's offset in its tile
  };
  const size_t izs = (size_t)g.ny * g.nx;
  const size_t fxy = (size_t)yc * g.nx + xc;  // the lane's (clamped) voxel column
  const uint32_t sy = g.ny > 1 ? (uint32_t)g.nx * 4u : 0u, sz = g.nz > 1 ? (uint32_t)izs * 4u : 0u;  // Small
  auto stage_a = [&](int z, int oz) {
    Pending p;
    const float* wz = lut_row(lut, g.dz, oz);
#pragma unroll
    for (int n = 0; n < 4; ++n) p.w[n] = wz[n];
    p.fx = fixed[(size_t)z * izs + fxy];
    // T as the forward kernel forms it
    const F3 t{fmaf(p.w[3], Q[3].x, fmaf(p.w[2], Q[2].x, fmaf(p.w[1], Q[1].x, p.w[0] * Q[0].x))),
               fmaf(p.w[3], Q[3].y, fmaf(p.w[2], Q[2].y, fmaf(p.w[1], Q[1].y, p.w[0] * Q[0].y))),
               fmaf(p.w[3], Q[3].z, fmaf(p.w[2], Q[2].z, fmaf(p.w[1], Q[1].z, p.w[0] * Q[0].z)))};
    const float px = (float)x + t.x, py = (float)y + t.y, pz = (float)z + t.z;
    if constexpr (Small) p.s = trilinear_load_small<Pairs>(moving, g.nx, g.ny, g.nz, sy, sz, px, py, pz);
    else p.s = trilinear_load<Pairs>(moving, g.nx, g.ny, g.nz, px, py, pz);
    return p;
  };
  auto stage_b = [&](const Pending& p) {
    F3 d{0.f, 0.f, 0.f};
    if (act) {
      // the SSD kernel's residual and gradient
      const Sample s = trilinear_finish(p.s);
      const float res = s.w - p.fx;
      l2 = fmaf(res, res, l2);
      const float two_r = 2.f * res;
      d = F3{two_r * s.gx, two_r * s.gy, two_r * s.gz};
    }
    // the adjoint's z-accumulation
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      acc[n].x = fmaf(p.w[n], d.x, acc[n].x);
      acc[n].y = fmaf(p.w[n], d.y, acc[n].y);
      acc[n].z = fmaf(p.w[n], d.z, acc[n].z);
    }
  };

  // the np voxel planes from z of one z-tile
  auto planes = [&](int z, int np) {
    // two register sets, used in turn (a copy from one to the other would
    // wait for the loads it copies)
    Pending p0 = stage_a(z, 0);
    int k = 0;
    for (; k + 2 < np; k += 2) {
      const Pending p1 = stage_a(z + k + 1, k + 1);
      stage_b(p0);
      p0 = stage_a(z + k + 2, k + 2);
      stage_b(p1);
    }
    if (k + 1 < np) {
      const Pending p1 = stage_a(z + k + 1, k + 1);
      stage_b(p0);
      stage_b(p1);
    } else {
      stage_b(p0);
    }
  };

  // (with two-plane slabs the sum runs at every plane: 300 x 256 x 200 at spacing 1 took 633 us
  // with the windows formed there, 506 so)
  AdjWindows win;
  if constexpr (!Staged) win = adj_windows(a, AdjTiles{a}, b);
  const auto march_ops = fused_march(
      [&] {
#pragma unroll
        for (int n = 0; n < 3; ++n) Q[n] = Q[n + 1];
      },
      planes,
      [&](int n, int k) { put(n, acc[k]); },
      [&](int n, int czl, int np) {
        const int k = wave / kAdjWaves;
        if (any && k < np) contract(k == 0 ? n : k + 1, czl + k);
      },
      [&](int n) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = k + n < 4 ? acc[k + n] : F3{0.f, 0.f, 0.f};
      },
      [&](int czl, int np) {
        adj_combine_slabs(a, Staged ? adj_windows(a, AdjTiles{a}, b) : win, b, slabs, part + (size_t)(bz * nxy + bxy) * adj_brick_stride(a), czl, np,
                          Staged ? czl : czl & 1, tid, kThreads);
      },
      [&] {
        loss += l2;
        l2 = 0.f;
      });
  fused_walk<Staged>(a, bxy, zend, b, bz, ring_ops, march_ops);

  // the workgroup's loss partial: fixed-order tree
  red[tid] = loss;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {  // at most 1024 threads
    if (tid < h && tid + h < kThreads) red[tid] += red[tid + h];
    __syncthreads();
  }
  if (tid == 0) lpart[item] = red[0];
}

}  // namespace

size_t fused_workspace_bytes(const AdjGeom& a) {
  const size_t p = (adj_workspace_bytes(a) + 255) / 256 * 256;
  return p + (size_t)a.x.nb * a.y.nb * a.z.nb * sizeof(float);
}

// The fused step's tail in one launch: workgroups [0, nblk) are pass 2 (the
// fixed-order gather of each control point's partials), and with `descend`
// also the descent update grid -= eta grad of the points they gather (pass 1
// has finished reading the grid: it ran before, on the same stream); workgroup
// nblk sums the loss partials in a fixed order.
constexpr int kTailThreads = kGatherThreads;

template <bool Small>
__global__ __launch_bounds__(kTailThreads) __attribute__((amdgpu_waves_per_eu(8))) void fused_tail_kernel(
    const float* __restrict__ part, float* __restrict__ grad, float* __restrict__ grid, float eta, int descend,
    const float* __restrict__ lpart, int nlp, float* __restrict__ loss, AdjGeom a, int nblk) {
  if ((int)blockIdx.x == nblk) {
    __shared__ float red[kTailThreads];
    float acc = 0.f;
    for (int i = threadIdx.x; i < nlp; i += kTailThreads) acc += lpart[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kTailThreads / 2; h > 0; h >>= 1) {
      if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0];
    return;
  }
  adj_gather_block<Small>(part, a, AdjMap{a}, xcd_remap(blockIdx.x, nblk), threadIdx.x, [&](size_t i, const F3& gv) {
    stf3(grad + i * 3, gv);
    if (descend) {  // the descent kernel's update, on the same values
      float* p = grid + i * 3;
      stf3(p, F3{fmaf(-eta, gv.x, p[0]), fmaf(-eta, gv.y, p[1]), fmaf(-eta, gv.z, p[2])});
    }
  });
}

hipError_t launch_ssd_fused(const float* grid, const float* moving, const float* fixed, float* grad, float* loss,
                            const AdjGeom& adj, const float* lut, void* workspace, hipStream_t s, float* descend_grid,
                            float eta) {
  const AdjGeom a = fused_geom(adj);
  float* part = static_cast<float*>(workspace);
  float* lpart = reinterpret_cast<float*>(static_cast<char*>(workspace) +
                                          (adj_workspace_bytes(a) + 255) / 256 * 256);
  const FusedSplit fs = fused_split(a);
  const long items = (long)a.x.nb * a.y.nb * fs.nz;
  const int cols = fused_cols(a);
  const FusedLds lds = cols == 32 ? fused_lds<32>(a) : fused_lds<64>(a);
  const dim3 gridd((unsigned)items), block((unsigned)(kFusedRows * cols));
  const size_t bytes = (size_t)lds.total * sizeof(float);
  // 32-bit byte offsets into the images
  const bool small = (double)a.g.nx * a.g.ny * a.g.nz * 4 < 4294967296.0;
#define BSI_FUSED_LAUNCH(L, STAGED, PAIRS, COLS)                                                                    \
  do {                                                                                                               \
    const auto k = small ? &fused_pass1_kernel<L, STAGED, PAIRS, true, COLS>                                        \
                         : &fused_pass1_kernel<L, STAGED, PAIRS, false, COLS>;                                      \
    hipLaunchKernelGGL(k, gridd, block, bytes, s, grid, moving, fixed, part, lpart, a, fs, lut);                      \
  } while (0)
  // a volume one voxel wide samples its x-neighbours one by one
  const bool staged = adj_staged(a), one = fused_loads<64>(lds.slot) <= 1;
  constexpr int kMost = FusedShape<64>::max_loads;
  if (cols == 32) {
    if (fused_loads<32>(lds.slot) <= 2) BSI_FUSED_LAUNCH(2, false, 1, 32);
    else BSI_FUSED_LAUNCH(FusedShape<32>::max_loads, false, 1, 32);
  } else if (a.g.nx < 2) {
    if (staged) BSI_FUSED_LAUNCH(kMost, true, 0, 64);
    else BSI_FUSED_LAUNCH(kMost, false, 0, 64);
  } else if (one) {
    if (staged) BSI_FUSED_LAUNCH(1, true, 1, 64);
    else BSI_FUSED_LAUNCH(1, false, 1, 64);
  } else {
    if (staged) BSI_FUSED_LAUNCH(kMost, true, 1, 64);
    else BSI_FUSED_LAUNCH(kMost, false, 1, 64);
  }
#undef BSI_FUSED_LAUNCH
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t nblk = adj_gather_blocks(a);
  if (nblk + 1 > kMaxLaunchThreads / kTailThreads) return hipErrorInvalidConfiguration;  // 2^32 control points
  const auto tail = a.part_bytes != 0 ? &fused_tail_kernel<true> : &fused_tail_kernel<false>;
  hipLaunchKernelGGL(tail, dim3((unsigned)(nblk + 1)), dim3(kTailThreads), 0, s, part, grad, descend_grid, eta,
                     descend_grid != nullptr ? 1 : 0, lpart, (int)items, loss, a, (int)nblk);
  return hipGetLastError();
}

}  // namespace bsi
