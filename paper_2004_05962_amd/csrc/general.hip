// BSI for a control grid with real spacing and an origin offset: the paper's
// method needs the grid aligned to the voxels with integer spacing (Sec. 3.4),
// the limitation its conclusion names (Sec. 8).  Per axis:
//   control point a sits at voxel o + (a - 1) s      (s >= 1, -s < o <= 0),
//   voxel x: t = (x - o) / s, window i = floor(t) .. i + 3, weights B(t - i),
//   g = floor((n - 1 - o) / s) + 4 points.
// The window start i = floor((x - o)/s) is decided exactly, from the FP32
// values of s and o, with FP32 error-free transformations (gen_locate); the
// same code runs on the host (grid size) and the device, so every decision
// agrees.  The offset u = t - i and the weights are FP32.  Nothing on the
// device is FP64.
//
// Forward: the aligned kernel's pipeline (forward.hip) with weights computed
// per coordinate instead of looked up per offset: x weights once per lane, y
// weights once per wave, and the window start and z weights of every plane of
// the workgroup's z range once, into an LDS table.  Tiles have varying voxel
// counts; the window of 4 contracted planes advances whenever floor(t_z) does
// (by one, since s >= 1), with the next plane loaded while the current tile is
// written and one barrier per tile.
//
// Adjoint: the per-axis tables i(x), B(u(x)) and the first voxel of every
// tile are computed once per call into the workspace; then the aligned
// adjoint's two passes (adjoint_device.h) over cells of up to 32 x 8 voxel columns,
// with the tables in place of equal tiles.  Deterministic, no atomics.
#include <cmath>

#include "adjoint_device.h"
#include "general_device.h"

namespace bsi {

namespace {

// Window start and the four FP32 basis weights at u (B0..B3 of Eq. 1).
__device__ __forceinline__ int gen_weights(const GenAxis& a, int v, float (&w)[4]) {
  float u;
  const int i = gen_locate(a, v, u);
  const float r = 1.f - u, u2 = u * u;
  const float sixth = 1.f / 6.f;
  w[0] = r * r * r * sixth;
  w[1] = fmaf(3.f * u2, u - 2.f, 4.f) * sixth;
  w[2] = fmaf(3.f * u, fmaf(-u, u, u) + 1.f, 1.f) * sixth;
  w[3] = u2 * u * sixth;
  return i;
}

template <class T>
struct GenFwdSmem {
  FwdSmem<3, T> f;
  float zw[kGenMaxZ][4];  // z weights of the workgroup's planes
  int zt[kGenMaxZ];       // their window start floor(t_z)
};

// Edge: rows off 64-byte boundaries, written with edge stores (FwdEdgeStore).
// T: the 4 x 1 shape for spacings of at least T::min_spacing in x and y.
template <bool Edge, class T>
__global__ __launch_bounds__(kFwdThreads) void gen_fwd_kernel(const float* __restrict__ grid,
                                                               float* __restrict__ field, VolGeom g, GenGeom q,
                                                               int nbx, int nby, int zchunk) {
  __shared__ GenFwdSmem<T> sm;
  int id = xcd_runs(blockIdx.x, gridDim.x);
  const int bxi = id % nbx;
  id /= nbx;
  const int byi = id % nby;
  const int bzi = id / nby;
  const int tid = threadIdx.x;
  const int x0 = bxi * kWave, y0 = byi * kFwdRows;
  const int z0 = bzi * zchunk, z1 = min(g.nz, z0 + zchunk);  // z1 - z0 <= kGenMaxZ
  const int lane = tid & (kWave - 1);
  const int wave = uniform(tid / kWave);
  // s >= 1: 64 voxels span at most 63 tile steps, so the window fits the
  // staging layout (at most T::max_cx x T::max_cy points)
  const int cx0 = gen_tile(q.x, x0);
  const int ncx = gen_tile(q.x, min(x0 + kWave, g.nx) - 1) - cx0 + 4;
  const int cy0 = gen_tile(q.y, y0);
  const int ncy = gen_tile(q.y, min(y0 + kFwdRows, g.ny) - 1) - cy0 + 4;
  const FwdStage<3, T> map = fwd_stage_map<3, T>(g, cx0, ncx, cy0, ncy, tid);
  for (int i = tid; i < z1 - z0; i += kFwdThreads) {
    float w[4];
    sm.zt[i] = gen_weights(q.z, z0 + i, w);
#pragma unroll
    for (int n = 0; n < 4; ++n) sm.zw[i][n] = w[n];
  }

  const int x = x0 + lane, y = y0 + wave;
  const bool active = x < g.nx && y < g.ny;
  const int xc = min(x, g.nx - 1), yc = min(y, g.ny - 1);
  float bx[4], wy[4];
  const int tx = gen_weights(q.x, xc, bx);
  const int ty = gen_weights(q.y, yc, wy);
  const int base = (ty - cy0) * fwd_pitch<3, T>() + (tx - cx0) * 3;

  int tz = gen_tile(q.z, z0);
  // Warm-up as in the aligned forward: planes tz .. tz+3 loaded together, through
  // the two slots in pairs into q0, q1, q2; plane tz+3 stays in slot 1.
  float r[fwd_loads<3, T>()];
  FwdVal<3> q0, q1, q2;
  {
    auto contract = [&](const float* slot) { return fwd_contract<3, T>(slot, base, bx[0], bx[1], bx[2], bx[3], wy); };
    float r1[fwd_loads<3, T>()], r2[fwd_loads<3, T>()], r3[fwd_loads<3, T>()];
    fwd_fetch<3, T>(grid, g, map, tz, r);
    fwd_fetch<3, T>(grid, g, map, tz + 1, r1);
    fwd_fetch<3, T>(grid, g, map, tz + 2, r2);
    fwd_fetch<3, T>(grid, g, map, tz + 3, r3);
    fwd_stage<3, T>(sm.f.ring[0], tid, r);
    fwd_stage<3, T>(sm.f.ring[1], tid, r1);
    __syncthreads();  // (also orders the z table before any read)
    q0 = contract(sm.f.ring[0]);
    q1 = contract(sm.f.ring[1]);
    __syncthreads();
    fwd_stage<3, T>(sm.f.ring[0], tid, r2);
    fwd_stage<3, T>(sm.f.ring[1], tid, r3);
    __syncthreads();
    q2 = contract(sm.f.ring[0]);
    __syncthreads();  // slot 0 is free for plane tz + 4
  }
  int slot3 = 1;

  const size_t zstride = (size_t)g.ny * g.nx * 3;
  float* out = field + (((size_t)z0 * g.ny + yc) * g.nx + xc) * 3;
  FwdEdgeStore<3> edge(field, g, z0, yc, x0, xc);
  int z = z0;
  for (;;) {
    const FwdVal<3> q3 = fwd_contract<3, T>(sm.f.ring[slot3], base, bx[0], bx[1], bx[2], bx[3], wy);
    int zend = z;  // the planes of tile tz in this chunk (s >= 1: the next one is tz + 1)
    while (zend < z1 && sm.zt[zend - z0] == tz) ++zend;
    const bool more = zend < z1;
    // its new plane tz + 4 = t_z(zend) + 3 <= gz - 1: in bounds
    if (more) fwd_fetch<3, T>(grid, g, map, tz + 4, r);
    for (; z < zend; ++z, out += zstride) {
      const float* wz = sm.zw[z - z0];
      float t[3];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        t[c] = fmaf(wz[3], q3.v[c], fmaf(wz[2], q2.v[c], fmaf(wz[1], q1.v[c], wz[0] * q0.v[c])));
      if constexpr (Edge) edge.store(active, t);
      else if (active) fwd_store<3>(out, t);
    }
    if (!more) break;
    fwd_stage<3, T>(sm.f.ring[slot3 ^ 1], tid, r);
    __syncthreads();
    slot3 ^= 1;
    ++tz;
    q0 = q1;
    q1 = q2;
    q2 = q3;
  }
}

// The three axes' tables in one launch: workgroups [0, nb[0]) take x, then y, then z.
struct GenTables3 {
  GenAxis ax[3];
  int* tile[3];
  float* w[3];
  int* first[3];
  int nb[3];  // workgroups per axis
};

// Thread k of an axis's workgroups writes entry k of its tables: tile[k] =
// i(k) and w[k] = B(u(k)) for k < n, and first[k] = min{v : i(v) >= k} for
// k <= g (first[g] = n), found by bisection on the exact i(v), so the three
// tables need no order between them.
__global__ __launch_bounds__(256) void gen_tables3_kernel(GenTables3 p) {
  int blk = blockIdx.x, i = 0;
  while (i < 2 && blk >= p.nb[i]) blk -= p.nb[i++];
  const GenAxis a = p.ax[i];
  const int k = blk * 256 + threadIdx.x;
  if (k < a.n) {
    float b[4];
    p.tile[i][k] = gen_weights(a, k, b);
#pragma unroll
    for (int s = 0; s < 4; ++s) p.w[i][4 * k + s] = b[s];
  }
  if (k <= a.g) {
    int lo = 0, hi = a.n;  // i(v) is nondecreasing in v
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (gen_tile(a, mid) < k) lo = mid + 1;
      else hi = mid;
    }
    p.first[i][k] = lo;
  }
}

// ---------------------------------------------------------------------------
// The adjoint: the aligned pass 1 and pass 2 (adjoint_device.h) with the tables.
// What bounds them is the same.  512 x 512 x 256, spacing 5.3 x 4.7 x 5.1: pass 1 164 us,
// 195 as moments per tile lane with two barriers per control plane; pass 2 12.1
// against 16; 64^3: both and the tables 19.5 us against 58; 120 x 100 x 80, spacing
// 1.5 x 1.2 x 1.1: 54 against 207.

// The cell's weight matrices from the tables (as adj_cell_weights).
__device__ __forceinline__ AdjWeights gen_cell_weights(const VolGeom& g, const AdjCell& c, const int* __restrict__ tx,
                                                       const float* __restrict__ wx, const int* __restrict__ ty,
                                                       const float* __restrict__ wy, int lane) {
  const int m = lane % kAdjTile, q = lane / kAdjTile;
  // weight of the cell's voxel v (of n, the first at v0) at control index c0 + m
  auto weight = [&](const int* tile, const float* w, int v0, int n, int v, int c0, int size) {
    const int u = gen_weight_voxel(v0, n, v, size), l = c0 + m - tile[u];
    const float b = w[4 * u + (l & 3)];
    return v < n && (uint32_t)l < 4u ? (b == 0.f ? -0.f : b) : 0.f;
  };
  AdjWeights r;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r.x[h][i] = weight(tx, wx, c.x0, c.nx, kAdjTile * h + 4 * q + i, c.cx0, g.nx);
    r.y[h] = weight(ty, wy, c.y0, c.ny, adj_step_row(h, q), c.cy0, g.ny);
  }
  return r;
}

// A wave's march along z: the plane's weights, and the end of its tile; the next
// tile's end is loaded a tile ahead.
struct GenZ {
  const float* w;
  const int* first;
  int z, t, end, next, last;
  __device__ __forceinline__ GenZ(const float* w_, const int* first_, int z0, int t0, int last_)
      : w(w_), first(first_), z(z0), t(t0), end(first_[t0 + 1]), next(first_[min(t0 + 2, last_)]), last(last_) {}
  __device__ __forceinline__ const float* weights() const { return w + 4 * z; }
  __device__ __forceinline__ bool step() {
    if (++z != end) return false;
    ++t;
    end = next;
    next = first[min(t + 2, last)];
    return true;
  }
};

template <bool Staged, bool Narrow>
__global__ __launch_bounds__(kAdjThreads) __attribute__((amdgpu_waves_per_eu(adj_wpe(Narrow)))) void gen_pass1_kernel(
    const float* __restrict__ dfield, float* __restrict__ part, AdjGeom a, const int* __restrict__ tx,
    const int* __restrict__ ty, const int* __restrict__ fz, const float* __restrict__ wx, const float* __restrict__ wy,
    const float* __restrict__ wz) {
  extern __shared__ float gen_slabs[];
  const int brick = xcd_remap(blockIdx.x, gridDim.x);
  const GenTiles tiles{tx, ty};
  const AdjBrick b = gen_brick(a, tiles, fz, brick);
  adj_brick_of<true, Staged, Narrow>(dfield, part, a, tiles, b, brick, gen_brick_cz(a, b), GenZ(wz, fz, b.z0, b.cz0, a.g.gz),
                             [&](const AdjCell& c) { return gen_cell_weights(a.g, c, tx, wx, ty, wy, threadIdx.x % kWave); },
                             gen_slabs, threadIdx.x);
}

template <bool Small>
__global__ __launch_bounds__(kGatherThreads) __attribute__((amdgpu_waves_per_eu(8))) void gen_pass2_kernel(
    const float* __restrict__ part, float* __restrict__ grad, AdjGeom a, const int* __restrict__ tx,
    const int* __restrict__ ty, const int* __restrict__ fx, const int* __restrict__ fy) {
  adj_gather_block<Small>(part, a, GenMap{a, tx, ty, fx, fy}, xcd_remap(blockIdx.x, gridDim.x), threadIdx.x,
                          [&](size_t i, const F3& v) { stf3(grad + i * 3, v); });
}

constexpr size_t align256(size_t b) { return (b + 255) / 256 * 256; }

struct GenWork {
  int* tile[3];
  float* w[3];
  int* first[3];  // first voxel of every tile, per axis (g + 1 entries)
  float* part;    // brick partials of the z-first adjoint
};

size_t gen_layout(const GenGeom& q, const AdjGeom& a, void* base, GenWork* wk) {
  char* p = static_cast<char*>(base);
  size_t off = 0;
  const GenAxis* ax[3] = {&q.x, &q.y, &q.z};
  for (int i = 0; i < 3; ++i) {
    if (wk) wk->tile[i] = reinterpret_cast<int*>(p + off);
    off += align256((size_t)ax[i]->n * sizeof(int));
    if (wk) wk->w[i] = reinterpret_cast<float*>(p + off);
    off += align256((size_t)ax[i]->n * 4 * sizeof(float));
  }
  for (int i = 0; i < 3; ++i) {
    if (wk) wk->first[i] = reinterpret_cast<int*>(p + off);
    off += align256((size_t)(ax[i]->g + 1) * sizeof(int));
  }
  if (wk) wk->part = reinterpret_cast<float*>(p + off);
  off += align256(adj_workspace_bytes(a));
  return off;
}

unsigned blocks_for(long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

int32_t make_gen_geom(const int32_t dims[3], const float spacing[3], const float origin[3], GenGeom* q, VolGeom* g) {
  if (!dims || !spacing || !origin) {
    set_error("dims, spacing and origin must be non-null");
    return BSI_ERR_INVALID_ARG;
  }
  GenAxis* ax[3] = {&q->x, &q->y, &q->z};
  for (int i = 0; i < 3; ++i) {
    const double s = spacing[i], o = origin[i];
    if (dims[i] < 1 || !std::isfinite(s) || !std::isfinite(o) || s < 1.0 || !(o <= 0.0 && o > -s)) {
      set_error("need dims >= 1, spacing >= 1 and -spacing < origin <= 0 on every axis");
      return BSI_ERR_INVALID_ARG;
    }
    if (s > BSI_MAX_SPACING || dims[i] > BSI_MAX_DIM) {
      set_error("spacing above BSI_MAX_SPACING or an axis above BSI_MAX_DIM");
      return BSI_ERR_UNSUPPORTED;
    }
    ax[i]->s = s;
    ax[i]->o = o;
    ax[i]->n = dims[i];
    ax[i]->g = gen_tile(*ax[i], dims[i] - 1) + 4;
  }
  const double rows = (double)dims[1] * dims[2];
  if (rows > 2.0e9 || rows * dims[0] * 3 > 9.0e18 / 16) {
    set_error("volume too large");
    return BSI_ERR_UNSUPPORTED;
  }
  g->nx = dims[0];
  g->ny = dims[1];
  g->nz = dims[2];
  g->dx = g->dy = g->dz = 1;  // unused: the general kernels take tiles from q
  g->gx = q->x.g;
  g->gy = q->y.g;
  g->gz = q->z.g;
  // the forward's staging map is the aligned forward's (signed 32-bit offsets)
  if ((double)g->nx * g->ny * 3 >= 4294967296.0) {
    set_error("a voxel plane (nx * ny) above 1.43e9 voxels");
    return BSI_ERR_UNSUPPORTED;
  }
  return check_control_plane(g->gx, g->gy);
}

FwdLaunch make_gen_fwd_launch(const VolGeom& g, const GenGeom& q, bool aligned) {
  const int nbx = (g.nx + kWave - 1) / kWave, nby = (g.ny + kFwdRows - 1) / kFwdRows;
  const long base = (long)nbx * nby;
  int chunks = (int)((kFwdTargetBlocks + base - 1) / base);
  chunks = std::max(chunks, (g.nz + kGenMaxZ - 1) / kGenMaxZ);  // the z table holds kGenMaxZ planes
  // chunks of about 25 planes, 48 where a tile holds fewer than 4, as in the aligned
  // forward (512 x 512 x 256, spacing 5.3 x 4.7 x 5.1: 153 us with 25, 167 with the
  // 128 that the target leaves; 512 x 300 x 200, spacing 4: 76 and 82; 512 x 512 x 256,
  // spacing 3: 163 with 48, 177 with 25; fewer than 3: 72, spacing 2: 192 us against 201).
  // Rows off 64-byte boundaries: 50 planes, and at
  // least 4 tiles (510 x 512 x 256, spacing 5.3 x 4.7 x 5.1: 150 us with 50, 165 with 25; spacing
  // 10.5 on every axis 131 and 143; 301 x 300 x 300, 1.5 x 1.5 x 12.5: 64 and 70).
  const int planes = q.z.s < 3.f && aligned ? 72
                     : q.z.s < 4.f          ? 48
                     : aligned              ? 25
                                            : std::max(50, (int)(4.f * q.z.s));
  // (narrow volumes of very many rows: as many chunks as a launch's threads allow)
  const long most = std::max(1L, (long)(kMaxLaunchThreads / ((int64_t)kFwdThreads * base)));
  chunks = std::max(chunks, (int)std::min<long>(most, (g.nz + planes - 1) / planes));
  chunks = std::max(1, std::min(chunks, g.nz));
  const int zchunk = (g.nz + chunks - 1) / chunks;
  return FwdLaunch{nbx, nby, (g.nz + zchunk - 1) / zchunk, zchunk};
}

hipError_t launch_forward_general(const float* grid, float* field, const VolGeom& g, const GenGeom& q,
                                  hipStream_t s) {
  // rows on 64-byte boundaries: non-temporal stores; otherwise edge stores
  const bool aligned = (g.nx * 12) % 64 == 0 && reinterpret_cast<uintptr_t>(field) % 64 == 0;
  const auto [nbx, nby, nbz, zchunk] = make_gen_fwd_launch(g, q, aligned);
  const dim3 gd((unsigned)((long)nbx * nby * nbz)), bd(kFwdThreads);
  using T1 = FwdTile<kFwdRows, 1, 1>;
  using T3 = FwdTile<kFwdRows, 1, 1, 3>;
  if (q.x.s >= 3.f && q.y.s >= 3.f) {
    if (aligned) hipLaunchKernelGGL((gen_fwd_kernel<false, T3>), gd, bd, 0, s, grid, field, g, q, nbx, nby, zchunk);
    else hipLaunchKernelGGL((gen_fwd_kernel<true, T3>), gd, bd, 0, s, grid, field, g, q, nbx, nby, zchunk);
  } else {
    if (aligned) hipLaunchKernelGGL((gen_fwd_kernel<false, T1>), gd, bd, 0, s, grid, field, g, q, nbx, nby, zchunk);
    else hipLaunchKernelGGL((gen_fwd_kernel<true, T1>), gd, bd, 0, s, grid, field, g, q, nbx, nby, zchunk);
  }
  return hipGetLastError();
}

size_t general_workspace_bytes(const GenGeom& q, const VolGeom& g) {
  return gen_layout(q, make_gen_adj(q, g), nullptr, nullptr);
}

hipError_t launch_adjoint_general(const float* dfield, float* grad, const GenGeom& q, const VolGeom& g, void* workspace,
                                  hipStream_t s) {
  const AdjGeom a = make_gen_adj(q, g);
  const int64_t nbricks = (int64_t)a.x.nb * a.y.nb * a.z.nb, nblk = adj_gather_blocks(a);
  if (nbricks > kMaxLaunchThreads / kAdjThreads || nblk > kMaxLaunchThreads / kGatherThreads) return hipErrorInvalidValue;
  GenWork wk;
  gen_layout(q, a, workspace, &wk);
  GenTables3 tp;
  const GenAxis* ax[3] = {&q.x, &q.y, &q.z};
  for (int i = 0; i < 3; ++i) {
    tp.ax[i] = *ax[i];
    tp.tile[i] = wk.tile[i];
    tp.w[i] = wk.w[i];
    tp.first[i] = wk.first[i];
    tp.nb[i] = (int)blocks_for(std::max(ax[i]->n, ax[i]->g + 1));
  }
  hipLaunchKernelGGL(gen_tables3_kernel, dim3((unsigned)(tp.nb[0] + tp.nb[1] + tp.nb[2])), dim3(256), 0, s, tp);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const auto pass1 = adj_narrow(a) ? (adj_staged(a) ? &gen_pass1_kernel<true, true> : &gen_pass1_kernel<false, true>)
                                   : (adj_staged(a) ? &gen_pass1_kernel<true, false> : &gen_pass1_kernel<false, false>);
  hipLaunchKernelGGL(pass1, dim3((unsigned)nbricks), dim3(kAdjThreads), adj_lds_bytes(a), s, dfield, wk.part, a,
                     wk.tile[0], wk.tile[1], wk.first[2], wk.w[0], wk.w[1], wk.w[2]);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const auto pass2 = a.part_bytes != 0 ? &gen_pass2_kernel<true> : &gen_pass2_kernel<false>;
  hipLaunchKernelGGL(pass2, dim3((unsigned)nblk), dim3(kGatherThreads), 0, s, wk.part, grad, a, wk.tile[0], wk.tile[1],
                     wk.first[0], wk.first[1]);
  return hipGetLastError();
}

}  // namespace bsi
