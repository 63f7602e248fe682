// SSD registration step around BSI: trilinear warp, SSD loss + gradient with
// respect to the displacement field, and the gradient-descent update.
//
// p(x) = x + T(x) is formed in FP32 (the precision that decides the cell);
// corners on voxel centres, p clamped to [0, n-1]; at an exact integer p the
// cell [p, p+1] is used; a coordinate on or beyond the border (p <= 0 or
// p >= n-1) gets zero gradient.
#include "bsi_internal.h"
#include "warp_device.h"

namespace bsi {

namespace {

// Sum of v over the workgroup, in a fixed order, in thread 0: over each wave by
// lane exchanges, then the waves' sums in wave order.
__device__ __forceinline__ float col_block_sum(float v, float* red) {
#pragma unroll
  for (int h = kWave / 2; h > 0; h >>= 1) v += __shfl_down(v, h);
  const int wave = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) red[wave] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int w = 1; w < kColThreads / kWave; ++w) s += red[w];
  return s;
}

// What one pass over the voxels does: Grad: the SSD residual, its gradient and the
// loss partial; otherwise the warped image.  Small: the image is below 4 GiB.
// Bounds: reading the field and the images once and writing the result once (20
// bytes per voxel for the warp, 32 for the SSD); per voxel about 80 instructions and
// 4 gathers of 8 bytes.  Warp at 303 x 167 x 212 62 us, SSD at 294 x 130 x 208 57; one voxel
// per thread in workgroups of a row's 256 voxels, with 64-bit addresses per corner,
// took 115 (half of the workgroups with one wave at work) and 87.
template <bool Grad, bool Small, int Pairs>
__global__ __launch_bounds__(kColThreads) void sample_kernel(const float* __restrict__ field,
                                                              const float* __restrict__ image,
                                                              const float* __restrict__ fixed, VolGeom g,
                                                              ColLaunch L, float* __restrict__ out,
                                                              float* __restrict__ partials) {
  const int item = xcd_runs(blockIdx.x, gridDim.x);
  const int pb = item % L.npb, zb = item / L.npb;
  const size_t plane = (size_t)g.nx * g.ny;
  const size_t p0 = (size_t)pb * kColThreads;
  const int t = threadIdx.x;
  const bool act = p0 + t < plane;
  const int lt = act ? t : (int)(plane - 1 - p0);  // idle lanes read the last column, store nothing
  const uint32_t p = (uint32_t)p0 + (uint32_t)lt;  // below 2^32 / 3
  const int y = (int)(p / (uint32_t)g.nx), x = (int)(p - (uint32_t)y * (uint32_t)g.nx);
  const int z0 = zb * L.zchunk, z1 = min(g.nz, z0 + L.zchunk);
  const float fx = (float)x, fy = (float)y;
  const uint32_t sy = g.ny > 1 ? (uint32_t)g.nx * 4u : 0u, sz = g.nz > 1 ? (uint32_t)plane * 4u : 0u;
  auto load = [&](const F3& d, int z) {
    const float px = fx + d.x, py = fy + d.y, pz = (float)z + d.z;
    if constexpr (Small) return trilinear_load_small<Pairs>(image, g.nx, g.ny, g.nz, sy, sz, px, py, pz);
    else return trilinear_load<Pairs>(image, g.nx, g.ny, g.nz, px, py, pz);
  };
  float l2 = 0.f;
  auto finish = [&](const SampleIn& in, int z, float fix) {
    const Sample s = trilinear_finish(in);
    const size_t v = (size_t)z * plane + p0;
    if constexpr (Grad) {
      const float r = s.w - fix;
      if (act) {
        l2 = fmaf(r, r, l2);
        const float two_r = 2.f * r;
        stf3(out + v * 3 + lt * 3, F3{two_r * s.gx, two_r * s.gy, two_r * s.gz});
      }
    } else {
      if (act) out[v + lt] = s.w;
    }
  };
  auto disp = [&](int z) { return ldf3(field + ((size_t)z * plane + p0) * 3 + lt * 3); };
  auto fix = [&](int z) { return Grad ? fixed[(size_t)z * plane + p0 + lt] : 0.f; };
  // two planes at a time: their gathers are in flight together, and the next two
  // displacements with them
  F3 d0 = disp(z0), d1 = disp(min(z0 + 1, z1 - 1));
  for (int z = z0; z < z1; z += 2) {
    const SampleIn s0 = load(d0, z), s1 = load(d1, z + 1);
    const float f0 = fix(z), f1 = fix(min(z + 1, z1 - 1));
    d0 = disp(min(z + 2, z1 - 1));
    d1 = disp(min(z + 3, z1 - 1));
    finish(s0, z, f0);
    if (z + 1 < z1) finish(s1, z + 1, f1);
  }
  if constexpr (Grad) {
    __shared__ float red[kColThreads / kWave];
    const float s = col_block_sum(l2, red);
    if (t == 0) partials[blockIdx.x] = s;
  }
}

constexpr int kReduceThreads = 1024;

__global__ __launch_bounds__(kReduceThreads) void sum_kernel(const float* __restrict__ partials, long n,
                                                              float* __restrict__ out) {
  __shared__ float red[kReduceThreads];
  // 8 loads in flight: one workgroup sums up to tens of thousands of partials
  float s = 0.f;
  long i = threadIdx.x;
  for (; i + 7 * kReduceThreads < n; i += 8 * kReduceThreads) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = partials[i + k * kReduceThreads];
#pragma unroll
    for (int k = 0; k < 8; ++k) s += v[k];
  }
  for (; i < n; i += kReduceThreads) s += partials[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = kReduceThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

constexpr int kAxpyThreads = 256;

__global__ __launch_bounds__(kAxpyThreads) void descent_kernel(float* __restrict__ grid,
                                                                const float* __restrict__ grad, float eta,
                                                                int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kAxpyThreads;
  for (int64_t i = (int64_t)blockIdx.x * kAxpyThreads + threadIdx.x; i < n; i += stride)
    grid[i] = fmaf(-eta, grad[i], grid[i]);
}

template <bool Grad>
hipError_t launch_sample(const float* field, const float* image, const float* fixed, const VolGeom& g, float* out,
                         float* partials, long* blocks, hipStream_t s) {
  const ColLaunch L = make_col_launch(g);
  *blocks = (long)L.npb * L.nzb;
  if (*blocks > kMaxLaunchThreads / kColThreads) return hipErrorInvalidConfiguration;  // a field beyond device memory
  const bool small = (double)g.nx * g.ny * g.nz * 4 < 4294967296.0;
  const dim3 grid((unsigned)*blocks), block(kColThreads);
#define BSI_SAMPLE(SMALL, PAIRS) \
  hipLaunchKernelGGL((sample_kernel<Grad, SMALL, PAIRS>), grid, block, 0, s, field, image, fixed, g, L, out, partials)
  if (g.nx < 2) {  // x-neighbours as single loads
    if (small) BSI_SAMPLE(true, 0);
    else BSI_SAMPLE(false, 0);
  } else {
    if (small) BSI_SAMPLE(true, 1);
    else BSI_SAMPLE(false, 1);
  }
#undef BSI_SAMPLE
  return hipGetLastError();
}

}  // namespace

// The workspace of bsi_ssd_grad: one float per row of 256 voxels, which is at
// least the number of loss partials (sample_kernel's workgroups).
size_t ssd_partial_count(const VolGeom& g) { return (size_t)((g.nx + 255) / 256) * g.ny * g.nz; }

hipError_t launch_warp(const float* field, const float* image, const VolGeom& g, float* out,
                       hipStream_t s) {
  long blocks = 0;
  return launch_sample<false>(field, image, nullptr, g, out, nullptr, &blocks, s);
}

hipError_t launch_ssd_grad(const float* field, const float* moving, const float* fixed,
                           const VolGeom& g, float* dfield, float* loss, float* partials,
                           hipStream_t s) {
  long blocks = 0;
  hipError_t e = launch_sample<true>(field, moving, fixed, g, dfield, partials, &blocks, s);
  if (e != hipSuccess) return e;
  return launch_sum(partials, blocks, loss, s);
}

hipError_t launch_sum(const float* partials, long n, float* out, hipStream_t s) {
  hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(kReduceThreads), 0, s, partials, n, out);
  return hipGetLastError();
}

hipError_t launch_descent(float* grid, const float* grad, float eta, int64_t count, hipStream_t s) {
  int64_t blocks = (count + kAxpyThreads - 1) / kAxpyThreads;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(descent_kernel, dim3((unsigned)blocks), dim3(kAxpyThreads), 0, s, grid, grad, eta, count);
  return hipGetLastError();
}

}  // namespace bsi
