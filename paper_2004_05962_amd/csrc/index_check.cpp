// Host-side check of the kernels' index arithmetic (test infrastructure).
//
// Runs, on the CPU, the same geometry functions and __host__ __device__
// address helpers the kernels use, for every workgroup / lane / control point
// of a launch, and checks that every global load and store lies inside its
// buffer (dfield, field, grid, workspace), that every LDS index lies inside
// its array, and that pass 2 reads only partials pass 1 wrote.  Nothing here
// touches a device.  Built next to libbsi.so and called by the CPU tests.
#include <cstdio>
#include <string>
#include <vector>

#include "adjoint_device.h"
#include "bsi_internal.h"
#include "fused_device.h"
#include "general_device.h"
#include "warp_device.h"

namespace bsi {
namespace {

struct Check {
  std::string msg;
  bool ok = true;
  bool fail(const std::string& m) {
    if (ok) msg = m;
    ok = false;
    return false;
  }
};

#define REQUIRE(c, what)                                                         \
  do {                                                                           \
    if (!(c)) return ck.fail(std::string(what) + " [" #c "]");                   \
  } while (0)

// Loads and LDS indices of pass 1 (adj_brick_of) for one brick of cz control planes.
template <bool Narrow, class Tiles>
bool check_brick_lanes(const AdjGeom& a, const Tiles& tiles, const AdjBrick& b, int cz, Check& ck) {
  const VolGeom& g = a.g;
  const size_t plane = (size_t)g.nx * g.ny * 12;
  const size_t lds = adj_lds_bytes(a) / sizeof(float);
  REQUIRE(cz <= a.z.cm && b.Cx <= a.x.cm && b.Cy <= a.y.cm, "window within the partials' extents");
  REQUIRE(b.ye - b.y0 <= kAdjCellsY * kAdjCellY && b.xe - b.x0 <= kAdjCellsX * a.cell, "brick within its cells");
  REQUIRE(a.slots >= 2 && (!adj_staged(a) || cz <= a.slots), "slots for the brick's planes");
  REQUIRE(adj_lds_bytes(a) <= 80000, "LDS request of two workgroups per CU");
  std::vector<int> voxels((size_t)(b.xe - b.x0) * (b.ye - b.y0), 0), points((size_t)b.Cx * b.Cy, 0);
  for (int w = 0; w < kAdjWaves; ++w) {
    const AdjCell c = adj_cell_of(a, tiles, b, w);
    const bool any = c.nx > 0 && c.ny > 0;
    if (adj_staged(a) && !any) continue;  // the wave only meets the barrier
    REQUIRE(c.Cx <= kAdjTile && c.Cx <= a.cw && c.Cy <= kAdjTile && c.Cy <= a.ch,
            "window within a matrix tile and the slab");
    if (any) {
      REQUIRE(c.cx0 >= b.cx0 && c.cx0 + c.Cx <= b.cx0 + b.Cx && c.cy0 >= b.cy0 && c.cy0 + c.Cy <= b.cy0 + b.Cy,
              "cell window within the brick's");
      for (int j = 0; j < c.Cy; ++j)
        for (int i = 0; i < c.Cx; ++i) points[(size_t)(c.cy0 - b.cy0 + j) * b.Cx + c.cx0 - b.cx0 + i] = 1;
      // a slab entry of the last slot, row and column
      REQUIRE((size_t)adj_slab_at(a, a.slots - 1, w) + adj_slab(a) <= lds, "slab store outside the LDS request");
      REQUIRE(a.cw % 4 == 0 && adj_slab_point(a, 2, a.ch - 1, a.cw - 4) + 4 <= adj_slab(a), "slab store outside its slab");
      REQUIRE(a.ch <= kAdjTile && a.cw <= kAdjTile && adj_slab_point(a, 2, c.Cy - 1, c.Cx - 1) < adj_slab(a),
              "slab read outside its slab");
      // the fused step reads the finished plane's voxels of the cell from F, 16 rows of 64
      REQUIRE(c.x0 - b.x0 + kAdjCellX <= kWave && c.y0 - b.y0 + kAdjCellY <= kAdjCellsY * kAdjCellY,
              "cell within the fused step's rows");
    }
    const int cnx = any ? c.nx : 1, cny = any ? c.ny : 1;
    const size_t base = ((size_t)(any ? c.y0 : b.y0) * g.nx + (any ? c.x0 : b.x0)) * 12;
    for (int lane = 0; lane < kWave; ++lane) {
      uint32_t off[kAdjSteps<Narrow>];
      adj_cell_offsets<Narrow>(g.nx, cnx, cny, lane, off);
      for (int s = 0; s < kAdjSteps<Narrow>; ++s) {
        REQUIRE(base + off[s] + 12 <= plane, "pass-1 load outside its voxel plane");
        REQUIRE(off[s] + 12 <= adj_cell_bytes(g.nx, cnx, cny), "pass-1 load outside its buffer");
        const size_t v = (base + off[s]) / 12;
        const int x = (int)(v % g.nx), y = (int)(v / g.nx);
        REQUIRE(x >= b.x0 && x < b.xe && y >= b.y0 && y < b.ye, "pass-1 load outside its brick");
        const int col = adj_lane_col<Narrow>(lane), row = adj_lane_row<Narrow>(lane, s);
        if (any && col < c.nx && row < c.ny) {
          REQUIRE(x == c.x0 + col && y == c.y0 + row, "pass-1 lane's voxel");
          ++voxels[(size_t)(y - b.y0) * (b.xe - b.x0) + x - b.x0];
        }
      }
    }
  }
  for (int n : voxels) REQUIRE(n == 1, "every voxel of the brick has one lane");
  for (int n : points) REQUIRE(n == 1, "every window point of the brick lies in a cell's window");
  // the rows that the first product's steps take: each of the cell's rows once
  int rows = 0;
  for (int t = 0; t < 2; ++t)
    for (int k = 0; k < 4; ++k) rows |= 1 << adj_step_row(t, k);
  REQUIRE(rows == (1 << kAdjCellY) - 1, "product steps cover the cell's rows");
  return true;
}

template <class Tiles>
bool check_brick(const AdjGeom& a, const Tiles& tiles, const AdjBrick& b, int cz, Check& ck) {
  return adj_narrow(a) ? check_brick_lanes<true>(a, tiles, b, cz, ck) : check_brick_lanes<false>(a, tiles, b, cz, ck);
}

bool check_adj_brick(const AdjGeom& a, const AdjBrick& b, Check& ck) {
  REQUIRE(b.z0 == b.cz0 * a.g.dz, "z-bricks start on tile boundaries (the march starts at offset 0)");
  return check_brick(a, AdjTiles{a}, b, adj_brick_cz(a, b), ck);
}

// Pass 2's offsets in 32 bits with up to three bricks past their spans, and its
// workgroups: every control point taken exactly once.
bool check_gather(const AdjGeom& a, Check& ck) {
  const VolGeom& g = a.g;
  const size_t ws = adj_workspace_bytes(a) / sizeof(float);
  static_assert(4 * (uint64_t)kAdjGatherSmall <= (uint64_t)1 << 32);
  REQUIRE(a.part_bytes == (ws * 4 <= kAdjGatherSmall ? ws * 4 : 0), "pass-2 buffer over the partials");
  REQUIRE(a.lx >= 0 || (a.part_bytes != 0 && (int64_t)g.gx * g.gy * g.gz <= 1 << 20), "points of the wave-per-point form");
  {
    std::vector<unsigned char> hit((size_t)g.gx * g.gy * g.gz, 0);
    const int64_t nblk = adj_gather_blocks(a);
    REQUIRE(nblk < ((int64_t)1 << 31), "pass-2 grid above 2^31 workgroups");
    for (int64_t blk = 0; blk < nblk; ++blk)
      for (int t = 0; t < kGatherThreads; t += a.lx < 0 ? kWave : 1) {
        int cx, cy, cz;
        if (!adj_gather_index(a, (int)blk, t, cx, cy, cz)) continue;
        REQUIRE(0 <= cx && cx < g.gx && 0 <= cy && cy < g.gy && 0 <= cz && cz < g.gz, "pass-2 point off the grid");
        unsigned char& h = hit[((size_t)cz * g.gy + cy) * g.gx + cx];
        REQUIRE(h == 0, "pass-2 point taken twice");
        h = 1;
      }
    for (unsigned char h : hit) REQUIRE(h == 1, "pass-2 point never taken");
  }
  return true;
}

// Pass 1 (its bricks, via `brick_check`) and pass 2 of a two-pass adjoint with
// brick geometry `a`.
template <class BrickCheck>
bool check_adjoint(const AdjGeom& a, BrickCheck brick_check, Check& ck) {
  const VolGeom& g = a.g;
  const size_t ws = adj_workspace_bytes(a) / sizeof(float);
  const int nb = a.x.nb * a.y.nb * a.z.nb;
  REQUIRE(a.x.nb >= 1 && a.y.nb >= 1 && a.z.nb >= 1, "brick counts");
  REQUIRE((size_t)nb * adj_brick_stride(a) == ws, "workspace holds the bricks");
  // the window of every brick, as pass 1 writes it
  std::vector<int> Cx(nb), Cy(nb), Cz(nb);
  long voxels = 0;
  for (int id = 0; id < nb; ++id) {
    const AdjBrick b = adj_brick_geom(a, id);
    REQUIRE(0 <= b.x0 && b.x0 < b.xe && b.xe <= g.nx, "brick x range");
    REQUIRE(0 <= b.y0 && b.y0 < b.ye && b.ye <= g.ny, "brick y range");
    REQUIRE(0 <= b.z0 && b.z0 < b.ze && b.ze <= g.nz, "brick z range");
    REQUIRE(b.Cx <= a.x.cm, "x window (partials stride)");
    REQUIRE(b.Cy <= a.y.cm, "y window (partials stride)");
    const int cz = adj_brick_cz(a, b);
    REQUIRE(cz <= a.z.cm, "z window (partials stride)");
    REQUIRE(b.cx0 + b.Cx <= g.gx && b.cy0 + b.Cy <= g.gy && b.cz0 + cz <= g.gz, "window inside the grid");
    REQUIRE(b.cx0 == adj_brick_c0(a.x, id % a.x.nb, g.dx), "x window start");
    REQUIRE(b.cy0 == adj_brick_c0(a.y, id / a.x.nb % a.y.nb, g.dy), "y window start");
    REQUIRE(b.cz0 == adj_brick_c0(a.z, id / (a.x.nb * a.y.nb), g.dz), "z window start");
    const size_t last = (size_t)id * adj_brick_stride(a) + adj_part_offset(a, cz - 1, b.Cy - 1, b.Cx - 1);
    REQUIRE(last + 3 <= ws, "partial store outside the workspace");
    if (!brick_check(a, b, ck)) return false;
    Cx[id] = b.Cx;
    Cy[id] = b.Cy;
    Cz[id] = cz;
    voxels += (long)(b.xe - b.x0) * (b.ye - b.y0) * (b.ze - b.z0);
  }
  REQUIRE(voxels == (long)g.nx * g.ny * g.nz, "bricks tile the volume");
  // per axis: brick b meets the support [(c-3)d, (c+1)d) of control index c
  // exactly when b lies in c's span (pass 2 misses no brick and adds no other)
  const AdjAxis* axes[3] = {&a.x, &a.y, &a.z};
  const int nn[3] = {g.nx, g.ny, g.nz}, dd[3] = {g.dx, g.dy, g.dz}, gg[3] = {g.gx, g.gy, g.gz};
  for (int ax = 0; ax < 3; ++ax)
    for (int c = 0; c < gg[ax]; ++c) {
      const AdjSpan sp = adj_span(*axes[ax], c, dd[ax], nn[ax]);
      const int lo = imax(0, (c - 3) * dd[ax]), hi = imin(nn[ax], (c + 1) * dd[ax]);
      for (int b = 0; b < axes[ax]->nb; ++b) {
        const int b0 = adj_brick_begin(*axes[ax], nn[ax], b), b1 = adj_brick_begin(*axes[ax], nn[ax], b + 1);
        const bool meets = b0 < hi && lo < b1;
        REQUIRE(meets == (b >= sp.lo && b <= sp.hi), "pass-2 span differs from the bricks meeting the support");
      }
    }
  if (!check_gather(a, ck)) return false;
  // pass 2: every brick a control point reads holds that point in its window
  for (int cz = 0; cz < g.gz; ++cz)
    for (int cy = 0; cy < g.gy; ++cy)
      for (int cx = 0; cx < g.gx; ++cx) {
        const AdjSpan sx = adj_span(a.x, cx, g.dx, g.nx), sy = adj_span(a.y, cy, g.dy, g.ny),
                      sz = adj_span(a.z, cz, g.dz, g.nz);
        REQUIRE(0 <= sx.lo && sx.lo <= sx.hi && sx.hi < a.x.nb, "x span");
        REQUIRE(0 <= sy.lo && sy.lo <= sy.hi && sy.hi < a.y.nb, "y span");
        REQUIRE(0 <= sz.lo && sz.lo <= sz.hi && sz.hi < a.z.nb, "z span");
        for (int bz = sz.lo; bz <= sz.hi; ++bz)
          for (int by = sy.lo; by <= sy.hi; ++by)
            for (int bx = sx.lo; bx <= sx.hi; ++bx) {
              const int id = (bz * a.y.nb + by) * a.x.nb + bx;
              const int cxl = cx - adj_brick_c0(a.x, bx, g.dx), cyl = cy - adj_brick_c0(a.y, by, g.dy),
                        czl = cz - adj_brick_c0(a.z, bz, g.dz);
              REQUIRE(0 <= cxl && cxl < Cx[id] && 0 <= cyl && cyl < Cy[id] && 0 <= czl && czl < Cz[id],
                      "pass 2 reads a partial pass 1 did not write");
              REQUIRE(adj_part_addr(a, bx, by, bz, cx, cy, cz) + 3 <= ws, "pass-2 load outside the workspace");
            }
      }
  return true;
}

// The sampling kernels' columns and z-chunks, and their loss partials.
bool check_columns(const VolGeom& g, Check& ck) {
  const ColLaunch c = make_col_launch(g);
  const int64_t plane = (int64_t)g.nx * g.ny;
  REQUIRE(c.npb >= 1 && (int64_t)c.npb * kColThreads >= plane && (int64_t)(c.npb - 1) * kColThreads < plane,
          "column blocks cover the plane");
  REQUIRE(c.nzb >= 1 && c.zchunk >= 1 && (int64_t)c.nzb * c.zchunk >= g.nz && (int64_t)(c.nzb - 1) * c.zchunk < g.nz,
          "z-chunks cover the volume");
  REQUIRE((size_t)c.npb * c.nzb <= ssd_partial_count(g), "loss partials within the SSD workspace");
  return true;
}

bool check_adjoints(const VolGeom& g, Check& ck) { return check_adjoint(make_adj_geom(g), check_adj_brick, ck); }

// The marching forward (fwd_block) with workgroup shape T and C components.
template <int C, class T>
bool check_forward_march(const VolGeom& g, Check& ck, long target = kFwdTargetBlocks,
                         int planes = T::strips > 1 ? kFwdChunkWide : kFwdChunk) {
  const FwdLaunch L = make_fwd_launch(g, target, T::width, T::rows, planes);
  REQUIRE(L.zchunk % g.dz == 0 && L.zchunk > 0, "z chunks of whole tiles");
  REQUIRE((long)L.nbz * L.zchunk >= g.nz && (long)(L.nbz - 1) * L.zchunk < g.nz, "z chunks cover the volume");
  const size_t cplane = (size_t)g.gx * g.gy * C;
  for (int bz = 0; bz < L.nbz; ++bz)
    for (int by = 0; by < L.nby; ++by)
      for (int bx = 0; bx < L.nbx; ++bx) {
        const int x0 = bx * T::width, y0 = by * T::rows, z0 = bz * L.zchunk, z1 = imin(g.nz, z0 + L.zchunk);
        REQUIRE(x0 < g.nx && y0 < g.ny && z0 < z1, "forward workgroup inside the volume");
        const FwdWindow w = fwd_window(g, x0, y0, T::width, T::rows);
        REQUIRE(w.ncx <= T::max_cx && w.ncy <= T::max_cy, "forward window within the staging capacity");
        REQUIRE(w.cx0 + w.ncx <= g.gx && w.cy0 + w.ncy <= g.gy, "forward window inside the grid");
        // planes read: tiles z0/dz .. (z1-1)/dz, each with its 3 successors
        REQUIRE((z1 - 1) / g.dz + 3 < g.gz, "forward planes inside the grid");
        if (bz == 0 && by == 0)  // the staging map depends on the column window only through cx0, ncx
          for (int tid = 0; tid < T::threads; ++tid) {
            const FwdStage<C, T> m = fwd_stage_map<C, T>(g, w.cx0, w.ncx, w.cy0, w.ncy, tid);
            for (int k = 0; k < fwd_loads<C, T>(); ++k)
              REQUIRE(m.goff[k] < 0 || (size_t)m.goff[k] < cplane, "staged load outside its control plane");
          }
      }
  return true;
}

// The span forward: every span's control window and LDS request.
template <int C>
bool check_forward_span(const VolGeom& g, Check& ck) {
  const int R = span_rows(g, C);
  if (R == 0) return true;  // the span kernel is not used for this geometry
  REQUIRE((double)R * g.nx * C * 4 < 2147483648.0, "span bytes fit the buffer record");
  REQUIRE((g.nx - 1) / g.dx + 3 < g.gx, "span columns inside the grid");
  const int nyb = (g.ny + R - 1) / R;
  for (int yb = 0; yb < nyb; ++yb) {
    const int y0 = yb * R, y1 = imin(g.ny, y0 + R);
    REQUIRE(y0 < y1, "span rows inside the volume");
    for (int z = 0; z < g.nz; ++z) {
      const FwdSpanWindow w = fwd_span_window(g, z, y0, y1);
      REQUIRE(w.tz + 3 < g.gz, "span planes inside the grid");
      REQUIRE(w.ty0 + w.nry <= g.gy, "span control rows inside the grid");
      REQUIRE(w.nry <= fwd_span_ctl_rows(R, g.dy), "span window within its LDS request");
      REQUIRE((size_t)(w.nry + (y1 - y0)) * g.gx * C * sizeof(float) <= fwd_span_lds(R, g.dy, g.gx, C),
              "span LDS use within the request");
    }
  }
  return true;
}

// The shape's instances for every smallest spacing that the geometry allows.
template <int C, int R, int S, int V>
bool check_forward_shape(const VolGeom& g, Check& ck, long target = kFwdTargetBlocks,
                         int planes = S > 1 ? kFwdChunkWide : kFwdChunk) {
  const int d = imin(g.dx, g.dy);
  return check_forward_march<C, FwdTile<R, S, V>>(g, ck, target, planes) &&
         (d < 2 || check_forward_march<C, FwdTile<R, S, V, 2>>(g, ck, target, planes)) &&
         (d < 3 || check_forward_march<C, FwdTile<R, S, V, 3>>(g, ck, target, planes)) &&
         (d < 4 || check_forward_march<C, FwdTile<R, S, V, 4>>(g, ck, target, planes)) &&
         (d < 5 || check_forward_march<C, FwdTile<R, S, V, 5>>(g, ck, target, planes));
}

// The batched forward's shapes and z-split targets (the schedule knobs).
bool check_forward_batched(const VolGeom& g, Check& ck) {
  for (const auto& [target, planes] : {std::pair{512L, 0}, {2048L, 0}, {(long)kFwdLeastItems, kFwdChunkBatch}})
    if (!(check_forward_shape<3, 4, 1, 1>(g, ck, target, planes) && check_forward_shape<3, 2, 2, 1>(g, ck, target, planes) &&
          check_forward_shape<3, 8, 1, 1>(g, ck, target, planes)))
      return false;
  return true;
}

bool check_forward(const VolGeom& g, Check& ck) {
  return check_forward_shape<3, kFwdRows, 1, 1>(g, ck) && check_forward_shape<3, 2, 8, 1>(g, ck) &&
         check_forward_shape<1, kFwdRows, 1, 4>(g, ck) && check_forward_shape<1, kFwdRows, 1, 1>(g, ck) &&
         check_forward_span<3>(g, ck) && check_forward_span<1>(g, ck) && check_forward_batched(g, ck);
}

// The adjoint of the real-spacing grid (general.hip): its bricks, cells, LDS
// request, partial offsets and pass-2 spans, with host tables built by the
// same exact window-start function the device uses.
bool check_general_adjoint(const GenGeom& q, const VolGeom& vol, Check& ck) {
  const GenAxis* ax[3] = {&q.x, &q.y, &q.z};
  std::vector<int> tile[3], first[3];
  for (int i = 0; i < 3; ++i) {
    const GenAxis& A = *ax[i];
    tile[i].resize((size_t)A.n);
    for (int v = 0; v < A.n; ++v) tile[i][(size_t)v] = gen_tile(A, v);
    REQUIRE(tile[i][0] == 0 && tile[i][(size_t)A.n - 1] == A.g - 4, "window starts span the grid");
    for (int v = 1; v < A.n; ++v) {
      const int d = tile[i][(size_t)v] - tile[i][(size_t)v - 1];
      REQUIRE(d == 0 || d == 1, "window starts step by 0 or 1 (spacing >= 1)");
    }
    first[i].resize((size_t)A.g + 1);
    for (int t = 0; t <= A.g; ++t) {
      int lo = 0, hi = A.n;
      while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (tile[i][(size_t)mid] < t) lo = mid + 1;
        else hi = mid;
      }
      first[i][(size_t)t] = lo;
    }
  }
  // the forward's window of 64 voxels x 4 rows within its staging capacity
  {
    using T1 = FwdTile<kFwdRows, 1, 1>;
    using T3 = FwdTile<kFwdRows, 1, 1, 3>;
    const bool three = q.x.s >= 3.f && q.y.s >= 3.f;
    for (int x0 = 0; x0 < q.x.n; x0 += kWave) {
      const int n = tile[0][(size_t)imin(x0 + kWave, q.x.n) - 1] - tile[0][(size_t)x0] + 4;
      REQUIRE(n <= (three ? T3::max_cx : T1::max_cx), "forward window columns");
    }
    for (int y0 = 0; y0 < q.y.n; y0 += kFwdRows) {
      const int n = tile[1][(size_t)imin(y0 + kFwdRows, q.y.n) - 1] - tile[1][(size_t)y0] + 4;
      REQUIRE(n <= (three ? T3::max_cy : T1::max_cy), "forward window rows");
    }
  }
  const AdjGeom a = make_gen_adj(q, vol);
  const GenTiles tiles{tile[0].data(), tile[1].data()};
  const size_t ws = adj_workspace_bytes(a) / sizeof(float);
  REQUIRE(a.z.nb * a.z.k >= q.z.g - 3 && (a.z.nb - 1) * a.z.k < q.z.g - 3, "z-bricks cover the z-tiles");
  const long nbricks = (long)a.x.nb * a.y.nb * a.z.nb;
  REQUIRE(nbricks < (1L << 31), "pass-1 grid");
  std::vector<int> Cx((size_t)a.x.nb), Cy((size_t)a.y.nb), Cz((size_t)a.z.nb);
  long voxels = 0;
  for (long id = 0; id < nbricks; ++id) {
    const AdjBrick b = gen_brick(a, tiles, first[2].data(), (int)id);
    REQUIRE(b.x0 < b.xe && b.y0 < b.ye && b.z0 < b.ze && b.xe <= q.x.n && b.ye <= q.y.n && b.ze <= q.z.n,
            "brick inside the volume");
    REQUIRE(tile[2][(size_t)b.z0] == b.cz0 && (b.z0 == 0 || tile[2][(size_t)b.z0 - 1] < b.cz0),
            "z-bricks start on tile boundaries");
    REQUIRE(tile[2][(size_t)b.ze - 1] - b.cz0 + 4 == gen_brick_cz(a, b), "control planes of the brick");
    if (!check_brick(a, tiles, b, gen_brick_cz(a, b), ck)) return false;
    for (int w = 0; w < kAdjWaves; ++w) {
      const AdjCell c = adj_cell_of(a, tiles, b, w);
      if (adj_staged(a) && (c.nx <= 0 || c.ny <= 0)) continue;  // the wave reads no weights
      for (int v = 0; v < kAdjCellX; ++v) {
        const int ux = gen_weight_voxel(c.x0, c.nx, v, q.x.n), uy = gen_weight_voxel(c.y0, c.ny, v % kAdjCellY, q.y.n);
        REQUIRE(0 <= ux && ux < q.x.n && 0 <= uy && uy < q.y.n, "cell weights read outside the axis's tables");
        REQUIRE(v >= c.nx || ux == c.x0 + v, "cell weights of the lane's voxel");
        REQUIRE(v >= c.ny || v >= kAdjCellY || uy == c.y0 + v, "cell weights of the lane's row");
      }
    }
    Cx[(size_t)(id % a.x.nb)] = b.Cx;
    Cy[(size_t)(id / a.x.nb % a.y.nb)] = b.Cy;
    Cz[(size_t)(id / a.x.nb / a.y.nb)] = gen_brick_cz(a, b);
    voxels += (long)(b.xe - b.x0) * (b.ye - b.y0) * (b.ze - b.z0);
  }
  REQUIRE(voxels == (long)q.x.n * q.y.n * q.z.n, "bricks tile the volume");
  // the march along z: every step's tile end is read inside the table (GenZ)
  REQUIRE((int)first[2].size() == q.z.g + 1, "first-voxel table");
  if (!check_gather(a, ck)) return false;
  // pass 2, per axis: a brick lies in c's span exactly when its voxels meet c's
  // support, and then its window holds c
  const GenMap map{a, tile[0].data(), tile[1].data(), first[0].data(), first[1].data()};
  for (int i = 0; i < 3; ++i)
    for (int c = 0; c < ax[i]->g; ++c) {
      const AdjSpan sp = i == 0 ? map.span_x(c) : i == 1 ? map.span_y(c) : map.span_z(c);
      const AdjAxis& X = i == 0 ? a.x : i == 1 ? a.y : a.z;
      const int lo = first[i][(size_t)imax(0, c - 3)], hi = first[i][(size_t)c + 1];
      REQUIRE(0 <= sp.lo && sp.lo <= sp.hi && sp.hi < X.nb, "pass-2 span");
      for (int b = 0; b < X.nb; ++b) {
        const int b0 = i == 2 ? first[2][(size_t)(b * X.k)] : b * X.w;
        const int b1 = i == 2 ? first[2][(size_t)imin((b + 1) * X.k, q.z.g - 3)] : imin(ax[i]->n, (b + 1) * X.w);
        REQUIRE((b0 < hi && lo < b1) == (b >= sp.lo && b <= sp.hi), "pass-2 span differs from the bricks meeting the support");
        if (b < sp.lo || b > sp.hi) continue;
        const int c0 = i == 2 ? b * X.k : tile[i][(size_t)b0];
        const int window = i == 0 ? Cx[(size_t)b] : i == 1 ? Cy[(size_t)b] : Cz[(size_t)b];
        REQUIRE(c - c0 >= 0 && c - c0 < window, "pass 2 reads a partial pass 1 did not write");
      }
    }
  REQUIRE(map.part_x(a.x.nb - 1, tile[0][(size_t)((a.x.nb - 1) * a.x.w)] + a.x.cm - 1) +
                  map.part_y(a.y.nb - 1, tile[1][(size_t)((a.y.nb - 1) * a.y.w)] + a.y.cm - 1) +
                  map.part_z(a.z.nb - 1, (a.z.nb - 1) * a.z.k + a.z.cm - 1) + 3 <= ws,
          "pass-2 load outside the workspace");
  return true;
}

// One LDS region of the fused step: what it holds, and the barrier interval of its
// last store and read.  A store and another access of one region lie in different
// intervals; a read finds the plane it is meant for.
struct LdsRegion {
  int holds = -1, stored = -1, read = -1;
  bool store(int what, int now) {
    const bool ok = stored < now && read < now;
    holds = what;
    stored = now;
    return ok;
  }
  bool load(int what, int now) {
    read = now;
    return holds == what && stored < now;
  }
};

// The order of the fused step's LDS accesses (fused_start, fused_walk) for one workgroup.
template <bool Staged>
bool check_fused_walk(const AdjGeom& a, int bxy, int bz0, int bz1, Check& ck) {
  const VolGeom& g = a.g;
  const int nxy = a.x.nb * a.y.nb, zend = adj_brick_begin(a.z, g.nz, bz1);
  AdjBrick b = adj_brick_geom(a, bz0 * nxy + bxy);
  int bz = bz0, now = 0, z = b.z0;
  LdsRegion ring[2], F[4];
  std::vector<LdsRegion> slab((size_t)a.slots);
  int in[4] = {-1, -1, -1, -1};     // control planes in the register sets
  int Q[4] = {-1, -1, -1, -1};      // and in Q
  int acc = b.cz0, full = 0;        // control plane of accumulator 0, accumulators that hold something
  int summed = 0, closed = 0;       // planes of brick bz in its partials, bricks in the loss
  bool ok = true;
  auto must = [&](bool c, const char* what) {
    if (ok && !c) {
      ck.fail(std::string("fused step, brick ") + std::to_string(bz) + ", plane " + std::to_string(z) + ": " + what);
      ok = false;
    }
  };
  auto slot_of = [&](int czl) { return (size_t)(Staged ? czl : czl & 1); };
  auto planes = [&](int z0, int np) {
    must(z0 == z && np >= 1 && z0 / g.dz == (z0 + np - 1) / g.dz && z0 % g.dz == 0, "planes of one z-tile");
    for (int n = 0; n < 4; ++n) must(Q[n] == z0 / g.dz + n, "Q of the tile's planes");
    if (z0 == b.z0) {
      must(full == 0, "empty accumulators at a brick's start");
      acc = b.cz0;
    }
    must(acc == z0 / g.dz, "accumulators of the tile's planes");
    full = 4;
    z = z0 + np;
  };
  const auto ring_ops = fused_ring(
      [&](int cz) {
        for (int k = 0; k < 4; ++k) in[k] = cz + k;
        must(cz >= 0 && cz + 3 < g.gz, "load inside the grid");
      },
      [&](int k, int cz) {
        must(in[k] == cz, "the loaded plane is stored");
        must(ring[cz & 1].store(cz, now), "ring slot stored while other waves may still read it");
      },
      [&](int cz) {
        in[0] = cz;
        must(cz >= 0 && cz < g.gz, "load inside the grid");
      },
      [&](int n, int cz) {
        must(ring[cz & 1].load(cz, now), "ring slot read before a barrier follows its store");
        Q[n] = cz;
      },
      [&] { ++now; });
  const auto march_ops = fused_march(
      [&] {
        for (int n = 0; n < 3; ++n) Q[n] = Q[n + 1];
      },
      planes, [&](int n, int k) { must(F[n].store(acc + k, now), "F stored while other waves may still read it"); },
      [&](int n, int czl, int np) {
        for (int k = 0; k < np; ++k) {
          must(F[k == 0 ? n : k + 1].load(b.cz0 + czl + k, now), "F read before a barrier follows its store");
          must(slab[slot_of(czl + k)].store(czl + k, now), "slab stored while other waves may still read it");
        }
      },
      [&](int n) {
        acc += n;
        full = imax(0, full - n);
      },
      [&](int czl, int np) {
        must(czl == summed, "planes summed in order");
        for (int k = 0; k < np; ++k)
          must(slab[slot_of(czl + k)].load(czl + k, now), "slab read before a barrier follows its store");
        summed += np;
        if (summed == adj_brick_cz(a, b)) summed = 0;  // the brick is complete
      },
      [&] {
        must(summed == 0 && z == b.ze, "the brick's loss after its last plane");
        ++closed;
      });
  fused_start(g, b.cz0, zend, ring_ops);
  fused_walk<Staged>(a, bxy, zend, b, bz, ring_ops, march_ops);
  must(z == zend && bz == bz1 - 1 && summed == 0 && full == 0 && closed == bz1 - bz0, "every plane and brick");
  return ok;
}

// The voxels of F that each cell of a brick contracts: in F, and of the cell's own columns.
template <int Cols>
bool check_fused_cells(const AdjGeom& a, const AdjBrick& b, Check& ck) {
  constexpr int kFRow = FusedShape<Cols>::f_row;
  REQUIRE(b.xe - b.x0 <= Cols && b.ye - b.y0 <= kFusedRows, "a lane per column of the brick");
  for (int w = 0; w < kAdjWaves; ++w) {
    const AdjCell c = adj_cell_geom(a, b, w);
    if (c.nx <= 0 || c.ny <= 0) continue;  // the wave contracts nothing
    for (int lane = 0; lane < kWave; ++lane)
      for (int s = 0; s < kAdjSteps<FusedShape<Cols>::narrow>; ++s) {
        const int e = fused_f_at<Cols>(b, c, lane, s), row = e / kFRow, x = b.x0 + e % kFRow / 3;
        REQUIRE(e >= 0 && row < kFusedRows && e % kFRow + 3 <= Cols * 3, "fused contraction outside F");
        REQUIRE(x >= c.x0 && x < c.x0 + c.nx, "fused contraction of another cell's column");
        REQUIRE(adj_lane_row<FusedShape<Cols>::narrow>(lane, s) < c.ny ? b.y0 + row == c.y0 + adj_lane_row<FusedShape<Cols>::narrow>(lane, s) : b.y0 + row >= b.ye,
                "fused contraction of another cell's row");
      }
  }
  return true;
}

// The staging of a brick's control planes: every float of the window by one thread, from
// inside the grid's plane to its place in the slot.
template <int L, int Threads>
bool check_fused_stage(const AdjGeom& a, const AdjBrick& b, const FusedLds& lds, Check& ck) {
  std::vector<int> hit((size_t)lds.slot, 0);
  for (int tid = 0; tid < Threads; ++tid) {
    const FusedStage<L> m = fused_stage_map<L, Threads>(a, b, tid);
    for (int k = 0; k < L; ++k) {
      if (m.src[k] < 0) continue;
      REQUIRE(m.src[k] < (int64_t)a.g.gx * a.g.gy * 3, "staging load outside the control plane");
      REQUIRE(m.dst[k] >= 0 && m.dst[k] < lds.slot, "staging store outside the slot");
      const int row = m.dst[k] / (a.x.cm * 3), i = m.dst[k] % (a.x.cm * 3);
      REQUIRE(m.src[k] == ((b.cy0 + row) * a.g.gx + b.cx0) * 3 + i, "staged float of the window");
      ++hit[(size_t)m.dst[k]];
    }
  }
  for (int y = 0; y < b.Cy; ++y)
    for (int i = 0; i < b.Cx * 3; ++i)
      REQUIRE(hit[(size_t)(y * a.x.cm * 3 + i)] == 1, "every float of the window is staged once");
  return true;
}

template <int Cols>
bool check_fused_lds(const AdjGeom& a, Check& ck) {
  using S = FusedShape<Cols>;
  const FusedLds lds = fused_lds<Cols>(a);
  REQUIRE(lds.total * (int64_t)sizeof(float) <= 160 * 1024 / S::per_cu, "LDS request of the workgroups of a CU");
  REQUIRE(lds.ring >= lds.F + (adj_staged(a) ? 4 : 2) * kFusedRows * S::f_row && lds.red >= lds.ring + 2 * lds.slot &&
              lds.slabs >= lds.red + S::threads && lds.slabs % 4 == 0 &&
              lds.total >= lds.slabs + adj_slab_at(a, a.slots - 1, kAdjWaves - 1) + adj_slab(a),
          "LDS regions apart");
  REQUIRE(fused_loads<Cols>(lds.slot) <= S::max_loads, "staged loads per thread");
  for (int i = 0; i < a.x.nb * a.y.nb; ++i) {
    const AdjBrick b = adj_brick_geom(a, i);
    if (!check_fused_cells<Cols>(a, b, ck)) return false;
    constexpr int kFew = S::max_loads / 2;
    if (!(fused_loads<Cols>(lds.slot) <= kFew ? check_fused_stage<kFew, S::threads>(a, b, lds, ck)
                                              : check_fused_stage<S::max_loads, S::threads>(a, b, lds, ck)))
      return false;
  }
  return true;
}

bool check_fused(const AdjGeom& a, Check& ck) {
  if (!(fused_cols(a) == 32 ? check_fused_lds<32>(a, ck) : check_fused_lds<64>(a, ck))) return false;
  const FusedSplit fs = fused_split(a);
  REQUIRE(fs.deep >= 1 && fs.nz * fs.deep >= a.z.nb && (fs.nz - 1) * fs.deep < a.z.nb, "workgroups cover the z-bricks");
  for (int i = 0; i < fs.nz; ++i) {  // a column's bricks have the same planes in every column
    const int bz0 = i * fs.deep, bz1 = imin(bz0 + fs.deep, a.z.nb);
    if (!(adj_staged(a) ? check_fused_walk<true>(a, 0, bz0, bz1, ck) : check_fused_walk<false>(a, 0, bz0, bz1, ck)))
      return false;
  }
  return true;
}

}  // namespace
}  // namespace bsi

using namespace bsi;

extern "C" {

// 0: every check passed; 1: a check failed (message in msg); -1: invalid geometry.
int bsi_check_indices(const int32_t dims[3], const int32_t spacing[3], char* msg, int msglen) {
  VolGeom g;
  if (make_geom(dims, spacing, &g)) {
    std::snprintf(msg, msglen, "invalid geometry");
    return -1;
  }
  Check ck;
  check_adjoints(g, ck) && check_forward(g, ck) && check_columns(g, ck);
  std::snprintf(msg, msglen, "%s", ck.msg.c_str());
  return ck.ok ? 0 : 1;
}

// 0: every check of the real-spacing adjoint passed; 1: one failed; -1: invalid geometry.
int bsi_check_general_indices(const int32_t dims[3], const float spacing[3], const float origin[3], char* msg,
                              int msglen) {
  GenGeom q;
  VolGeom g;
  if (make_gen_geom(dims, spacing, origin, &q, &g)) {
    std::snprintf(msg, msglen, "invalid geometry");
    return -1;
  }
  Check ck;
  check_general_adjoint(q, g, ck);
  std::snprintf(msg, msglen, "%s", ck.msg.c_str());
  return ck.ok ? 0 : 1;
}

// The batched kernels' item loops (batch_items): over several totals and
// grids, one workgroup per item and persistent, every item is taken exactly
// once and every workgroup's loop ends within ceil(total / grid) passes.
int bsi_check_batch_items(char* msg, int msglen) {
  Check ck;
  auto run_order = [&](int64_t total, int grid, bool persistent, bool runs) -> bool {
    std::vector<int> hit((size_t)total, 0);
    const int64_t max_pass = (total + grid - 1) / grid;
    for (int b = 0; b < grid; ++b) {
      int64_t passes = 0;
      for (ItemRange r = batch_items(b, grid, total, persistent, runs); r.first < total; r.first += r.step) {
        REQUIRE(r.first >= 0, "item below zero");
        REQUIRE(++passes <= max_pass, "a workgroup's item loop does not end");
        ++hit[(size_t)r.first];
      }
    }
    for (int h : hit) REQUIRE(h == 1, "an item taken other than once");
    return true;
  };
  auto run = [&](int64_t total, int grid, bool persistent) -> bool {
    return run_order(total, grid, persistent, false) && run_order(total, grid, persistent, true);
  };
  for (int64_t total : {1L, 2L, 7L, 8L, 9L, 100L, 1000L, 4097L, 20000L}) {
    if (!run(total, (int)total, false)) break;
    for (int grid : {1, 3, 8, 256, 512, 1024})
      if (grid <= total && !run(total, grid, true)) break;
    if (!ck.ok) break;
  }
  std::snprintf(msg, msglen, "%s", ck.msg.c_str());
  return ck.ok ? 0 : 1;
}

// 0: the fused SSD step's LDS accesses are in bounds and ordered by its barriers; 1: a violation
// (message in msg); -1: invalid geometry.  info: z-bricks per workgroup, and
// whether the slabs hold every plane of a brick.
int bsi_check_fused(const int32_t dims[3], const int32_t spacing[3], int32_t info[2], char* msg, int msglen) {
  VolGeom g;
  if (make_geom(dims, spacing, &g)) {
    std::snprintf(msg, msglen, "invalid geometry");
    return -1;
  }
  Check ck;
  const AdjGeom a = fused_geom(make_adj_geom(g));
  info[0] = fused_split(a).deep;
  info[1] = adj_staged(a);
  check_fused(a, ck);
  std::snprintf(msg, msglen, "%s", ck.msg.c_str());
  return ck.ok ? 0 : 1;
}

// How the fused SSD step splits a volume: brick columns, z-bricks, planes per z-brick,
// z-bricks per workgroup, workgroups along z, workgroups of a round.
int bsi_check_fused_split(const int32_t dims[3], const int32_t spacing[3], int32_t out[6]) {
  VolGeom g;
  if (make_geom(dims, spacing, &g)) return -1;
  const AdjGeom a = fused_geom(make_adj_geom(g));
  const FusedSplit f = fused_split(a);
  out[0] = a.x.nb * a.y.nb;
  out[1] = a.z.nb;
  out[2] = a.z.w;
  out[3] = f.deep;
  out[4] = f.nz;
  out[5] = kAdjCus * (fused_cols(a) == 32 ? FusedShape<32>::per_cu : 1);
  return 0;
}

// The largest thread counts of the forward launches of one volume, and of a batch that
// holds it alone (every shape and z split): aligned (spacing), scalar, real spacing
// (the same spacing, origin 0), batched.
int bsi_check_launch_threads(const int32_t dims[3], const int32_t spacing[3], int64_t out[4]) {
  VolGeom g, gg;
  GenGeom q;
  const float s[3] = {(float)spacing[0], (float)spacing[1], (float)spacing[2]}, o[3] = {0.f, 0.f, 0.f};
  if (make_geom(dims, spacing, &g) || make_gen_geom(dims, s, o, &q, &gg)) return -1;
  auto threads = [](const FwdLaunch& L, int64_t t) { return (int64_t)L.nbx * L.nby * L.nbz * t; };
  auto shape = [&](auto tile, int planes) {
    using T = decltype(tile);
    return threads(make_fwd_launch(g, kFwdTargetBlocks, T::width, T::rows, planes), T::threads);
  };
  out[0] = std::max(shape(FwdTileDefault{}, kFwdChunk), shape(FwdTile<2, 8, 1>{}, kFwdChunkWide));
  out[1] = std::max(shape(FwdTile<kFwdRows, 1, 4>{}, kFwdChunk), shape(FwdTileDefault{}, kFwdChunk));
  out[2] = 0;
  for (bool aligned : {false, true}) {
    const FwdLaunch f = make_gen_fwd_launch(gg, q, aligned);
    if (f.zchunk > kGenMaxZ || f.zchunk < 1 || (int64_t)f.nbz * f.zchunk < gg.nz) return 1;
    out[2] = std::max(out[2], threads(f, kFwdThreads));
  }
  out[3] = 0;
  for (const auto& [target, planes] : {std::pair{512L, 0}, {2048L, 0}, {(long)kFwdLeastItems, kFwdChunkBatch}})
    for (const auto& [width, rows] : {std::pair{64, 4}, {128, 2}, {64, 8}}) {
      const int64_t items = threads(make_fwd_launch(g, target, width, rows, planes), 1);
      const PassGrid p = pass_grid(items, 0, 256, width * rows);
      if (!p.persistent && p.blocks != items) return 1;
      out[3] = std::max(out[3], p.blocks * width * rows);
    }
  return 0;
}

}  // extern "C"
