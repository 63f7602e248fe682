// The fused SSD step's use of LDS, shared by its kernel (fused.hip) and the host index
// checker: sizes, layout, and the order of a workgroup's stores, reads and barriers.
#pragma once

#include "adjoint_device.h"

namespace bsi {

// A workgroup's threads: a voxel column each, 16 rows of a brick.  Cols: the columns that a row
// of threads holds (fused_cols): 64, a wave per row, or 32 for narrow cells (spacings 1 and 2),
// 8 waves, and two workgroups per CU.  300 x 256 x 200 at spacing 1: 506 us, with a wave per
// row of 26 columns 1036; 300 x 300 x 200 at spacing 2 207, rows of 44 283 (48 threads a row 275).
constexpr int kFusedRows = kAdjCellsY * kAdjCellY;
template <int Cols>
struct FusedShape {
  static constexpr int threads = kFusedRows * Cols, waves = threads / kWave;
  static constexpr bool narrow = Cols <= 2 * kAdjTile;
  // Floats per row of F: the columns, padded so that the 2 rows (narrow: 4) a cell's lanes
  // read at once start 32 banks apart (48: the 16 lanes' floats).
  static constexpr int f_row = Cols * 3 + (Cols == 64 ? 32 : 16);
  static constexpr int max_loads = Cols == 64 ? 2 : 4;  // staged floats per thread
  static constexpr int per_cu = narrow ? 2 : 1;         // workgroups
};
static_assert(FusedShape<64>::f_row % 64 == 32 && FusedShape<32>::f_row % 64 == 48);
__host__ __device__ inline int fused_cols(const AdjGeom& a) { return a.g.nx >= 2 && adj_narrow(a) ? 32 : 64; }
// The adjoint's bricks, so its partials and bits; narrow ones always with two-plane slabs, which
// leave room for the second workgroup.
__host__ __device__ inline AdjGeom fused_geom(AdjGeom a) {
  if (fused_cols(a) == 32) a.slots = 2;
  return a;
}

// LDS (floats): F (two in turn, and with whole slabs two more for a brick's last
// three planes), the two-slot ring of staged control planes (the brick's window,
// pitch x.cm points), the reduction, the slabs.
struct FusedLds {
  int F, ring, slot, red, slabs, total;
};
template <int Cols>
__host__ __device__ inline FusedLds fused_lds(const AdjGeom& a) {
  using S = FusedShape<Cols>;
  FusedLds l;
  l.F = 0;
  l.ring = (adj_staged(a) ? 4 : 2) * kFusedRows * S::f_row;
  l.slot = a.y.cm * a.x.cm * 3;
  l.red = l.ring + 2 * l.slot;
  l.slabs = (l.red + S::threads + 3) / 4 * 4;  // 16-byte aligned
  l.total = l.slabs + a.slots * kAdjWaves * adj_slab(a);
  return l;
}
// Offset in F of this lane's voxel of its row s of a cell, its column clamped into the
// cell as the adjoint's loads are (adj_cell_offsets): an infinity in a neighbour's
// column must not decide how this cell is summed.  (Rows past the cell lie past the
// brick, and hold zeros.)
template <int Cols>
__host__ __device__ inline int fused_f_at(const AdjBrick& b, const AdjCell& c, int lane, int s) {
  using S = FusedShape<Cols>;
  return (c.y0 - b.y0 + adj_lane_row<S::narrow>(lane, s)) * S::f_row +
         (c.x0 - b.x0 + imin(adj_lane_col<S::narrow>(lane), c.nx - 1)) * 3;
}
// Staged floats per thread.  One plane's window is at most 1653 floats (29 x 19 points, at
// spacing 1), and at most 1024 from spacings 3 x 2 on.  One load more, which no
// window needs, cost the two-plane kernels 12 to 24 bytes of scratch per lane.
template <int Cols>
__host__ __device__ constexpr int fused_loads(int slot) {
  return (slot + FusedShape<Cols>::threads - 1) / FusedShape<Cols>::threads;
}
constexpr int kFusedMaxWindow = (kAdjCellsX * adj_cell(1) + 3) * (kFusedRows + 3) * 3;
static_assert(fused_loads<64>(kFusedMaxWindow) == FusedShape<64>::max_loads &&
              fused_loads<32>(kFusedMaxWindow) == FusedShape<32>::max_loads);

// Staging map: thread tid takes floats e = tid + k threads of the Cy x Cx x 3
// window of a control plane, into a slot with row pitch x.cm points.
template <int L>
struct FusedStage {
  int src[L];  // float offset within a control plane, -1 outside the window
  int dst[L];
};

template <int L, int Threads>
__host__ __device__ inline FusedStage<L> fused_stage_map(const AdjGeom& a, const AdjBrick& b, int tid) {
  FusedStage<L> m;
  const int wrow = b.Cx * 3;
#pragma unroll
  for (int k = 0; k < L; ++k) {
    const int e = tid + k * Threads;
    const int cyl = e / wrow, i = e - cyl * wrow;
    const bool in = cyl < b.Cy;
    m.src[k] = in ? ((b.cy0 + cyl) * a.g.gx + b.cx0) * 3 + i : -1;
    m.dst[k] = cyl * a.x.cm * 3 + i;
  }
  return m;
}

// A workgroup takes `deep` consecutive z-bricks of one (x, y) brick column: it
// marches on through their borders with the planes it has contracted, and
// only the adjoint's partials are cut there.  So the depth of a workgroup is
// chosen for this kernel, which runs one workgroup per CU (two of 32 columns): the CUs take the
// workgroups in rounds, and a round costs a workgroup's planes and its start and end, about
// kFusedRoundCost planes.  Of the depths with the fewest planes for each number of
// rounds, the cheapest is taken.  512 x 400 x 220, spacing 6 (200 brick columns of 5 bricks):
// 277 us as 200 workgroups in one round, 273 as 1000 in 4, 354 as 400 in 2; 152 x 343 x 409,
// spacing 3: 194 us as 462, 311 as 264, which are 2 rounds as well.  Measured with every depth
// of 17 sizes: costs of 8 to 10 choose the fastest or one within 2%.
constexpr int kFusedRoundCost = 9, kFusedRounds = 16;
struct FusedSplit {
  int deep, nz;  // z-bricks per workgroup, workgroups along z
};
__host__ __device__ inline FusedSplit fused_split(const AdjGeom& a) {
  const int64_t round = kAdjCus * (fused_cols(a) == 32 ? FusedShape<32>::per_cu : 1);
  const int64_t base = (int64_t)a.x.nb * a.y.nb, first = (base + round - 1) / round;
  FusedSplit f{a.z.nb, 1};
  int64_t best = -1;
  for (int64_t r = first; r < first + kFusedRounds; ++r) {
    const int64_t most = r * round / base;  // workgroups along z in r rounds, at least 1
    const int deep = (int)((a.z.nb + most - 1) / most), nz = (a.z.nb + deep - 1) / deep;
    const int64_t rounds = (base * nz + round - 1) / round;
    const int64_t cost = rounds * (imin(deep * a.z.w, a.g.nz) + kFusedRoundCost);
    if (best < 0 || cost < best) {
      best = cost;
      f = FusedSplit{deep, nz};
    }
  }
  return f;
}

// What a workgroup does, as the steps that fused_start and fused_walk put in order; every
// thread takes each of them.  Planes cz are the grid's, czl = cz - b.cz0 the brick's.
template <class Load4, class Fill, class Load, class Take, class Barrier>
struct FusedRing {
  Load4 load4;      // (cz): load control planes cz .. cz + 3 into four register sets
  Fill fill;        // (k, cz): set k, plane cz, to ring slot cz & 1
  Load load;        // (cz): load plane cz into set 0
  Take take;        // (n, cz): Q[n] from the slot of plane cz
  Barrier barrier;
};
template <class Shift, class Planes, class Put, class Cells, class Move, class Sum, class Close>
struct FusedMarch {
  Shift shift;      // Q[n] = Q[n + 1]
  Planes planes;    // (z, np): the voxel planes [z, z + np) of one z-tile, with Q
  Put put;          // (n, k): accumulator k to F[n]
  Cells cells;      // (n, czl, np): four waves each contract F[n], F[2], F[3] (np of them) into the slabs of planes czl .. czl + np - 1
  Move move;        // (n): the accumulators move down by n, zeros above
  Sum sum;          // (czl, np): slabs of planes czl .. czl + np - 1 into brick bz's partials
  Close close;      // after a brick's last plane: its loss joins the workgroup's
};
template <class... T>
__host__ __device__ __forceinline__ FusedRing<T...> fused_ring(T... t) {
  return FusedRing<T...>{t...};
}
template <class... T>
__host__ __device__ __forceinline__ FusedMarch<T...> fused_march(T... t) {
  return FusedMarch<T...>{t...};
}

// Q of the 4 control planes of the first z-tile, and the load of the next one.  Two
// accesses of one LDS region by different waves, one of them a store, lie on two sides
// of a barrier, here and in fused_walk:
// - ring slot cz & 1: filled with plane cz, read by take(cz), then filled with plane
//   cz + 2.  At a z-tile's border plane tz + 4 replaces tz + 2, which was taken
//   before the previous border's barrier, at the first border before the barrier
//   that ends the start (left out where no border follows); take(tz + 4) follows the
//   emission's barrier.
// - F[0], F[1] in turn: a store to F[turn] two planes on follows a barrier that the
//   contracting waves reach after their reads.  F[2], F[3]: once a brick.
// - slabs: with whole slabs a barrier on either side of the brick's sum (the next
//   plane's barrier is the later one); with two planes' slabs the barrier of plane
//   czl + 1 lies between the sum of czl and the store of czl + 2.
template <class Ring>
__host__ __device__ __forceinline__ void fused_start(const VolGeom& g, int tz, int zend, const Ring& op) {
  // the four loads together, through the two slots in pairs (one plane at a time waited
  // for memory four times)
  op.load4(tz);
  op.fill(0, tz);
  op.fill(1, tz + 1);
  op.barrier();
  op.take(0, tz);
  op.take(1, tz + 1);
  op.barrier();
  op.fill(2, tz + 2);
  op.fill(3, tz + 3);
  op.barrier();
  op.take(2, tz + 2);
  op.take(3, tz + 3);
  // the next tile's new plane tz + 4 (when another tile follows inside the
  // workgroup's range, it is at most ceil(nz/dz) + 2 = gz - 1)
  if ((tz + 1) * g.dz < zend) {
    op.barrier();  // the slot of plane tz + 2 is free for it
    op.load(tz + 4);
  }
}

// The z-bricks from b (number bz) on of brick column bxy, up to plane zend.
template <bool Staged, class Ring, class March>
__host__ __device__ __forceinline__ void fused_walk(const AdjGeom& a, int bxy, int zend, AdjBrick& b, int& bz,
                                                    const Ring& r, const March& op) {
  const VolGeom& g = a.g;
  int tz = b.cz0;  // z-bricks are whole tiles: b.z0 = tz * dz
  int turn = 0;  // which F the next plane goes to
  // The finished plane, accumulator 0: to F, and by the cells' waves into the slabs
  auto emit = [&](int czl) {
    op.put(turn, 0);
    r.barrier();
    op.cells(turn, czl, 1);
    if constexpr (!Staged) {
      r.barrier();
      op.sum(czl, 1);
    }
    turn ^= 1;
    op.move(1);
  };
  for (int z = b.z0; z < zend;) {  // one z-tile (the volume's last may be partial)
    const int np = imin(g.dz, zend - z);
    op.planes(z, np);
    z += np;
    const bool more = z < zend;
    if (more) r.fill(0, tz + 4);
    emit(tz - b.cz0);
    if (more) {
      op.shift();
      r.take(3, tz + 4);
    }
    if (z == b.ze) {  // the brick's last three control planes, then the next brick
      const int czl = tz - b.cz0 + 1;
      if constexpr (!Staged) {
#pragma unroll 1
        for (int n = 0; n < 3; ++n) emit(czl + n);
      } else {
        // together: F[turn] and the two that no other plane uses, a plane per four waves
        op.put(turn, 0);
        op.put(2, 1);
        op.put(3, 2);
        r.barrier();
        op.cells(turn, czl, 3);
        turn ^= 1;
        op.move(4);
        r.barrier();
        op.sum(0, adj_brick_cz(a, b));
      }
      op.close();
      if (more) b = adj_brick_geom(a, ++bz * (a.x.nb * a.y.nb) + bxy);
    }
    if (more) {
      ++tz;
      if ((tz + 1) * g.dz < zend) r.load(tz + 4);
    }
  }
}

}  // namespace bsi
