// Two time steps per sweep: the fused step applied twice inside one pass over
// the state, for domains periodic along both axes (included at the end of
// hlbm_device.hpp).
//
// The one-step sweep reads the ten planes once and writes them once per
// step, and on large FP32 grids that traffic bounds it (8192^2: 5.8 TB/s).  Here
// a workgroup reads the state at level n once and writes level n + 2 once:
// the per-node arithmetic of each step is the one-step kernel's, in the
// same order (FP64 results are bitwise those of two single steps), and level
// n + 1 lives only in registers and LDS rings.
//
// Geometry.  Output tile: CW columns from x0, `rows` rows from y0.  Level
// n + 2 there needs level n + 1 on a radius-2 halo (CW + 4 columns, rows + 4
// rows), which needs level n on a radius-4 halo: CW + 8 columns, rows + 8
// rows.  Lanes 0..CW-1 hold the tile's columns (aligned loads and stores),
// lanes CW..CW+7 the four halo columns on each side; the rest of the last
// wave repeats the first halo column.  A column's ring position is ri = column -
// (x0 - 4).  Virtual row j is grid row y0 - 4 + j.
//
// Stages per level (A: moments, B: collision, C: streaming and entropy, the
// functions of the one-step sweep), on the ring positions that have their
// stencils: A1 on 0..CW+7, B1 on 1..CW+6, C1 on 2..CW+5; C1's output (the
// nine populations and the entropy of level n + 1 at the lane's own node)
// feeds A2 in registers on the same lanes; B2 on 3..CW+4; C2 on the tile.
// Iteration i runs A1(i + 1), B1(i) and C2(i - 4), a barrier, issues the loads
// of row i + 3 and runs C1(i - 1) -> A2(i - 1) and B2(i - 2), and a second
// barrier: each half holds one stage of each kind, and each level keeps the
// one-step sweep's order between its own stages, so its rings have the same
// depths: 22 rows of CW + 8 per level, 34.3 KB at CW = 184, four workgroups
// of three whole waves per compute unit (155 registers, three waves per SIMD).
//
// Two rows of loads are in flight, in two register sets that alternate (the
// loop is unrolled by two): with one, a row's loads had half an iteration, about
// a microsecond, to arrive.  us per step with one -> two: 200^2 8.2 -> 7.1,
// 500^2 11.1 -> 9.7, 900^2 16.3 -> 15.1, 1500 x 1100 23.1 -> 21.7 (each on its
// best tile), 8192^2 647 -> 619.  The batch kernel keeps one row in flight: its
// per-domain arguments leave no room (168 registers with spills; 16 x 1024^2
// 1229 -> 1286 us for a data step).
//
// The stores are plain: a 184-column row's ends share cache lines with the
// neighbouring tiles', which run beside it on the same XCD, and the L2 joins
// the two halves; non-temporal stores wrote both partial lines to memory (8192^2
// 686 -> 634 us per step without them).
//
// Boundaries: out-of-range columns and rows wrap.  A halo lane then computes
// level n + 1 of the wrapped node from the wrapped stencil, bit for bit what
// the node's own lane computes, so periodic domains of any size (including
// ragged tiles and grids thinner than the halo) are exact.  Clamped
// boundaries need ghost copies of level n + 1 (along x the edge column's, which is
// in the ring, along y rows of their own), which this sweep does not form; they
// and walls take the one-step kernel.
#pragma once

namespace hlbm {
namespace HLBM_NS {

template <int CW>
struct TileRings2 {
  static constexpr int W = CW + 8;
  LevelRings<W> L1, L2;
};

// Lanes of a two-step tile: its CW columns and the 8 halo columns, rounded up to
// whole waves.  Single domains run tiles of 64 and 120 columns split (below): twice
// as many threads.
constexpr int step2_lanes(int cw) { return (cw + 8 + 63) / 64 * 64; }
constexpr bool step2_split(int cw) { return cw == 64 || cw == 120; }
constexpr int step2_threads(int cw) { return step2_lanes(cw) * (step2_split(cw) ? 2 : 1); }

template <int CW, bool kBatch = false>
__device__ __forceinline__ void sweep_tile2(const DomainArgs &d, const real *src0, real *dst0,
                                            unsigned *status, const int rows, const int bx,
                                            const int by, const unsigned frozen,
                                            TileRings2<CW> &R) {
  const int t = threadIdx.x;
  const real *src[kPlanes];
  real *dst[kPlanes];
#pragma unroll
  for (int q = 0; q < kPlanes; ++q) {
    src[q] = src0 + (long long)q * d.plane;
    dst[q] = dst0 + (long long)q * d.plane;
  }
  const int x0 = bx * CW, y0 = by * rows;
  // lane -> ring position: tile lanes at 4..CW+3, halo lanes at 0..3 and CW+4..CW+7
  const int h = t - CW;
  const int ri = t < CW ? t + 4 : (h < 4 ? h : (h < 8 ? CW + h : 0));
  const bool c1 = ri >= 2 && ri <= CW + 5;  // level n + 1 is valid on these lanes
  const int vx = x0 - 4 + ri;
  const bool c2 = t < CW && vx < d.nx;
  const int cx = map_index(vx, d.nx, d.bcx);
  const int nrow = min(rows, d.ny - y0);
  constexpr unsigned kEl = sizeof(real);
  Health health, health2;
  LevelRegs g1, g2;

  RowWalk walk(y0 - 4, d.ny, d.bcy);
  // rows in flight: an even and an odd one (batch: one)
  constexpr int kAhead = kBatch ? 1 : 2;
  real lda[kPlanes], ldb[kPlanes];
  auto load_row = [&](real (&to)[kPlanes]) {  // the next row
    const unsigned off = (unsigned)(walk.next(d.ny, d.bcy) * d.pitch + cx) * kEl;
#pragma unroll
    for (int q = 0; q < kPlanes; ++q) to[q] = load_at(src[q], off);
  };
  auto stage_a1 = [&](const int z, const real (&ld)[kPlanes]) {
    real F[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) F[q] = ld[q];
    level_a(d, g1, R.L1, z, ri, F, ld[9], health);
  };

  // Rows mod 3: m = i mod 3, mp = (i + 1) mod 3.
  int m = 0, mp = 1;
  auto out_row = [&](const int k, const int z) {  // C2(k)
    real Fo[kQ], snew;
    level_c(g2, R.L2, z, mp, ri, Fo, snew);
    if (c2) {
      const unsigned off = (unsigned)((y0 + k - 4) * d.pitch + vx) * kEl;
#pragma unroll
      for (int q = 0; q < kQ; ++q) store_at(dst[q], off, Fo[q]);
      store_at(dst[9], off, snew);
    }
  };
  // A1(i + 1), B1(i), (kOut) C2(i - 4), a barrier, the loads of row i + 1 + kAhead,
  // (kL2) C1(i - 1) -> A2(i - 1) and B2(i - 2), a barrier; z = i mod 2.
  auto row = [&](const int i, const int z, real (&in)[kPlanes], auto kL2, auto kOut) {
    stage_a1(1 - z, in);
    level_b(d, g1, R.L1, z, m, ri, d.sigma, d.sigma1);
    if constexpr (kOut.value) out_row(i - 4, z);
    __syncthreads();
    if (i + 1 + kAhead <= nrow + 7) load_row(in);
    if constexpr (kL2.value) {
      real Fo[kQ], snew;
      level_c(g1, R.L1, 1 - z, mp, ri, Fo, snew);
      level_a(d, g2, R.L2, 1 - z, ri, Fo, snew, health2);
      level_b(d, g2, R.L2, z, mp, ri, d.sigma, d.sigma1);
    }
    m = mp;
    mp = mp == 2 ? 0 : mp + 1;
    __syncthreads();
  };

  load_row(lda);
  if constexpr (kAhead == 2) load_row(ldb);
  stage_a1(0, lda);
  load_row(lda);
  if (barrier_skip<kBatch>(frozen)) return;
  using No = Flag<false>;
  using Yes = Flag<true>;
  const int last = nrow + 6;
  if constexpr (kBatch) {
    for (int i = 0; i < 3; ++i) row(i, i & 1, lda, No(), No());
    for (int i = 3; i < 8; ++i) row(i, i & 1, lda, Yes(), No());
    for (int i = 8; i <= last; ++i) row(i, i & 1, lda, Yes(), Yes());
  } else {
    row(0, 0, ldb, No(), No());
    row(1, 1, lda, No(), No());
    row(2, 0, ldb, No(), No());
    for (int i = 3; i < 7; i += 2) {
      row(i, 1, lda, Yes(), No());
      row(i + 1, 0, ldb, Yes(), No());
    }
    row(7, 1, lda, Yes(), No());
    for (int i = 8; i <= last;) {  // (a strip of one row has none)
      row(i, 0, ldb, Yes(), Yes());
      if (++i > last) break;
      row(i, 1, lda, Yes(), Yes());
      ++i;
    }
  }
  out_row(nrow + 3, (nrow + 1) & 1);
  if constexpr (kBatch) __syncthreads();  // the next item reuses the rings
  if (health.bad() || (c1 && health2.bad())) atomicOr(status, 1u);
}

// The same sweep by two groups of waves: the first runs level n (loads, A1, B1,
// C1), the second level n + 1 (A2, B2, C2, stores), half an iteration behind,
// with level n + 1's rows handed over through LDS.  A wave issues one instruction
// every four cycles at most, so on grids that leave one or two waves on a SIMD an
// iteration lasts as long as one wave's instructions for both levels; half of
// them a wave, on twice the waves, take 1.2 instead of 1.45 us (one workgroup
// of 120 columns per CU).  us per step, one group -> two: 200^2 7.1 -> 5.9, 500^2
// 9.7 -> 9.1, 900^2 15.1 -> 13.8, 1500 x 1100 22.4 -> 20.9 (one state, resident
// in the last-level cache); level at 2048^2 and 8192^2.  Wider tiles keep one group: the hand-over leaves 184 columns two
// workgroups per CU instead of four (8192^2 629 -> 764).
template <int CW>
struct SplitRings2 {
  static constexpr int W = CW + 8;
  LevelRings<W> L1, L2;
  real over[kPlanes][W];  // a row of level n + 1, from the first group to the second
};

template <int CW>
__device__ __forceinline__ void sweep_tile2_split(const DomainArgs &d, const real *src0,
                                                  real *dst0, unsigned *status, const int rows,
                                                  const int bx, const int by,
                                                  SplitRings2<CW> &R) {
  constexpr int kGroup = step2_lanes(CW);
  const bool second = __builtin_amdgcn_readfirstlane((int)threadIdx.x >= kGroup);
  const int t = (int)threadIdx.x - (second ? kGroup : 0);
  const int x0 = bx * CW, y0 = by * rows;
  // lane -> ring position: tile lanes at 4..CW+3, halo lanes at 0..3 and CW+4..CW+7
  const int h = t - CW;
  const int ri = t < CW ? t + 4 : (h < 4 ? h : (h < 8 ? CW + h : 0));
  const int vx = x0 - 4 + ri;
  const int nrow = min(rows, d.ny - y0), last = nrow + 7;
  constexpr unsigned kEl = sizeof(real);
  Health health;
  LevelRegs g;
  // rows mod 3: m = i mod 3, mp = (i + 1) mod 3
  int m = 0, mp = 1;
  auto end_row = [&]() {
    m = mp;
    mp = mp == 2 ? 0 : mp + 1;
    __syncthreads();
  };
  if (!second) {
    const real *src[kPlanes];
#pragma unroll
    for (int q = 0; q < kPlanes; ++q) src[q] = src0 + (long long)q * d.plane;
    const int cx = map_index(vx, d.nx, d.bcx);
    RowWalk walk(y0 - 4, d.ny, d.bcy);
    real lda[kPlanes], ldb[kPlanes];  // rows in flight: even and odd ones
    auto load_row = [&](real (&to)[kPlanes]) {  // the next row
      const unsigned off = (unsigned)(walk.next(d.ny, d.bcy) * d.pitch + cx) * kEl;
#pragma unroll
      for (int q = 0; q < kPlanes; ++q) to[q] = load_at(src[q], off);
    };
    auto stage_a = [&](const int z, const real (&ld)[kPlanes]) {
      real F[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) F[q] = ld[q];
      level_a(d, g, R.L1, z, ri, F, ld[9], health);
    };
    // A1(i + 1), B1(i), a barrier, the loads of row i + 3, (kC) C1(i - 1) into the
    // hand-over, a barrier
    auto row = [&](const int i, const int z, real (&in)[kPlanes], auto kC) {
      stage_a(1 - z, in);
      level_b(d, g, R.L1, z, m, ri, d.sigma, d.sigma1);
      __syncthreads();
      if (i + 3 <= nrow + 7) load_row(in);
      if constexpr (kC.value) {
        real Fo[kQ], snew;
        level_c(g, R.L1, 1 - z, mp, ri, Fo, snew);
#pragma unroll
        for (int q = 0; q < kQ; ++q) R.over[q][ri] = Fo[q];
        R.over[9][ri] = snew;
      }
      end_row();
    };
    load_row(lda);
    load_row(ldb);
    stage_a(0, lda);
    load_row(lda);
    row(0, 0, ldb, Flag<false>());
    row(1, 1, lda, Flag<false>());
    row(2, 0, ldb, Flag<false>());
    for (int i = 3; i < last;) {
      row(i, 1, lda, Flag<true>());
      if (++i == last) break;
      row(i, 0, ldb, Flag<true>());
      ++i;
    }
    __syncthreads();
    __syncthreads();
    if (health.bad()) atomicOr(status, 1u);
  } else {
    real *dst[kPlanes];
#pragma unroll
    for (int q = 0; q < kPlanes; ++q) dst[q] = dst0 + (long long)q * d.plane;
    const bool c2 = t < CW && vx < d.nx;
    // A2(i - 2) from the hand-over, B2(i - 3), a barrier, (kOut) C2(i - 4), a barrier
    auto row = [&](const int i, auto kOut) {
      const int z = i & 1;
      real F[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) F[q] = R.over[q][ri];
      level_a(d, g, R.L2, z, ri, F, R.over[9][ri], health);
      level_b(d, g, R.L2, 1 - z, m, ri, d.sigma, d.sigma1);
      __syncthreads();
      if constexpr (kOut.value) {
        real Fo[kQ], snew;
        level_c(g, R.L2, z, mp, ri, Fo, snew);
        if (c2) {
          const unsigned off = (unsigned)((y0 + i - 8) * d.pitch + vx) * kEl;
#pragma unroll
          for (int q = 0; q < kQ; ++q) store_at(dst[q], off, Fo[q]);
          store_at(dst[9], off, snew);
        }
      }
      end_row();
    };
    for (int i = 0; i < 4; ++i) {
      __syncthreads();
      end_row();
    }
    for (int i = 4; i < 8; ++i) row(i, Flag<false>());
    for (int i = 8; i <= last; ++i) row(i, Flag<true>());
    // level n + 1 is valid on the ring positions that have its stencil
    if (ri >= 2 && ri <= CW + 5 && health.bad()) atomicOr(status, 1u);
  }
}

// Two steps of a whole periodic domain: one workgroup per tile.
template <int CW>
__global__ __launch_bounds__(step2_threads(CW))
__attribute__((amdgpu_waves_per_eu(HLBM_IS_F32 ? (step2_split(CW) ? 4 : 3) : 1)))
void k_step2(StepArgs a) {
  int bid = blockIdx.x;
  const int nblk = a.nbx * a.nby;
  if (a.xcd_remap) {
    const int per = (nblk + 7) >> 3;
    const int xcd = bid & 7, k = bid >> 3;
    const int full = nblk - (per - 1) * 8;
    bid = xcd < full ? xcd * per + k : full * per + (xcd - full) * (per - 1) + k;
  }
  const int bx = bid % a.nbx, by = bid / a.nbx;
  if constexpr (step2_split(CW)) {
    __shared__ SplitRings2<CW> R;
    sweep_tile2_split<CW>(a.d, a.src, a.dst, a.status, a.rows, bx, by, R);
  } else {
    __shared__ TileRings2<CW> R;
    sweep_tile2<CW>(a.d, a.src, a.dst, a.status, a.rows, bx, by, 0, R);
  }
}

// Two steps of a batch of periodic domains: the persistent walk over (domain,
// tile) items of the one-step batch kernel, with the two-step sweep.
template <int CW>
__global__ __launch_bounds__(step2_lanes(CW))
__attribute__((amdgpu_waves_per_eu(HLBM_IS_F32 ? 3 : 1))) void k_step_batch2(BatchArgs a) {
  __shared__ TileRings2<CW> R;
  const TileWalk walk = tile_walk(a.nitems);
  for (int it = walk.first; it < walk.end; it += walk.step) {
    const int4 w = a.items[it];
    const int dm = __builtin_amdgcn_readfirstlane(w.x);
    const DomainArgs d = a.doms[dm];
    const long long off = a.offs[dm];
    // after the loads it must not wait for (memory counters drain in order)
    const unsigned frozen = domain_frozen(a.status + dm);
    sweep_tile2<CW, true>(d, a.src_buf + off, a.dst_buf + off, a.status + dm, a.rows,
                          __builtin_amdgcn_readfirstlane(w.y),
                          __builtin_amdgcn_readfirstlane(w.z), frozen, R);
  }
}

}  // namespace HLBM_NS
}  // namespace hlbm
