// Host-side launch interface between the C ABI (hlbm_api.hip) and the
// per-precision kernel translation units.  Internal to the library.
#pragma once

#include <hip/hip_runtime.h>

namespace hlbm {

// Domain description in host precision; each translation unit converts it
// to its device argument struct.
struct HostDomain {
  long long plane;
  int nx, ny, pitch, bcx, bcy, flags;
  double mu, sigma, lambda, inv_cv, gm1, e2c, gamma, sgn_eps;
  double rho_ref, theta_ref, log_rho_ref, s_ref;
  double fref[9];
  double wall_u_lo, wall_u_hi, wall_theta;  // bcy == 2 (walls)
};

struct TileShape {
  int bw;        // tile width in columns (64, 128, 192 or 256); workgroup = bw + 64 lanes
  int rows;      // output rows per strip
  int xcd_remap; // 0 or 1
};

// Nominal tile shape of the single-domain step for an nx x ny grid; tile_w,
// tile_h > 0 are taken as given.  Automatic launches of up to a few rounds of
// workgroups run the shape of fit_tile instead, so the sizes below 2000^2 quoted
// here, measured on a sweep of six (FP64: two) workgroups per CU, only say what the
// queries report.
//  - 192-column tiles with 16-row strips measured fastest at 8192^2 in FP32
//    (row segments stay 256-byte aligned, the halo wave is a quarter of the
//    workgroup, 16-row strips beat taller ones).  FP64 (elem_size 8), which
//    held two workgroups per CU then, runs 2-5 % faster with 32-row strips
//    there.  Grids narrower than 1024 columns keep 128-column tiles with
//    32-row strips (less ragged); from 1024 columns on, 192 x 8 measured
//    best or tied in FP32 (1024^2 37.0-37.6 k MLUPS against 35.4-37.3 k for
//    128 x 8, 1500^2 43.6 k against 39.1 k).
//  - Small grids get 64-column tiles (nx <= 64) and strips halved down to 4
//    rows until about 768 workgroups exist in FP32 (half a round of six per
//    CU; at 1024^2 192 x 8, 768 workgroups, edges out 192 x 4) and 512 in
//    FP64, whose sweep holds two workgroups per CU, so 512 fill the chip
//    once (at 1024^2 128 x 16 runs 15.8 k MLUPS against 13.4 k for
//    128 x 8): a strip is swept serially, so a few tall strips would leave
//    the chip idle.
inline TileShape step_tile(int nx, int ny, int tile_w, int tile_h, int elem_size) {
  TileShape t;
  t.bw = tile_w ? tile_w : (nx <= 64 ? 64 : (nx >= 1024 ? 192 : 128));
  int rows = tile_h ? tile_h : (t.bw == 192 && elem_size == 4 ? 16 : 32);
  if (!tile_h) {
    const long long nbx = (nx + t.bw - 1) / t.bw;
    const long long want = elem_size == 8 ? 512 : 768;
    while (rows > 4 && nbx * ((ny + rows - 1) / rows) < want) rows /= 2;
  }
  if (rows > ny) rows = ny;
  t.rows = rows;
  t.xcd_remap = 1;
  return t;
}

// Nominal tile shape of the two-step sweep (periodic domains); as above, fit_tile
// replaces it on grids of a few rounds.  Its workgroup reads a
// radius-4 halo, rows + 8 rows for `rows` output rows, so it takes taller
// strips than the one-step sweep.  FP32 grids from 1024 columns on take
// 184-column tiles: tile plus halo fill three whole waves (192 columns leave
// a fourth wave with 8 of 64 lanes busy) and, with the s and theta rings cut
// to four rows, four workgroups fit a CU's LDS.  At 8192^2 (ms per step):
// 184 x 64 0.784, x 96 0.791, x 48 0.794, x 32 0.790 against 192 x 64 0.832
// (0.888 before the rings were cut); with plain stores and two rows of loads in
// flight 184 x 64 0.631, x 48 0.644, x 96 0.697.  Their strips are the tallest of 64,
// 32, 16 and 8 rows that give at least 768 workgroups and fill the last
// round of 1024 resident ones (four per CU on 256 CUs) at least three
// quarters: best or within 2 % of best at 1024^2 (8 rows), 1500^2 (16),
// 2048^2 (32), 3000^2 (64), 4096^2 (32), 6000^2 and 8192^2 (64), and
// 3-35 % faster than 192-column tiles from 1024^2 on, except level at
// 3000^2.  FP32 grids of 640 to 1023 columns take 120-column tiles (two
// whole waves, six workgroups per CU) with strips halved down to 8 rows
// until 768 workgroups exist: 8 rows at 768^2 and 1000^2, 29.3 and 41.3 k
// MLUPS against 25.0 and 30.9 k on 128-column tiles (at 512^2 the 128
// columns stay ahead, 13.8 against 13.1 k).  Narrower grids keep 128
// columns (halving the strips down to 8 rows until about 384 workgroups
// exist); FP64 keeps 128-column tiles, whose two levels of rings fit the
// LDS of one workgroup.
inline TileShape step2_tile(int nx, int ny, int tile_w, int tile_h, int elem_size) {
  TileShape t;
  const bool wide = nx >= 1024 && elem_size == 4;
  const bool mid = nx >= 640 && elem_size == 4;
  t.bw = tile_w ? tile_w : (nx <= 64 ? 64 : (wide ? 184 : (mid ? 120 : 128)));
  int rows = tile_h ? tile_h : 64;
  if (!tile_h) {
    const long long nbx = (nx + t.bw - 1) / t.bw;
    if (t.bw == 120) {
      while (rows > 8 && nbx * ((ny + rows - 1) / rows) < 768) rows /= 2;
    } else if (t.bw == 184) {
      constexpr long long kResident = 1024;
      for (; rows > 8; rows /= 2) {
        const long long nb = nbx * ((ny + rows - 1) / rows);
        const long long rounds = (nb + kResident - 1) / kResident;
        if (nb >= 768 && 4 * nb >= 3 * rounds * kResident) break;
      }
    } else {
      while (rows > 8 && nbx * ((ny + rows - 1) / rows) < 384) rows /= 2;
    }
  }
  if (rows > ny) rows = ny;
  t.rows = rows;
  t.xcd_remap = 1;
  return t;
}

// Modelled time of a row sweep over nb tiles of `rows` rows, `per_cu` workgroups
// of `waves` waves resident per compute unit: full rounds at the resident load
// plus the rest at its own, each (rows + fill of the pipeline) iterations of the
// time an iteration takes with that many waves per SIMD (measured on grids in the
// last-level cache, in units of 10 ns, by half waves per SIMD from one half up;
// below about two waves it hardly rises, the sweep then waits on its own
// latencies).
constexpr int kModelCUs = 256;
constexpr long long kLastLevelCache = 256LL << 20;  // bytes
inline long long sweep_cost(long long nb, int rows, int waves, int per_cu, int steps,
                            int elem_size, bool split = false) {
  static const int t_split[] = {110, 118, 126, 134, 152, 154, 177, 212};  // two-step, two groups
  static const int t_two[] = {145, 173, 178, 186, 232, 265};
  static const int t_one32[] = {115, 124, 140, 160, 182, 205, 225, 240, 260, 280, 305, 330};
  static const int t_one64[] = {185, 190, 257, 285, 330, 400};
  const int *time =
      split ? t_split : (steps == 2 ? t_two : (elem_size == 4 ? t_one32 : t_one64));
  const int last = split ? 7 : (steps == 1 && elem_size == 4 ? 11 : 5);
  const int fill = steps == 2 ? 8 : 4;
  const int resident = kModelCUs * per_cu;
  auto iter = [&](int wgs) {  // half waves per SIMD of the fullest CUs, as an index
    int per = (wgs + kModelCUs - 1) / kModelCUs;
    // two FP64 workgroups of two waves share a CU's first two SIMDs, and a row takes
    // as long as with three (2.33 us against 1.75 with one, 2.36 with three)
    if (waves == 2 && per == 2 && elem_size == 8) per = 3;
    int k = (per * waves + 1) / 2 - 1;
    // four groups' pairs a CU: not yet at its instruction rate while a tenth of the
    // slots are empty (two CUs of five then hold three)
    if (split && k == last && 10 * wgs <= 9 * resident) --k;
    return time[k > last ? last : k];
  };
  const long long rounds = nb < (1 << 30) ? (int)nb / resident : nb / resident;
  const int rest = (int)(nb - rounds * resident);
  return (rows + fill) * (rounds * iter(resident) + (rest ? iter(rest) : 0));
}

// Tile shape that an automatic launch takes (tile_w and tile_h both left to
// the library) in place of the nominal one above, on grids of a few rounds of
// resident workgroups.  There a strip height from a fixed list can leave the last
// round nearly empty: 1500 x 1100 in two-step strips of 184 x 8 is 1242
// workgroups, a second round of 218.  The shape is the one of least modelled time
// over all widths and heights.  us per step, nominal -> fitted: FP32 two-step
// 1500 x 1100 31.0 -> 20.9, 900^2 (one step before) 23.2 -> 13.9, 500^2 11.8 ->
// 9.2, 200^2 9.9 -> 5.9, 2048^2 55.2 -> 50.4; one-step 2048 x 512 26.8 -> 23.9;
// FP64 600^2 25.8 -> 23.7, 200^2 13.9 -> 11.4.
//
// The model has no term for memory, so two kinds of grids keep the nominal shape:
//  - one-step FP32 sweeps of a state larger than the last-level cache (one buffer
//    of ten planes), where 192 x 16 is best or level: us per step, nominal against
//    fitted, 3000^2 159 / 161, 3500^2 213 / 241, 4096^2 281 / 283; below that the
//    fit wins (2500^2 115 / 113, 6000 x 1000 109 / 107, 2048^2 82.5 / 80);
//  - grids of at least four full rounds of nominal tiles (8192^2: 64 rows 631 us
//    per step, 48 644, 96 697).  Nominal strips cut short to fill their last
//    round reach four rounds early: 2400^2 to 2500^2 stay on 184 x 8, which the model
//    puts at 1.7 to 1.8 times its best shape.
struct FitShape {
  int bw, waves, per_cu, max_nx;  // width, waves per workgroup, resident workgroups per CU
  bool split = false;             // two groups of waves (two-step sweep)
};
inline TileShape fit_tile(int nx, int ny, const TileShape &nominal, int elem_size, int steps) {
  static const FitShape two[] = {
      {64, 4, 4, 64, true}, {120, 4, 4, 1 << 30, true}, {184, 3, 4, 1 << 30}};
  static const FitShape one32[] = {
      {64, 2, 12, 1 << 30}, {128, 3, 8, 1 << 30}, {192, 4, 6, 1 << 30}, {256, 5, 4, 1 << 30}};
  static const FitShape one64[] = {{64, 2, 6, 1 << 30}, {128, 3, 4, 1 << 30}, {192, 4, 3, 1 << 30}};
  const FitShape *shapes = steps == 2 ? two : (elem_size == 4 ? one32 : one64);
  const int count = steps == 2 ? 3 : (elem_size == 4 ? 4 : 3);
  auto tiles = [&](int bw, int rows) {
    return (long long)((nx + bw - 1) / bw) * ((ny + rows - 1) / rows);
  };
  if (steps == 1 && elem_size == 4 && 40LL * nx * ny > kLastLevelCache) return nominal;
  for (int k = 0; k < count; ++k)
    if (shapes[k].bw == nominal.bw &&
        tiles(nominal.bw, nominal.rows) >= 4LL * kModelCUs * shapes[k].per_cu)
      return nominal;
  TileShape best = nominal;
  long long least = -1;
  for (int k = 0; k < count; ++k) {
    const FitShape &f = shapes[k];
    if (nx > f.max_nx) continue;
    for (int rows = ny < 2 ? ny : 2; rows <= ny && rows <= 128; rows += rows < 48 ? 1 : 4) {
      const long long cost =
          sweep_cost(tiles(f.bw, rows), rows, f.waves, f.per_cu, steps, elem_size, f.split);
      if (least < 0 || cost < least || (cost == least && f.bw > best.bw)) {
        least = cost;
        best.bw = f.bw;
        best.rows = rows;
      }
    }
  }
  return best;
}

// Domains of at most this many nodes, counting the ghosts at distance one on
// clamped axes, are stepped by one workgroup that holds them (k_resident): two
// nodes a thread fill its LDS in FP64.
constexpr int kResidentNodes = 1024;
inline int resident_nodes(long long nx, long long ny, int bcx, int bcy) {
  const long long n = (nx + (bcx ? 2 : 0)) * (ny + (bcy ? 2 : 0));
  return n > kResidentNodes ? kResidentNodes + 1 : (int)n;
}
// Steps of one such launch at most (about 10 ms).
constexpr int kResidentSteps = 4096;

// Elements from one state row to the next: nx rounded up to 64, so that every
// row, and with it every tile's row segment, starts 256-byte aligned (FP32).
// Rows of other widths lost 5 % (6000 and 14000 columns, rows 64-byte
// aligned) to 26 % (15446 columns, 24 bytes off a 64-byte boundary) of the
// step rate of their aligned neighbours.  The columns past nx are never read
// or written.
inline int row_pitch(int nx) { return (nx + 63) / 64 * 64; }

// Elements from one state plane to the next (elem_size 4 or 8): pitch x ny
// rounded up to 64.  A node's ten values sit at the same offset in every
// plane, and the step reads the same row segment from all ten at once.  With
// a plane size that is a multiple of a large power of two (8192^2 FP32: 256
// MiB) those ten segments land on the same HBM channels and banks.  Planes of
// 4 MiB or more therefore get a stride of a multiple of 128 KiB plus 64 KiB +
// 256 B (at most 0.2 MiB of padding per plane): 3 % faster at 8192^2 FP32
// than the bare 256 MiB stride, 1-2 % at 4096^2 and 6000^2.  Smaller planes
// keep a 64-element stride.
inline long long plane_stride(int nx, int ny, int elem_size) {
  const size_t es = (size_t)elem_size;
  const size_t elems = ((size_t)row_pitch(nx) * (size_t)ny + 63) / 64 * 64;
  if (elems * es < ((size_t)4 << 20)) return (long long)elems;
  const size_t unit = (size_t)128 << 10;
  const size_t bytes = (elems * es + unit - 1) / unit * unit + ((size_t)64 << 10) + 256;
  return (long long)(bytes / es);
}

// A pending learned correction for the tile kernels to apply as they load
// the state (x == nullptr: none): the moments and increments the
// correction kernels take, and the partial sums of correct_sums.
struct TileCorr {
  const float *x = nullptr, *dl = nullptr;
  const double *partials = nullptr;
  int conserve = 0;
};

#define HLBM_DECLARE_LAUNCHERS(NS)                                                          \
  namespace NS {                                                                            \
  hipError_t step(const HostDomain &d, const void *src, void *dst, unsigned *status,        \
                  const TileShape &tile, hipStream_t st);                                   \
  hipError_t step2(const HostDomain &d, const void *src, void *dst, unsigned *status,       \
                   const TileShape &tile, hipStream_t st);                                  \
  hipError_t resident(const HostDomain &d, const void *src, void *dst, unsigned *status,    \
                      int steps, hipStream_t st);                                          \
  hipError_t init(const HostDomain &d, const void *rho, const void *ux, const void *uy,     \
                  const void *s, void *dst, hipStream_t st);                                \
  hipError_t wall(const HostDomain &d, void *state, hipStream_t st);                        \
  hipError_t moments(const HostDomain &d, const void *state, void *rho, void *ux, void *uy, \
                     void *s, void *theta, hipStream_t st);                                 \
  hipError_t populations(const HostDomain &d, void *state, void *F9, const void *s,         \
                         int to_state, hipStream_t st);                                     \
  hipError_t reduce(const HostDomain &d, const void *state, double *partials, int nparts,   \
                    double *out, hipStream_t st);                                           \
  hipError_t entropy(const void *rho, const void *theta, void *s, long long n, double gamma, \
                     hipStream_t st);                                                       \
  size_t domain_args_bytes();                                                               \
  void pack_domains(const HostDomain *h, int count, void *host_out);                        \
  hipError_t step_batch(const void *doms, const long long *offs, const void *items,          \
                        int nitems, const void *src, void *dst, unsigned *status, int rows, \
                        int cw, int grid, hipStream_t st);                    \
  int batch_blocks_per_cu(int cw);                                                          \
  hipError_t step_batch2(const void *doms, const long long *offs, const void *items,         \
                         int nitems, const void *src, void *dst, unsigned *status, int rows,\
                         int cw, int grid, hipStream_t st);                   \
  int batch2_blocks_per_cu(int cw);                                                         \
  hipError_t step_tile_batch(const void *doms, const long long *offs, const void *items,     \
                             int nitems, const void *src, void *dst, unsigned *status,       \
                             int tw, int th, int grid, void *mom,              \
                             const long long *foffs,                                         \
                             long long mom_sc, const TileCorr &corr, hipStream_t st);        \
  int tile_blocks_per_cu(int tw, int th);                                                   \
  bool tile_shape_supported(int tw, int th);                                                \
  hipError_t step_tile_batch2(const void *doms, const long long *offs, const void *items,    \
                              int nitems, const void *src, void *dst, unsigned *status,      \
                              int tw, int th, int grid, void *mom,             \
                              const long long *foffs,                                        \
                              long long mom_sc, const TileCorr &corr, hipStream_t st);       \
  int tile2_blocks_per_cu(int tw, int th);                                                  \
  bool tile2_shape_supported(int tw, int th);                                               \
  hipError_t correct(const void *doms, const long long *offs, int count, long long n,       \
                     void *state, const float *x, const float *dl, double *partials,        \
                     int conserve, hipStream_t st);                                         \
  size_t correct_partials_bytes(int count);                                                 \
  hipError_t correct_sums(const void *doms, const long long *offs, int count, long long n,  \
                          const float *x, const float *dl, double *partials, hipStream_t st); \
  hipError_t correct_apply(const void *doms, const long long *offs, int count, long long n, \
                           void *state, const float *x, const float *dl,                   \
                           const double *partials, int conserve, hipStream_t st);          \
  hipError_t batch_moments(const void *doms, const long long *offs, const long long *foffs, \
                           int count, long long maxn, const void *state, void *rho, void *ux,  \
                           void *uy, void *s, void *theta, hipStream_t st);                  \
  }

HLBM_DECLARE_LAUNCHERS(f32)
HLBM_DECLARE_LAUNCHERS(f64)

constexpr int kReduceParts = 1024;  // workgroups of the first reduction pass
constexpr int kReduceVals = 6;

}  // namespace hlbm
