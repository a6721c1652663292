// Host-side helpers shared by the single-solve runtime and the serving pool:
// workspace layout, argument checks, kernel descriptors, launcher choice.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/vklb.h"
#include "vklb_launch.hpp"

namespace vklb {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }

inline int nvars(int kind, int dim) {
  switch (kind) {
    case VKLB_SHALLOW_WATER: return dim + 1;
    case VKLB_EULER: return dim + 2;
    case VKLB_MHD_GLM: return 9;
    case VKLB_LINEAR: return 1;
  }
  return 0;
}

struct Layout {
  size_t state_off, stage_off, fa_off, fb_off, part_off, diag_off, total;
  long long stride;
  int p, Q;
  int slots;  // stored slots of p planes per buffer: Q, or Q + 1 with the low part of U
  size_t elem;
};

// Stored basis (the kernels' BASIS) from vklb_options::basis: 0 all Q
// populations, 1 moving populations + U, 2 as 1 with U compensated (FP32).
// Default: FP64 populations; FP32 compensated in 1D (runs there take tens of
// thousands of steps and the launch, not HBM, bounds the step) and delta in 2D.
// -1: not a valid choice.
inline int resolve_basis(int opt, vklb_precision prec, int dim) {
  switch (opt) {
    case 0: return prec == VKLB_FP32 ? (dim == 1 ? 2 : 1) : 0;
    case 1: return 0;
    case 2: return 1;
    case 3: return prec == VKLB_FP32 ? 2 : -1;
  }
  return -1;
}

constexpr int kDiagBlocks = 512;
// Step grids of more workgroups than this fold each launch's partials into
// one entry (vklb_options.fold_partials = 0).
constexpr int kFoldAbove = 2048;

// Upper bound of the step grid over every strip width / band height choice.
inline long long max_step_blocks(const vklb_grid* g) {
  if (g->dim == 1) return (g->n[0] + 253) / 254;
  return ((g->n[0] + 63) / 64) * g->n[1];
}

// Cells from one row to the next in the population buffers: nx in 1D; in 2D
// nx rounded up to a multiple of 64, so that the 64 cells of a row a
// wavefront loads or stores start at a multiple of 64 whatever nx is, and
// each of its plane accesses is one aligned run of the blocked layout. The
// padding cells are never read or written by a step.
inline long long row_stride(const vklb_grid* g) {
  return g->dim == 2 ? (g->n[0] + 63) / 64 * 64 : g->n[0];
}

// basis: as resolve_basis returns it (sizes the population buffers).
inline bool layout_of(const vklb_system* sys, vklb_lattice lat, const vklb_grid* g, vklb_precision prec, int basis,
                      Layout* L) {
  if (!sys || !g) return false;
  if (g->dim != 1 && g->dim != 2) return false;
  if ((lat == VKLB_D1Q3) != (g->dim == 1)) return false;
  const int p = nvars(sys->kind, g->dim);
  if (p == 0) return false;
  const long long nx = g->n[0], ny = g->dim == 2 ? g->n[1] : 1;
  if (nx < 1 || ny < 1 || nx > (1ll << 30) || ny > (1ll << 30)) return false;
  const long long cells = nx * ny;
  if (cells > (1ll << 31) - 1) return false;
  // population buffers: padded rows in 2D (64-bit indices on the device; the
  // 2^31 limit is on natural cell indices, which non-physical reports carry)
  const long long pcells = row_stride(g) * ny;
  L->p = p;
  L->Q = g->dim == 1 ? 3 : 5;
  L->slots = L->Q + (basis == 2 ? 1 : 0);
  L->elem = prec == VKLB_FP32 ? 4 : 8;
  L->stride = (pcells + kBlock - 1) / kBlock * kBlock;  // whole storage blocks
  const size_t plane = size_t(L->stride) * L->elem;
  L->state_off = 0;
  L->stage_off = align_up(sizeof(DevState));
  L->fa_off = align_up(L->stage_off + size_t(p) * cells * 8);
  L->fb_off = align_up(L->fa_off + size_t(L->slots) * p * plane);
  L->part_off = align_up(L->fb_off + size_t(L->slots) * p * plane);
  L->diag_off = align_up(L->part_off + size_t(2) * 2 * max_step_blocks(g) * 8);
  L->total = align_up(L->diag_off + size_t(kDiagBlocks) * 9 * 2 * 8 + 256);
  return true;
}


// 2D: strip width; 1D: workgroup size (256 lanes measured faster than 512 at
// every 1D benchmark size: more, smaller workgroups start sooner).
inline int default_width(int dim, long long nx) {
  if (dim == 1) return 256;
  return nx <= 64 ? 64 : (nx <= 128 ? 128 : 256);
}
// Rows per 2D band of the kernels that store populations, for strips of
// `width` columns: the fewest (from 2 to 512) that let every workgroup be
// resident at once. A taller band leaves SIMDs idle, a shorter one starts a
// second round of workgroups that is nearly empty and re-reads more edge rows.
// Resident are two wavefronts per SIMD in FP32 and for FP64 shallow water and
// the linear system, one for FP64 Euler and MHD, by the march's registers.
// (The rule was the tallest power of two that gives 2048 wavefronts: 4 rows
// for Euler 1001^2, whose 8-row bands make 2016.) Measured on MI355X, us per
// step, that rule -> this one: FP32 Euler 1001^2 39.4 (4 rows) -> 31.3 (8), 700 x
// 1300 34.8 (4) -> 27.2 (8), 1024 x 768 25.0 (4) -> 22.9 (6), 300^2 11.7 (4) -> 9.4
// (2); FP32 MHD 1024 x 768 64.7 (4) -> 55.1 (6), 640 x 900 58.5 (4) -> 49.0 (6);
// FP64 Euler 640 x 900 57.8 (4) -> 42.6 (11), FP64 MHD 165 (4) -> 132 (11). Unchanged
// where the sides are powers of two: 2048^2 32 rows, 4096^2 128, 8192^2 512, and
// 8 for MHD 1024^2.
inline int default_band(int kind, vklb_precision prec, const vklb_grid* g, int width) {
  const long long strips = (g->n[0] + width - 1) / width, ny = g->dim == 2 ? g->n[1] : 1;
  const long long waves_per_group = (width + 63) / 64;
  const bool one = prec == VKLB_FP64 && (kind == VKLB_EULER || kind == VKLB_MHD_GLM);
  const long long resident = (one ? 1024 : 2048) / waves_per_group;  // workgroups
  long long band = (strips * ny + resident - 1) / resident;
  band = band < 2 ? 2 : (band > 512 ? 512 : band);
  while (band < 512 && strips * ((ny + band - 1) / band) > resident) ++band;
  return int(band);
}
// Largest band: the MHD march of the delta bases collides a band's halo cells
// into LDS for up to 64 rows; the others take any height.
constexpr int kMaxBand = 4096;
inline int max_band(int kind, int dim, int basis) {
  return kind == VKLB_MHD_GLM && dim == 2 && basis >= 1 ? 64 : kMaxBand;
}
// Rows of halo columns per batch (1..32): measured fastest on MI355X with the
// default bands, one batch per band (MHD 8 rows; the others 32, 3% over 2).
inline int default_halo(int kind) { return kind == VKLB_MHD_GLM ? 8 : 32; }

// Solves with omega = 1 keep U alone (vklb_omega1.hpp): the collision then
// returns the equilibrium of U, so the populations between two steps carry
// nothing that U does not. 1D FP64 shallow water keeps its populations, and
// its every bit: the dam break amplifies a rounding up to 10^8 times at its
// rarefaction head (reading of its growth in the oracle's tests), so any
// other rounding would show in its results.
inline bool keeps_u(int kind, int dim, vklb_precision prec, double omega) {
  return omega == 1.0 && !(kind == VKLB_SHALLOW_WATER && dim == 1 && prec == VKLB_FP64);
}

// Workgroups of a step of such a solve (2D: a wavefront per 64 columns and
// `band` rows), and its default band.
inline long long ustep_waves(const vklb_grid* g, int band) {
  return ((g->n[0] + 63) / 64) * ((g->n[1] + band - 1) / band);
}
// 1D: tiles of 256 cells (a fifth wavefront for the sides) where they need at
// most `most` workgroups per compute unit and tiles of 254 one more on a few
// units, which the others wait for. With more workgroups a unit the fifth
// wavefront costs more than the 0.8 % of tiles it saves: from two on for FP64
// MHD (its registers), three for FP32 MHD, eight for the others. us per step with tiles
// of 254 / 256 on MI355X: Euler FP32 65,536 cells 3.68 / 3.61, 131,072 4.56 / 4.38,
// 262,144 6.38 / 5.87, 524,288 10.8 / 11.2, 2^20 15.5 / 17.4, 2^24 194 / 236; FP64
// 65,536 4.18 / 3.94, 262,144 7.27 / 7.19, 2^20 18.5 / 22.3; shallow water FP32
// 262,144 5.57 / 5.20, 2^20 13.0 / 14.8; MHD FP32 65,536 6.34 / 6.28, 131,072 8.98 /
// 8.11, 196,608 10.6 / 10.7, 2^20 33.0 / 44.6; MHD FP64 65,536 8.62 / 8.01, 131,072
// 11.7 / 14.5, 2^20 49.7 / 105. Where both take the same rounds 254 is faster: Euler
// FP32 16,384 cells 3.26 / 3.49, 98,304 3.94 / 4.23.
constexpr long long kCUs = 256;
inline bool uside_of(int kind, vklb_precision prec, const vklb_grid* g) {
  if (g->dim != 1) return false;
  const long long a = (g->n[0] + utile1d(true) - 1) / utile1d(true), b = (g->n[0] + utile1d(false) - 1) / utile1d(false);
  const int most = kind != VKLB_MHD_GLM ? 4 : (prec == VKLB_FP32 ? 2 : 1);
  return a <= most * kCUs && (a + kCUs - 1) / kCUs < (b + kCUs - 1) / kCUs;
}
inline int ustep_grid_of(const vklb_grid* g, int band, bool side) {
  if (g->dim == 1) return int((g->n[0] + utile1d(side) - 1) / utile1d(side));
  return int((ustep_waves(g, band) + kUWaves - 1) / kUWaves);
}
// Rows per band of such a step: as few as let every wavefront be resident at
// once, so that a grid is one round of wavefronts whatever its sides are; a
// shorter band collides more edge rows (two half rows and the halo columns a
// band), a taller one leaves SIMDs short of wavefronts. Resident wavefronts
// per SIMD follow from the march's registers: four are enough in FP32 (SW,
// Euler; more would fit), two in FP64 and for MHD, one for FP64 MHD. At most
// 16 rows (MHD 32): large grids then take several rounds, whose wavefronts
// are out of step. Measured on MI355X (FP32, us per step by rows): Euler
// 2048^2 39.6 (8), 38.0 (16), 41.6 (32); 1024^2 17.0 (2), 13.3 (4), 13.4 (8);
// 512^2 8.4 (1), 7.0 (2), 7.6 (4); 4096^2 142 (16), 161 (32), 154 (64); 8192^2
// 507 (16), 541 (32), 557 (64); shallow water 500 x 333 6.3 (1), 6.2 (2), 6.2
// (3), 6.8 (4); MHD 1024^2 45.7 (4), 40.0 (8), 51.0 (16); 2048^2 136 (16), 132
// (32), 179 (64); 4096^2 508 (16), 518 (32), 510 (64); FP64 Euler 1024^2 28.0
// (4), 23.5 (8), 25.8 (16); FP64 MHD 512^2 41.5 (2), 33.2 (4), 50.1 (8). Grids of
// up to 1024 wavefront rows take one row each: Euler 200^2 5.2 (1), 5.7 (2), MHD
// 9.6 (1), 12.0 (2). Just above the resident count, and one row more: FP32
// Euler 1642 x 472, 4108 wavefronts of 4096, 13.1 (3), 11.3 (4); MHD 1199 x 1289,
// 2052 of 2048, 78.8 (12), 57.9 (13); FP64 Euler 1038 x 961 31.8 (8), 24.8 (9);
// FP64 MHD 342 x 1532 102 (9), 59.8 (10).
inline int default_uband(int kind, vklb_precision prec, const vklb_grid* g) {
  const bool mhd = kind == VKLB_MHD_GLM;
  const long long waves = 1024ll * (prec == VKLB_FP32 ? (mhd ? 2 : 4) : (mhd ? 1 : 2));
  const long long lines = (g->n[0] + 63) / 64 * g->n[1];
  if (lines <= 1024) return 1;  // a row each leaves no SIMD with two wavefronts
  const long long most = mhd ? 32 : 16;
  long long rows = (lines + waves - 1) / waves;
  rows = rows < 2 ? 2 : (rows > most ? most : rows);
  // a last band that is not full adds wavefronts: one row more where they
  // would start a second round that is nearly empty
  while (rows < most && ustep_waves(g, int(rows)) > waves) ++rows;
  return int(rows);
}

// Rows a wavefront of a U solve marches: the workgroup's four wavefronts share
// band_rows rows of strip_width columns (256 if not given), 64 columns each. So
// the tuner's 64-column strips of 4 to 64 rows are 1 to 16 rows a wavefront, the
// span default_uband takes its own from.
constexpr int kUStripWidth = 64 * kUWaves;
inline int uband_of(int band_rows, int strip_width) {
  const long long width = strip_width == 64 || strip_width == 128 ? strip_width : kUStripWidth;
  const long long rows = ((long long)band_rows * width + kUStripWidth - 1) / kUStripWidth;
  return int(std::min<long long>(rows, kMaxBand));
}

// Lanes of the one-workgroup kernel of a U solve of n cells: as asked
// (vklb_options.small_grid) where they hold the grid at up to four (256 lanes)
// or two cells each (MHD: one); else 256 or 512 lanes of one cell where they
// hold it so, 512 of two up to 1024 cells and 1024 of two above. Measured (us per
// step with 256 / 512 / 1024 lanes): FP32 Euler 300 cells 1.61 / 1.14 / 1.37, 700
// 2.22 / 1.54 / 1.64, 1000 2.75 / 1.87 / 2.11; FP64 Euler 1000 3.77 / 2.95 / 3.22;
// shallow water 1000 2.14 / 1.48 / 1.74.
inline int uwg_lanes(int kind, long long n, int asked) {
  const bool mhd = kind == VKLB_MHD_GLM;
  const int most = mhd ? 1 : (asked == 256 ? 4 : 2);
  if ((asked == 256 || asked == 512 || asked == 1024) && n <= (long long)asked * most) return asked;
  return n <= 256 ? 256 : (n <= (mhd ? 512 : 1024) ? 512 : 1024);
}

inline int step_grid_of(const vklb_grid* g, int width, int band) {
  if (g->dim == 1) return int((g->n[0] + width - 3) / (width - 2));
  return int(((g->n[0] + width - 1) / width) * ((g->n[1] + band - 1) / band));
}

// Tile shapes vklb_tune times for a solve with options `base`, its default
// shape among them. pool_2d: those of the serving pool's batched 2D kernels,
// in 128-column strips. There a U solve's wavefronts take four rows or more, also
// where the default is fewer: a sample is timed alone, which favours short
// bands, but in a full pool the wavefronts of other solves fill the chip and
// taller bands collide fewer edge rows. Solves/s of 400 mixed requests resident
// together, by rows of every U solve: 63 (1), 88 (2), 107 (4), 119 (8), 124 (16),
// 101 by the default rule, 103 by the fastest alone (1 to 5), 115 by these. (A pool
// of 12 requests is the other way round, ms: 11.2, 11.1, 11.8, 13.9, 18.8.)
inline std::vector<vklb_options> tune_candidates(int kind, vklb_precision prec, const vklb_grid* g, double omega,
                                                 const vklb_options& base, bool pool_2d) {
  std::vector<vklb_options> cand;
  const bool ust = keeps_u(kind, g->dim, prec, omega);
  vklb_options o = base;
  if (g->dim == 1) {
    // grids that run in one workgroup: its lane count (MHD has one shape)
    if (g->n[0] <= 1024 && kind != VKLB_MHD_GLM && base.small_grid >= 0) {
      for (int lanes : {256, 512, 1024}) {
        o.small_grid = lanes;
        cand.push_back(o);
      }
      return cand;
    }
    for (int w : {256, 512}) {
      if (ust && w > 256) continue;  // one shape
      o.strip_width = w;
      cand.push_back(o);
    }
    return cand;
  }
  const long long nx = g->n[0], ny = g->n[1];
  for (int w : {64, 128, 256}) {
    if (ust ? w != (pool_2d ? kUStripWidth : 64)
            : (pool_2d ? w != 128 : w > 64 && (nx + w - 1) / w * w - nx >= w / 2 && w != default_width(2, nx)))
      continue;  // (mostly idle lanes)
    const int rule = ust ? default_uband(kind, prec, g) * (kUStripWidth / w)
                         : std::min(default_band(kind, prec, g, w), max_band(kind, 2, resolve_basis(base.basis, prec, 2)));
    std::vector<int> bands = {4, 8, 16, 32, 64};
    if (std::find(bands.begin(), bands.end(), rule) == bands.end() && !(ust && pool_2d && rule < 4)) bands.push_back(rule);
    const int usual = ust ? 2 : default_halo(kind);  // (a U solve has one halo batch)
    for (int band : bands) {
      const int rows = ust ? uband_of(band, w) : band;
      if (band > 4 && band != rule && rows / 2 >= ny) continue;
      for (int halo : {2, 8, 16, 32}) {
        if (halo > band && !(band == rule && halo == usual)) continue;
        if (ust && halo != usual) continue;
        o.strip_width = w;
        o.band_rows = band;
        o.halo_rows = halo;
        cand.push_back(o);
      }
    }
  }
  return cand;
}

// Argument checks of vklb_create (Sec. 2.3 omega range, Sec. 3.2 CFL number,
// Sec. 3.4 dx == dy). Returns VKLB_OK or an error with a message.
inline vklb_status validate(const vklb_system* sys, vklb_lattice lat, const vklb_grid* grid, const vklb_speed* lambda,
                            double omega, const vklb_bc bc[2], const vklb_equilibrium* eq, vklb_precision prec,
                            const char** msg) {
  auto bad = [&](vklb_status st, const char* m) { *msg = m; return st; };
  if (!sys || !grid || !lambda || !bc || !eq) return bad(VKLB_ERR_ARG, "NULL argument");
  if (sys->kind < VKLB_SHALLOW_WATER || sys->kind > VKLB_LINEAR) return bad(VKLB_ERR_ARG, "unknown system");
  if (lat != VKLB_D1Q3 && lat != VKLB_D2Q5) return bad(VKLB_ERR_ARG, "unknown lattice");
  if (grid->dim != 1 && grid->dim != 2) return bad(VKLB_ERR_ARG, "grid dim must be 1 or 2");
  if ((lat == VKLB_D1Q3) != (grid->dim == 1)) return bad(VKLB_ERR_ARG, "lattice dimension does not match the grid");
  if (prec != VKLB_FP64 && prec != VKLB_FP32) return bad(VKLB_ERR_ARG, "unknown precision");
  if (!(omega > 0.0 && omega <= 2.0)) return bad(VKLB_ERR_ARG, "omega must be in (0, 2]");
  if (lambda->mode == VKLB_XI_CFL) {
    if (!(lambda->nu > 0.0 && lambda->nu <= 1.0)) return bad(VKLB_ERR_ARG, "nu must be in (0, 1]");
  } else if (lambda->mode == VKLB_XI_FIXED) {
    if (!(lambda->xi > 0.0) || !isfinite(lambda->xi)) return bad(VKLB_ERR_ARG, "xi must be > 0");
  } else {
    return bad(VKLB_ERR_ARG, "unknown speed mode");
  }
  if (eq->set < VKLB_EQ_WEIGHTED || eq->set > VKLB_EQ_DISCONTINUOUS) return bad(VKLB_ERR_ARG, "unknown equilibrium set");
  if (eq->set == VKLB_EQ_WEIGHTED) {
    if (!(eq->c >= 0.0) || !isfinite(eq->c)) return bad(VKLB_ERR_ARG, "c must be >= 0");
    if (!(eq->k >= 0.0)) return bad(VKLB_ERR_ARG, "k must be >= 0");
  }
  if (grid->n[0] < 1 || (grid->dim == 2 && grid->n[1] < 1)) return bad(VKLB_ERR_ARG, "empty grid");
  const double dx = (grid->hi[0] - grid->lo[0]) / double(grid->n[0]);
  if (!(dx > 0.0)) return bad(VKLB_ERR_ARG, "hi must exceed lo");
  if (grid->dim == 2) {
    const double dy = (grid->hi[1] - grid->lo[1]) / double(grid->n[1]);
    if (!(fabs(dx - dy) <= 1e-12 * dx)) return bad(VKLB_ERR_ARG, "the D2Q5 lattice needs dx == dy");
  }
  for (int a = 0; a < grid->dim; ++a) {
    if (bc[a] != VKLB_BC_PERIODIC && bc[a] != VKLB_BC_ZERO_GRADIENT && bc[a] != VKLB_BC_CHARACTERISTIC)
      return bad(VKLB_ERR_ARG, "unknown bc");
    if (bc[a] == VKLB_BC_CHARACTERISTIC && grid->dim != 1)
      return bad(VKLB_ERR_UNSUPPORTED, "characteristic boundaries: 1D only");
    if (bc[a] == VKLB_BC_CHARACTERISTIC && grid->n[0] < 2) return bad(VKLB_ERR_ARG, "characteristic boundaries need 2 cells");
  }
  if (sys->kind == VKLB_SHALLOW_WATER && !(sys->g > 0.0)) return bad(VKLB_ERR_ARG, "g must be > 0");
  if ((sys->kind == VKLB_EULER || sys->kind == VKLB_MHD_GLM) && !(sys->gamma > 1.0))
    return bad(VKLB_ERR_ARG, "gamma must be > 1");
  if (sys->kind == VKLB_MHD_GLM && !(sys->ch_factor > 0.0)) return bad(VKLB_ERR_ARG, "ch_factor must be > 0");
  Layout L;
  if (!layout_of(sys, lat, grid, prec, 0, &L)) return bad(VKLB_ERR_UNSUPPORTED, "grid too large or invalid");
  return VKLB_OK;
}

// After a step launch (or the initial reduction) that left the partials of
// parity `par`: fold them into entry 0 when the solve's launches read that
// entry alone (nred = 1).
inline hipError_t launch_fold(const SolveDesc& d, int par, hipStream_t s) {
  if (d.nred == d.nblocks) return hipSuccess;
  hipLaunchKernelGGL(k_fold_partials<1024>, dim3(1), dim3(1024), 0, s, d, par);
  return hipGetLastError();
}

// Checkpoint blobs hold the populations with their rows in grid order, so a
// blob does not depend on the band height of the solver that wrote it. Copy a
// population buffer between that order and the device's (mem_row; to_grid:
// device to grid order), in runs of 64 cells, which never cross a 256-cell
// block since rows are padded to a multiple of 64 cells.
inline void reorder_rows(const char* from, char* to, const SolveDesc& d, const Layout& L, bool down_odd, bool to_grid) {
  const size_t planes = size_t(L.slots) * L.p, run = size_t(64) * L.elem;
  auto off = [&](long long cell, size_t plane) {
    return ((size_t(cell) >> kBlockLog2) * planes + plane) * kBlock * L.elem + size_t(cell & (kBlock - 1)) * L.elem;
  };
  for (int r = 0; r < d.ny; ++r) {
    const long long m = mem_row(r, d.band, d.nfull, down_odd);
    for (long long x = 0; x < d.sx; x += 64) {
      const long long gc = (long long)r * d.sx + x, mc = m * d.sx + x;
      for (size_t pl = 0; pl < planes; ++pl)
        memcpy(to + off(to_grid ? gc : mc, pl), from + off(to_grid ? mc : gc, pl), run);
    }
  }
}

// Kernel descriptor of a solve whose workspace starts at `base`.
inline SolveDesc make_desc(char* base, const Layout& L, const vklb_system* sys, const vklb_grid* grid,
                           const vklb_speed* lambda, double omega, const vklb_bc bc[2], const vklb_equilibrium* eq,
                           int width, int band, int halo, bool batched = false) {
  SolveDesc d;
  memset(&d, 0, sizeof d);
  d.fa = base + L.fa_off;
  d.fb = base + L.fb_off;
  d.st = reinterpret_cast<DevState*>(base + L.state_off);
  d.stage = reinterpret_cast<const double*>(base + L.stage_off);
  d.part = reinterpret_cast<double*>(base + L.part_off);
  d.ph.g = sys->g;
  d.ph.gamma = sys->gamma;
  d.ph.ch_factor = sys->kind == VKLB_MHD_GLM ? sys->ch_factor : 0.0;
  d.ph.adv[0] = sys->adv[0];
  d.ph.adv[1] = sys->adv[1];
  d.ph.omega = omega;
  // the centered and discontinuous sets are weighted sets with fixed (c, k)
  double c = eq->c, k = eq->k;
  if (eq->set == VKLB_EQ_CENTERED) {
    c = grid->dim == 1 ? 1.0 / 3.0 : 1.0 / 5.0;
    k = 0.0;
  } else if (eq->set == VKLB_EQ_DISCONTINUOUS) {
    c = 0.0;
    k = INFINITY;
  }
  d.ph.c = c;
  d.ph.kinf = isinf(k) ? 1 : 0;
  d.ph.k = d.ph.kinf ? 0.0 : k;
  d.ph.alpha_local = eq->alpha_local ? 1 : 0;
  d.dx = (grid->hi[0] - grid->lo[0]) / double(grid->n[0]);
  // centered set: xi = sqrt(3/2 | 5/2) max|lambda| / eta (subcharacteristic rule)
  d.nu = eq->set == VKLB_EQ_CENTERED ? lambda->nu / sqrt(grid->dim == 1 ? 1.5 : 2.5) : lambda->nu;
  d.xi_fixed = lambda->xi;
  d.xi_mode = lambda->mode == VKLB_XI_CFL ? 0 : 1;
  d.nx = int(grid->n[0]);
  d.ny = grid->dim == 2 ? int(grid->n[1]) : 1;
  d.sx = int(row_stride(grid));
  d.stride = L.stride;
  d.bcx = bc[0] == VKLB_BC_PERIODIC ? 0 : (bc[0] == VKLB_BC_CHARACTERISTIC ? 2 : 1);
  d.bcy = (grid->dim == 2 ? bc[1] : bc[0]) == VKLB_BC_PERIODIC ? 0 : 1;
  d.band = band;
  d.nfull = grid->dim == 2 && band > 0 ? int(d.ny / band) : 0;
  d.halo = halo;
  d.nblocks = step_grid_of(grid, width, band);
  const vklb_precision prec = L.elem == 4 ? VKLB_FP32 : VKLB_FP64;
  if (keeps_u(sys->kind, grid->dim, prec, omega)) {
    // both U buffers in the first population buffer; the second one is the
    // room for a checkpoint's populations, whose rows are in grid order
    const size_t planes = size_t(L.slots > L.Q ? 2 : 1) * L.p;
    d.ustate = 1;
    d.us = (grid->n[0] + 63) / 64 * 64;
    d.pop = d.fb;
    d.fb = base + L.fa_off + planes * size_t(d.us) * d.ny * L.elem;
    d.nfull = 0;
    d.uside = !batched && uside_of(sys->kind, prec, grid);  // (a batched launch mixes the tiles of many solves)
    d.nblocks = ustep_grid_of(grid, band, d.uside);
  }
  d.nred = d.nblocks;
  return d;
}

inline Launchers pick_launchers(int kind, int dim, int prec, int basis, int width) {
  switch (kind) {
    case VKLB_SHALLOW_WATER: return launchers_sw(dim, prec, basis, width);
    case VKLB_EULER: return launchers_euler(dim, prec, basis, width);
    case VKLB_MHD_GLM: return launchers_mhd(dim, prec, basis, width);
    default: return launchers_linear(dim, prec, basis, width);
  }
}

// Fastest band and halo heights of the serving pool's batched 2D kernel for
// the solve of request r (vklb_tune over 128-column strips); defined with
// vklb_tune.
vklb_status tune_pool_shape(const vklb_request* r, vklb_precision prec, int steps, void* hip_stream, int* band,
                            int* halo, double* step_us);

inline int grid_for_cells(long long cells) {
  long long g = (cells + 255) / 256;
  return int(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

}  // namespace vklb
