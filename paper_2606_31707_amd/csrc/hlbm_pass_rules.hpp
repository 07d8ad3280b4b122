// hlbm_pass_rules.hpp -- how multi-step passes divide a lattice and which
// lattices take them (host only).
#pragma once

#include <cstdint>

#include "hlbm_host.hpp"

// 0: every lattice that can takes passes, of as many steps as there are kernels
// for (a build for the tests, which so reach them on small lattices).
#ifndef HLBM_PASS_RULES
#define HLBM_PASS_RULES 1
#endif

namespace hlbm {

// What a pass computes: plain steps, window steps (without an objective
// region; with a small one, whose single steps launch a region pass each; with
// a large one, whose terms the sweep adds), adjoint iterations (the objective's
// region small, large).
enum PassKind { PASS_PLAIN, PASS_WINDOW, PASS_WINDOW_REGION, PASS_ADJOINT, PASS_WINDOW_LARGE, PASS_ADJOINT_LARGE };

// Whether the populations and the porosity exceed the 256 MiB Infinity Cache.
inline bool beyond_caches(const hlbm_desc& d) {
  const int64_t plane = plane_stride((int64_t)d.nx * d.ny * d.nz, ssize_of(d.precision));
  return (int64_t)(ssize_of(d.precision) * q_of(d.stencil) + dsize_of(d.precision)) * plane > ((int64_t)256 << 20);
}

// ---- D2Q9: two or four steps -----------------------------------------------

// Strips and row chunks of a pass.
struct March2 {
  int strips, chunks, rows;  // strips along x, chunks along y, rows per chunk
};

// Rows per chunk: the number of iterations (rows plus the halo of the levels)
// times what an iteration costs with m workgroups on a compute unit.  Measured
// on 1100 x 410: a second wavefront on a SIMD adds 45 % to an iteration in
// FP64 and 9 % in FP32 (latency left by one is filled by the other), each
// further one 40 %.  Long chunks stop paying on lattices larger than the
// caches, where neighbouring chunks share their halo rows in L2
// (8192 x 4096 FP32: 8 rows 167 us, 16 rows 169, 58 rows 184; FP16S, whose
// rows are half as long, 150, 117 and 110).
inline March2 march2d_plan(const hlbm_desc& d, int K) {
  const int W = 64 - 2 * (K - 1), ny = d.ny;
  const bool f64 = d.precision == HLBM_FP64;
  March2 m;
  m.strips = (d.nx + W - 1) / W;
  const int most = d.precision == HLBM_FP16S ? 24 : 12;
  double best = 0.0;
  for (int rows = 1; rows <= most && rows <= ny; ++rows) {
    const int64_t groups = ((int64_t)m.strips * ((ny + rows - 1) / rows) + 3) / 4;
    const double per_cu = groups <= 1024 ? (double)((groups + 255) / 256) : groups / 256.0;
    const double share = f64 ? 0.55 + 0.47 * per_cu : (per_cu <= 2.0 ? 1.0 : 0.1 + 0.42 * per_cu);
    const double cost = (rows + 2 * (K - 1)) * share;
    if (rows == 1 || cost < best) {
      best = cost;
      m.rows = rows;
    }
  }
  m.chunks = (ny + m.rows - 1) / m.rows;
  return m;
}

// Steps (iterations) of a pass by the number of cells and the kernels.  Plain
// steps: four; two for FP16 lattices that stay in the caches, whose loads and
// conversions rather than bytes bound a pass (1100 x 410: 4.6 us a step with
// two, 5.0 with four; 8192 x 4096: 172 and 110).  Window steps: four; two in
// FP64, whose registers hold no more, and with a large region's terms in
// lattices that stay in the caches, where four levels spill more than they save (1024 x
// 512 with closure 15.7 us a step, two levels 13.0; 8192 x 4096 403 and 682).
// Adjoint: four on lattices with work for every SIMD, two on smaller ones, where
// the halo of four levels costs more than the launch it saves (400 x 160 FP32:
// 3.8 us an iteration with two, 4.5 with four; 1024 x 512 with the dissipation box
// 8.1 and 7.3, FP64 with the drag plane 12.5 and 11.6).
inline int pass_levels_2d(const hlbm_desc& d, PassKind kind) {
  switch (kind) {
    case PASS_PLAIN: return HLBM_PASS_RULES && d.precision == HLBM_FP16S && !beyond_caches(d) ? 2 : 4;
    case PASS_WINDOW:
    case PASS_WINDOW_REGION: return d.precision == HLBM_FP64 ? 2 : 4;
    case PASS_WINDOW_LARGE: return d.precision == HLBM_FP64 || (HLBM_PASS_RULES && !beyond_caches(d)) ? 2 : 4;
    default: return !HLBM_PASS_RULES || (int64_t)d.nx * d.ny >= 400000 ? 4 : 2;
  }
}

// Whether passes of that many steps beat single ones.  A pass takes the time of
// the rows that a wavefront goes through (its chunk and 2 (K - 1) more), times
// the workgroups of a compute unit; single steps that of the cells and, on
// small lattices, of their launches, worth `launch` rows: plain passes pay where
//   n >= share 256 4 W (rows' time - launch),   W = 64 - 2 (K - 1) own columns.
// Almost every 2D lattice lies above it; below it are narrow ones of thousands of
// rows (us a step, single / pass: 7 x 8990 FP64 with closure 6.2 / 8.8, 19 x 8747 FP32 with
// HRR and closure 5.9 / 8.1) and, for FP32 with HRR and closure, where the
// second workgroup of a compute unit is not for free, some of 50 to 400 thousand
// cells (289 x 835 5.7 / 6.5; 512 x 256 4.8 / 5.3; above it 400 x 160, 5.0 / 4.8).
// FP16S windows with closure and no region on channels whose wavefronts have two
// rows of their own for six of halo (4081 x 32 5.4 / 6.4, 904 x 135 5.4 / 5.6); FP64
// windows with a large region and closure, three rows a wavefront (512 x 256 7.6 /
// 9.0, 4081 x 32 8.0 / 8.7; two rows 904 x 135 8.8 / 7.3); in the adjoint of
// channels the strips of the outlet set the time of a pass of two: FP64 with three
// or more rows and one workgroup a compute unit (1700 x 148 7.2 / 8.0, 289 x 835 7.5 /
// 7.9; two rows 447 x 480 7.1 / 6.1), FP32 with a large region (556 x 584 7.4 / 8.0,
// 422 x 356 5.2 / 5.6; 904 x 135 5.6 / 4.8).  Of 5700 runs on other random lattices
// of 256 to 8 M cells 36 are more than 3 % slower than single steps, by 16 % at
// most; the mean is 0.71 of them.
inline bool passes_pay_2d(const hlbm_desc& d, PassKind kind, int K) {
  if (!HLBM_PASS_RULES) return true;
  const bool f64 = d.precision == HLBM_FP64, f32 = d.precision == HLBM_FP32;
  const bool les = d.smagorinsky_cs > 0.0, hrr = d.collision == HLBM_COLL_HRR, channel = d.bc_x == HLBM_BC_INLET_OUTLET;
  const March2 m = march2d_plan(d, K);
  const int64_t n = (int64_t)d.nx * d.ny, groups = ((int64_t)m.strips * m.chunks + 3) / 4;
  switch (kind) {
    case PASS_PLAIN: {
      if (!f64 && !les && !hrr) return true;
      const double per_cu = groups <= 1024 ? (double)((groups + 255) / 256) : groups / 256.0;
      const bool both = les && hrr;
      const double rows = (m.rows + 2.0 * (K - 1)) * (f32 && !both ? 0.25 + 0.75 * per_cu : per_cu);
      const double share = f32 ? 0.4 : (les || hrr ? 0.5 : 0.2), launch = f32 ? (both ? 7.0 : 12.0) : 9.0;
      return n >= share * 256.0 * 4.0 * (64 - 2 * (K - 1)) * (rows - launch);
    }
    case PASS_WINDOW: return !(d.precision == HLBM_FP16S && les && channel && m.rows == 2 && groups > 256);
    case PASS_WINDOW_LARGE: return !(f64 && les && channel && m.rows == 3 && groups <= 256);
    case PASS_ADJOINT: return !(f64 && channel && K == 2 && m.rows >= 3 && groups <= 256);
    case PASS_ADJOINT_LARGE:
      return !(channel && K == 2 && (f64 ? m.rows >= 3 && groups <= 256 : n >= 125000));
    default: return true;
  }
}

// Whether a packed list takes passes of two steps.  kind: PASS_PLAIN, PASS_WINDOW
// (a list with window members) or PASS_ADJOINT; with_other: the group's other
// list takes passes too, in the same launches; blocks: workgroups of its pass.
// Two lists in one launch for two steps instead of four launches pay at any size
// (us a step: FP64 4 x 26x13 ... 54x27 10.5 / 6.9, FP32 10.2 / 6.1; 14 x 636x318 ... 198
// / 140).  For one list a pass saves a launch of two and its longer chain costs
// more: on few workgroups, with FP64 window members (one body of 256 registers
// serves all members: 6 x 68x17 ... 5.9 / 9.4, 5 x 316x158 ... 24.6 / 28.5) and for FP32
// adjoints (4 x 113x56 ... 5.5 / 6.8, 9 x 301x1204 58 / 72), while FP64 adjoints gain
// from 400 workgroups on (276 blocks 7.8 / 8.7, 430 11.1 / 10.2), FP32 and FP16S
// windows from 150 (92 blocks 6.8 / 7.2, 173 9.6 / 7.7), plain lists from 200
// (74 blocks 4.6 / 4.8, 204 6.7 / 6.2).
inline bool packed_passes_pay(int precision, PassKind kind, bool with_other, int blocks) {
  if (!HLBM_PASS_RULES || with_other) return true;
  switch (kind) {
    case PASS_PLAIN: return blocks >= 200;
    case PASS_WINDOW: return precision != HLBM_FP64 && blocks >= 150;
    default: return precision == HLBM_FP64 && blocks >= 400;
  }
}

// ---- D3Q19: two steps ------------------------------------------------------

// Tiles and plane chunks of a pass.
struct March3 {
  int tx, ty, chunks, planes;  // tiles along x and y, chunks along z, planes per chunk
};

// Rows of a workgroup: three wavefronts a SIMD in FP32 (16 rows and four
// wavefronts, which share fewer recomputed rows but have 128 registers each:
// 870 instead of 845 us at 768x384x128, 227 instead of 203 at 756x168x84); two
// in FP64, whose state takes twice the registers.
constexpr int march3d_rows_of(bool f64) { return f64 ? 8 : 12; }

// A workgroup (one a compute unit) goes through the planes of its chunk and two
// beyond; the chunking with the fewest planes on the busiest compute unit, the
// start of a workgroup counted as another plane.  2048 chunks are enough for
// any number of planes: a tile's chunks fill the chip eight times over.
inline March3 march3d_plan(const hlbm_desc& d, int R) {
  March3 m;
  m.tx = (int)(((int64_t)d.nx + 61) / 62);
  m.ty = (int)(((int64_t)d.ny + R - 3) / (R - 2));
  const int64_t tiles = (int64_t)m.tx * m.ty;
  const int64_t nz = d.nz;
  double best = 0.0;
  for (int chunks = 1; chunks <= nz && chunks <= 2048; ++chunks) {
    const int64_t planes = (nz + chunks - 1) / chunks;
    const int64_t rounds = (tiles * ((nz + planes - 1) / planes) + 255) / 256;
    const double cost = (double)rounds * (planes + 3.0);
    if (chunks == 1 || cost < best) {
      best = cost;
      m.planes = (int)planes;
    }
  }
  m.chunks = (int)((nz + m.planes - 1) / m.planes);
  return m;
}

// Whether passes beat single steps.  A pass takes the time of the planes that
// the busiest compute unit goes through, I = rounds (planes + 2) of them, each
// 62 (R - 2) cells of its own; single steps that of the cells and, on small
// lattices, of their launches, worth `launch` planes.  So a pass pays where
//   n >= share 256 62 (R - 2) (I - launch),
// share being the part of the lanes' cells that have to be own, lattice cells:
// narrow or low tiles, half-empty rounds and the planes between chunks eat it.
// From 260 random lattices of 4 x 3 x 2 to 37 M cells, single / pass, us a
// step: above the line 757x215x14 FP64 216 / 169, 412x426x25 FP32 196 / 168,
// 16x16x16 FP64 6.6 / 5.7; below it 20x200x50 FP32 10.5 / 16.2 (tiles a third
// full), 63x375x145 FP32 141 / 172 (two tiles for 63 columns), 64x64x64 FP64
// with HRR and closure 14.9 / 20.5, 186x70x3 FP32 with closure 5.7 / 6.9.  The closure and the
// HRR collision lengthen a pass (issue-bound) and not a single step; walls
// lengthen a plane of a pass, an inlet a small single step.  FP64 window sums
// are bytes that a pass moves once, so that it pays earlier.  A FP64 population
// array of most of the Infinity Cache stays in it, two do not (77x106x176,
// 218 MB, 58.6 / 66.1).  The lattices above the line take 0.82 of the single
// steps' time in the mean; of other 150 random ones, the line drawn, one in
// 25 was more than 3 % and one in 400 more than 10 % slower than with single
// steps (25 % at most).
inline bool passes_pay_3d(const hlbm_desc& d, PassKind kind, const March3& m) {
  if (!HLBM_PASS_RULES) return true;
  const bool f64 = d.precision == HLBM_FP64;
  const double les = d.smagorinsky_cs > 0.0, hrr = d.collision == HLBM_COLL_HRR, inlet = d.bc_x == HLBM_BC_INLET_OUTLET,
               walls = d.bc_y != HLBM_BC_PERIODIC || d.bc_z != HLBM_BC_PERIODIC;
  const double n = (double)d.nx * d.ny * d.nz, bytes = 19.0 * (f64 ? 8.0 : 4.0) * n;
  double share = f64 ? 0.6 : 0.65, launch = 0.0;
  switch (kind) {
    case PASS_PLAIN:
      if (f64 && !inlet && bytes > (160.0 * (1 << 20)) && bytes < (256.0 * (1 << 20))) share = 0.85;
      launch = f64 ? 3.75 - 0.5 * les - 0.5 * hrr - 0.25 * les * hrr + 0.25 * inlet - 0.5 * walls
                   : 2.75 - 0.5 * les - 0.5 * hrr + 0.75 * inlet - 0.75 * walls;
      break;
    case PASS_WINDOW:
      if (f64) share = 0.5;
      launch = f64 ? 2.0 - 0.5 * walls : 3.0 - 0.25 * les + 0.5 * inlet - 0.75 * walls;
      break;
    case PASS_WINDOW_REGION:
      if (f64) share = 0.5;
      launch = f64 ? 3.5 - 0.25 * walls : 3.5;
      break;
    default: break;
  }
  const int R = march3d_rows_of(f64);
  const double tiles = (double)m.tx * m.ty;
  const int64_t rounds = ((int64_t)(tiles * m.chunks) + 255) / 256;
  const double I = (double)rounds * (m.planes + 2.0);
  return n >= share * 256.0 * 62.0 * (R - 2) * (I - launch);
}

// Steps that a pass of the lattice takes at most; 1: single steps.  m: its plan
// (D3Q19).  3D adjoint passes pay on every lattice that holds the second phi
// array (adjoint_passes_of).
inline int pass_limit(const hlbm_desc& d, PassKind kind, const March3& m) {
  if (d.stencil == HLBM_D2Q9) {
    const int K = pass_levels_2d(d, kind);
    return passes_pay_2d(d, kind, K) ? K : 1;
  }
  return kind == PASS_ADJOINT || kind == PASS_ADJOINT_LARGE || passes_pay_3d(d, kind, m) ? 2 : 1;
}

inline bool any_primal_pass_pays_3d(hlbm_desc d) {
  d.smagorinsky_cs = 0.0;
  const March3 m = march3d_plan(d, march3d_rows_of(d.precision == HLBM_FP64));
  return passes_pay_3d(d, PASS_PLAIN, m) || (d.collision == HLBM_COLL_BGK && (passes_pay_3d(d, PASS_WINDOW, m) ||
                                                                              passes_pay_3d(d, PASS_WINDOW_REGION, m)));
}

// ---- which lattices hold the arrays of passes ------------------------------

// Whether lattices of a descriptor take multi-step passes, and so hold a second
// population array (primal) and a second phi array (adjoint).  Single steps
// remain for a body force (tests), walls on the x axis (a value that bounces
// there stays on its row, which a strip does not provide for), one-row
// channels (their row is beside both walls), and rows whose byte offsets
// exceed 32 bits; in 3D fewer than two planes, and FP16S, whose conversions cost
// what the saved bytes give (192x96x64 21.5 us a step, 32.5 with passes;
// 756x168x84 with walls 158 and 198; 768x384x128 565 and 478); for the adjoint
// also the HRR collision (its frozen data would have to wait for the later
// levels as well).  J_MEA takes single steps too, but holds the second phi
// array: a window can be given another objective.  The 3D adjoint passes are
// bound by their instructions and pay only in FP64 beyond the caches (us an
// iteration, single / pass: FP64 756x168x84 798 / 533, 300x128x64 175 / 137,
// 240x110x66 (279 MB) 109 / 100, 192x96x64 (189 MB) 57 / 73; FP32 768x384x128
// 1195 / 1439, 192x96x64 34 / 44).  And in 3D single steps remain where no pass
// pays (passes_pay_3d; the closure can be switched off later, which makes a
// pass pay earlier).
inline bool primal_passes_of(const hlbm_desc* d) {
  if (d->stencil == HLBM_D3Q19 && (d->nz < 2 || d->precision == HLBM_FP16S || !any_primal_pass_pays_3d(*d))) return false;
  return d->bc_x != HLBM_BC_WALLS && d->ny >= 2 &&
         (3 * (int64_t)d->nx + 256) * 8 < ((int64_t)1 << 32) && d->force[0] == 0.0 && d->force[1] == 0.0 &&
         d->force[2] == 0.0;
}
inline bool adjoint_passes_of(const hlbm_desc* d) {
  if (d->stencil == HLBM_D3Q19 &&
      (d->nz < 2 || d->precision != HLBM_FP64 ||
       (HLBM_PASS_RULES && (int64_t)d->nx * d->ny * d->nz * 160 <= ((int64_t)256 << 20)) ||
       !passes_pay_3d(*d, PASS_ADJOINT, march3d_plan(*d, march3d_rows_of(true)))))
    return false;
  return d->bc_x != HLBM_BC_WALLS && d->ny >= 2 &&
         (3 * (int64_t)d->nx + 256) * 8 < ((int64_t)1 << 32) && d->collision == HLBM_COLL_BGK;
}

// Device bytes of the arrays that only the multi-step passes use, which a
// lattice does without where they do not fit: the second population array
// and, in FP64, a window step's region records; the second phi array.
inline uint64_t pass_bytes_primal(const hlbm_desc* d) {
  if (!primal_passes_of(d)) return 0;
  const uint64_t q = q_of(d->stencil), as = asize_of(d->precision);
  uint64_t b = (uint64_t)plane_stride((int64_t)d->nx * d->ny * d->nz, ssize_of(d->precision)) * q * ssize_of(d->precision);
  if (d->precision == HLBM_FP64)
    b += (uint64_t)round_up((int64_t)d->ny * d->nz, 128) * (uint64_t)region_copy_stride((int)q, (int)as) * as;
  return b;
}
inline uint64_t pass_bytes_adjoint(const hlbm_desc* d) {
  if (!adjoint_passes_of(d)) return 0;
  return (uint64_t)plane_stride((int64_t)d->nx * d->ny * d->nz, ssize_of(d->precision)) * asize_of(d->precision) *
         (uint64_t)q_of(d->stencil);
}

// Whether `bytes` of such arrays may be taken: half of the device stays free
// for what is needed, by this library or by others, which cannot ask for them
// back.
inline bool optional_fits(uint64_t avail, uint64_t total, uint64_t bytes) {
  return avail >= bytes && avail - bytes >= total / 2;
}

}  // namespace hlbm
