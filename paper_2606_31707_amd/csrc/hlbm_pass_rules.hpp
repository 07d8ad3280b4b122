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

// What a pass computes: plain steps, window steps (with a small objective
// region, whose single steps launch a region pass each, or without), adjoint
// iterations.
enum PassKind { PASS_PLAIN, PASS_WINDOW, PASS_WINDOW_REGION, PASS_ADJOINT };

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
    case PASS_ADJOINT: break;
  }
  const int R = march3d_rows_of(f64);
  const double tiles = (double)m.tx * m.ty;
  const int64_t rounds = ((int64_t)(tiles * m.chunks) + 255) / 256;
  const double I = (double)rounds * (m.planes + 2.0);
  return n >= share * 256.0 * 62.0 * (R - 2) * (I - launch);
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
