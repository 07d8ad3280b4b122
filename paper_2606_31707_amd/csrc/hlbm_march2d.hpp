// hlbm_march2d.hpp -- D2Q9 sweeps that take K steps in one pass over memory.
//
// A wavefront owns a strip of 64 columns and marches down its rows; the K
// time levels follow one another one row apart (level t works on row r - t
// when level 0 works on row r), so a row is loaded once, goes through all K
// levels in registers and is stored once.  Between the levels a population
// moves along x by a lane shift (DPP) and along y by staying in registers for
// up to two rows: per level boundary the nine values that a row still waits
// for.  No LDS and no barrier: wavefronts are independent.
//
// Input and output are the canonical layout (parity 0) in two arrays, read
// from one and written to the other: the last level pushes its post-collision
// values to the neighbours' slots, each slot having one writer.  Level t is
// valid on lanes [t, 63 - t], so 64 - 2 (K - 1) columns of a strip and the
// rows of its chunk are its own and the rest is recomputed by the neighbours.
// Every cell runs the per-cell code of the single-step sweeps, stored values
// are rounded to the storage type between the levels: the results are
// bitwise those of K single steps.
//
// What bounds it: a single step moves every population through memory once
// (the sweeps of hlbm_kernels.hpp run at what an in-place copy reaches); a
// pass of four moves them once for four steps, 2.9 times fewer bytes with the
// halo, and then the vector units and the latency of a row's chain of levels
// share the time (77 vector instructions a level in FP32, 84 in FP64).
// Microseconds a step, single step -> pass: 8192 x 4096 FP32 448 -> 167,
// FP64 912 -> 285, FP16S 228 -> 110; 1100 x 410 FP64 10.0 -> 6.1, FP32
// 6.5 -> 4.3; 220 x 41 FP64 4.0 -> 2.9, where launches and one wavefront's
// chain are all there is.
#pragma once

#include <type_traits>

#include "hlbm_kernels.hpp"

namespace hlbm {

hipError_t launch_window2d(hlbm_lattice_s* L, int K);  // K D2Q9 window steps (hlbm_window2d.hip)
hipError_t launch_march3d_adjoint(hlbm_lattice_s* L);  // two D3Q19 adjoint iterations
hipError_t launch_march3d(hlbm_lattice_s* L, bool window);  // two D3Q19 steps (hlbm_march3d.hip)

// Values of the lane one to the left (cx = +1 moves them right) / right.
// DPP wave_shr:1 / wave_shl:1; the end lanes get 0, which nobody uses.
__device__ __forceinline__ uint32_t lane_shift32(uint32_t v, int cx) {
  return cx > 0 ? (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xf, 0xf, true)
                : (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xf, 0xf, true);
}
template <typename T>
__device__ __forceinline__ T lane_shift(T v, int cx) {
  if (cx == 0) return v;
  if constexpr (sizeof(T) == 8) {
    union {
      T t;
      uint32_t w[2];
    } u;
    u.t = v;
    u.w[0] = lane_shift32(u.w[0], cx);
    u.w[1] = lane_shift32(u.w[1], cx);
    return u.t;
  } else {
    union {
      T t;
      uint32_t w;
    } u;
    u.t = v;
    u.w = lane_shift32(u.w, cx);
    return u.t;
  }
}

// Where a wavefront's lanes lie: x of the lane, the columns its neighbours
// have (periodic wrap), and what ends of the lattice the strip touches.
struct Strip {
  int gx;                  // column (may lie outside the lattice)
  int xm, x, xp;           // columns of the lane and of its neighbours, wrapped or clamped into [0, nx)
  bool own;                // the lane's column is the strip's own
  bool inlet, outlet;      // lane on the inlet / outlet column
  bool ends, any_outlet;   // the strip holds an inlet or outlet lane, an outlet lane (uniform)
};

template <int K>
__device__ __forceinline__ Strip make_strip(const Geo& g, int strip) {
  constexpr int W = 64 - 2 * (K - 1);
  Strip s;
  const int lane = threadIdx.x & 63;
  s.gx = strip * W - (K - 1) + lane;
  const bool per = g.bcx == BC_PERIODIC;
  auto col = [&](int x) {
    if (per) {
      x %= g.nx;
      return x < 0 ? x + g.nx : x;
    }
    return x < 0 ? 0 : (x >= g.nx ? g.nx - 1 : x);
  };
  s.x = col(s.gx);
  s.xm = col(s.gx - 1);
  s.xp = col(s.gx + 1);
  s.own = lane >= K - 1 && lane <= 64 - K && s.gx < g.nx;
  s.inlet = g.bcx == BC_INOUT && s.gx == 0;
  s.outlet = g.bcx == BC_INOUT && s.gx == g.nx - 1;
  s.ends = __ballot(s.inlet || s.outlet) != 0;
  s.any_outlet = __ballot(s.outlet) != 0;
  return s;
}

// The i-th direction with cy = CY in D2Q9 order.
template <int CY>
__device__ constexpr int dir9(int i) {
  int n = 0;
  for (int k = 0; k < 9; ++k)
    if (Lat<9>::cy[k] == CY && n++ == i) return k;
  return -1;
}

// What a level boundary holds between rows: the values moving up (cy = +1)
// from the last two rows (up[r & 1] of row r) and those staying on the last row.
template <typename T>
struct Wait {
  T up[2][3], mid[3];
};

// Hands the post-collision values c of a row to the next level: fills in what
// the row before it was still waiting for (s: all nine of that row) and keeps
// the rest.  ph: parity of the row within the loop.  EDGE 1, 2: o holds what the
// outlet lane gets from the virtual column (cx = -1 directions, in order);
// EDGE 2, beside a wall (at_wall: -1 the row is the first, +1 the last, +2 the one beyond
// the last) the values that would cross it bounce back on their row: those
// going down from the first row are its upward arrivals, those going up from
// the last row wait in the place of its upward values for the row beyond.
template <int EDGE, typename T>
__device__ __forceinline__ void hand_on(const int ph, const Strip& st, const int at_wall, const T (&c)[9],
                                        const T (&o)[3], Wait<T>& w, T (&s)[9]) {
  using L = Lat<9>;
  T sh[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) sh[k] = lane_shift(c[k], L::cx[k]);
  if (EDGE) {
    int n = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k)
      if (L::cx[k] == -1) sh[k] = st.outlet ? o[n++] : sh[k];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s[dir9<1>(i)] = w.up[ph][i];  // from two rows before
    s[dir9<0>(i)] = w.mid[i];
    s[dir9<-1>(i)] = sh[dir9<-1>(i)];
    w.up[ph][i] = sh[dir9<1>(i)];
    w.mid[i] = sh[dir9<0>(i)];
  }
  if (EDGE == 2 && __builtin_expect(at_wall != 0, 0)) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (at_wall == -1) w.up[ph ^ 1][i] = c[L::opp[dir9<1>(i)]];
      if (at_wall == 1) w.up[ph][i] = c[dir9<1>(i)];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (dir9<1>(j) == L::opp[dir9<-1>(i)] && at_wall == 2) s[dir9<-1>(i)] = w.up[ph ^ 1][j];
    }
  }
}

__device__ __forceinline__ int wrap_row(int y, int ny) {
  y %= ny;
  return y < 0 ? y + ny : y;
}

__device__ __forceinline__ uint64_t uni64(uint64_t v) { return (uint64_t)wave_uniform64((int64_t)v); }

// The row a wavefront loads: scalar base address of plane 0 (stepped plane to
// plane at the accesses), wrapped on a periodic y axis.
struct RowPtr {
  uint64_t base, row_bytes, lat_bytes;
  int y, ny;
  __device__ __forceinline__ RowPtr(const void* A, int row, int nx, int ny_, int size) {
    ny = ny_;
    y = row;
    while (y < 0) y += ny;
    while (y >= ny) y -= ny;
    row_bytes = (uint64_t)nx * (uint64_t)size;
    lat_bytes = row_bytes * (uint64_t)ny;
    base = uni64((uint64_t)A + row_bytes * (uint64_t)y);
  }
  __device__ __forceinline__ void next() {
    base += row_bytes;
    if (++y == ny) {
      y = 0;
      base -= lat_bytes;
    }
  }
};
template <typename S>
__device__ __forceinline__ typename Glob<S>::type* lane_ptr(uint64_t base, uint32_t off) {
  typedef typename Glob<char>::type gchar;
  return (typename Glob<S>::type*)((gchar*)base + off);
}

// Stores the last level's post-collision values c of row y to the slots they
// move to (B).  VIRT, o: the virtual column's values on the outlet lane.  Rows away
// from walls and periodic seams share one scalar base per plane (below: row
// y - 1 of plane 0); v: byte offsets of the three neighbour columns.
template <int EDGE, bool VIRT, typename S, typename T>
__device__ __forceinline__ void push_row(const Geo& g, const Strip& st, bool walls, const int y,
                                         uint64_t below, const uint32_t (&v)[3], uint64_t pstep, uint32_t rowb,
                                         const T (&c)[9], const T (&o)[3]) {
  using L = Lat<9>;
  uint64_t base[9];  // row y - 1 of each plane (formed ahead of the masked stores)
  base[0] = below;
#pragma unroll
  for (int k = 1; k < 9; ++k) {
    base[k] = base[k - 1] + pstep;
    asm("" : "+s"(base[k]));
  }
  if (!st.own) return;
  if (y > 0 && y < g.ny - 1) {
#pragma unroll
    for (int m = 0; m < 3; ++m) {  // directions along x: 0, then 1, then -1
      const int cx = m == 2 ? -1 : m;
      // what leaves through the inlet or outlet end is dropped
      if (!EDGE || cx == 0 || (cx > 0 ? !st.outlet : !st.inlet)) {
#pragma unroll
        for (int k = 0; k < 9; ++k)
          if (L::cx[k] == cx) *lane_ptr<S>(base[k], v[cx + 1] + (uint32_t)(L::cy[k] + 1) * rowb) = to_store<S>(c[k]);
      }
    }
    if (EDGE && VIRT && st.outlet) {
      int n = 0;
#pragma unroll
      for (int k = 0; k < 9; ++k)
        if (L::cx[k] == -1) *lane_ptr<S>(base[k], v[1] + (uint32_t)(L::cy[k] + 1) * rowb) = to_store<S>(o[n++]);
    }
    return;
  }
  // a row beside a wall or a periodic seam: the row offsets from row y - 1
  const int64_t up = (int64_t)rowb * (y < g.ny - 1 ? 2 : 2 - (int64_t)g.ny), down = (int64_t)rowb * (y > 0 ? 0 : g.ny);
  int n = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const bool bounce = walls && ((L::cy[k] < 0 && y == 0) || (L::cy[k] > 0 && y == g.ny - 1));  // uniform
    if (bounce) {  // to the opposite slot of the own cell
      *lane_ptr<S>(base[L::opp[k]] + rowb, v[1]) = to_store<S>(c[k]);
    } else {
      const uint64_t pr = base[k] + (uint64_t)(L::cy[k] < 0 ? down : (L::cy[k] > 0 ? up : (int64_t)rowb));
      if (!EDGE || L::cx[k] == 0 || (L::cx[k] > 0 ? !st.outlet : !st.inlet))
        *lane_ptr<S>(pr, v[L::cx[k] + 1]) = to_store<S>(c[k]);
      if (EDGE && VIRT && L::cx[k] == -1 && st.outlet) *lane_ptr<S>(pr, v[1]) = to_store<S>(o[n]);
    }
    if (L::cx[k] == -1) ++n;
  }
}

// Value of lane i (uniform) of v.
template <typename T>
__device__ __forceinline__ T lane_value(T v, int i) {
  if constexpr (sizeof(T) == 8) {
    union {
      T t;
      int w[2];
    } u;
    u.t = v;
    u.w[0] = __builtin_amdgcn_readlane(u.w[0], i);
    u.w[1] = __builtin_amdgcn_readlane(u.w[1], i);
    return u.t;
  } else {
    union {
      T t;
      int w;
    } u;
    u.t = v;
    u.w = __builtin_amdgcn_readlane(u.w, i);
    return u.t;
  }
}

// Velocity probe of a pass: step t of it records into out[t].
struct Probe {
  double* out[4];  // null: none
  int x, y, z;
};

Probe make_probe(const hlbm_lattice_s* L, int K);

// Mean-flow window of a pass (BGK).  Every step adds its values to the FP64 sums in
// step order, as single steps do; the sums pass through the levels in
// registers, so that memory holds them once a pass.  Objective terms: of a
// small region the levels record the cells' pre-collision state for the
// region pass (rec), of a large one (LARGE kernels) they add the terms (obj).
struct Window {
  double *rho, *j, *tau;
  ObjBox ob;
  double* obj;
  void* rec[4];  // records of level t (null: none); element type: the arithmetic type
};
Window make_window(const hlbm_lattice_s* L);

// Scalars of the collision (no body force: such lattices take single steps).
struct MarchColl {
  double tau0, omega0, kS;
  __device__ __forceinline__ Coll coll() const {
    Coll c;
    c.tau0 = tau0;
    c.omega0 = omega0;
    c.kS = kS;
    c.force[0] = c.force[1] = c.force[2] = 0.0;
    return c;
  }
};

// One wavefront's march over rows [y0, y1) of its strip.  Every level runs in
// every iteration (no branches): rows outside what a level needs are
// computed from whatever is there and reach no row that is stored.
// EDGE: 0 none, 1 the strip holds an inlet or outlet column, 2 the rows come
// near a wall, the probe or a small objective region (with or without an end).
// ACC: 0 plain, 1 window sums, 2 window sums and the terms of a large region,
// 3 either of the last or plain (no sums: wn.rho null).  SMAG: 2 by c.smag.
template <typename S, int K, bool HRR, int SMAG, int EDGE, int ACC>
__device__ __forceinline__ void march2d(const Geo& g, const Coll& c, const Strip& st, const int y0, const int y1,
                                        const S* __restrict__ A, S* __restrict__ B,
                                        const typename Prec<S>::Dd* __restrict__ dpor, const Probe& pr,
                                        const Window& wn) {
  using L = Lat<9>;
  using T = typename Prec<S>::T;
  using Dd = typename Prec<S>::Dd;
  constexpr int NB = K > 1 ? K - 1 : 1;
  // window sums: drho, j, tau_eff; ACC 2: and the objective terms of the region's cells
  constexpr int NO = Coef<9>::N, NW = SMAG ? 4 : 3, NT = ACC >= 2 ? NW + NO : NW;
  const bool walls = g.bcy != BC_PERIODIC;
  const int none = -0x40000000;
  const int row_first = walls ? 0 : none, row_last = walls ? g.ny - 1 : none;
  // recorded by the chunk that owns the cell
  const bool probe_lane =
      EDGE == 2 && pr.out[0] != nullptr && pr.y >= y0 && pr.y < y1 && st.own && !st.inlet && st.gx == pr.x;

  const int r0 = y0 - (K - 1), r_end = y1 + K - 2;
  const uint64_t pstep = uni64((uint64_t)g.plane * sizeof(S));
  RowPtr pa(A, r0, g.nx, g.ny, (int)sizeof(S)), pd(dpor, r0, g.nx, g.ny, (int)sizeof(Dd));
  const uint32_t off = lane_offset((uint32_t)st.x * (uint32_t)sizeof(S));
  const uint32_t offd = lane_offset((uint32_t)st.x * (uint32_t)sizeof(Dd));
  const uint32_t offb[3] = {lane_offset((uint32_t)st.xm * (uint32_t)sizeof(S)), off,
                            lane_offset((uint32_t)st.xp * (uint32_t)sizeof(S))};
  const uint32_t rowb = (uint32_t)g.nx * (uint32_t)sizeof(S);
  uint64_t below = uni64((uint64_t)B + (uint64_t)rowb * (uint64_t)(int64_t)(y0 - 1));
  auto load = [&](T (&s)[9], T& dd) {
    uint64_t pb = pa.base;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      s[k] = (T)*lane_ptr<const S>(pb, off);
      pb += pstep;
      asm("" : "+s"(pb));
    }
    dd = (T)*lane_ptr<const Dd>(pd.base, offd);
    pa.next();
    pd.next();
  };
  // What the pinned inlet column sends into the lattice (directions 1, 3 and
  // 8, the latter two alike) on row r0 + lane; the rest of that column is
  // used by no other.  A chunk's rows and halo fit the 64 lanes.
  T in1 = (T)0, in3 = (T)0;
  if (EDGE && st.ends) {
    const int row = wrap_row(r0 + (int)(threadIdx.x & 63), g.ny);
    const T ui = inlet_velocity<T>(g, row);
    in1 = (T)to_store<S>(inlet_value<9, T>(1, ui));
    in3 = (T)to_store<S>(inlet_value<9, T>(3, ui));
  }
  // window: rows of the sums, lanes that add to them and lanes in the region
  const uint32_t off8 = lane_offset((uint32_t)st.x * 8u);
  RowPtr pw(nullptr, r0, g.nx, g.ny, 8);
  uint64_t out_row = uni64((uint64_t)g.nx * 8u * (uint64_t)(int64_t)y0);
  const uint64_t sums[4] = {uni64((uint64_t)wn.rho), uni64((uint64_t)wn.j), uni64((uint64_t)wn.j + (uint64_t)g.plane * 8),
                            uni64((uint64_t)(SMAG == 2 && !wn.tau ? wn.rho : wn.tau))};
  const bool sums_on = ACC && (ACC != 3 || wn.rho != nullptr), tau_on = SMAG != 2 || wn.tau != nullptr;
  const bool adds = sums_on && st.own && !st.inlet;
  const int rx = st.gx - wn.ob.lo[0];
  const bool in_cols = ACC && wn.ob.active && adds && rx >= 0 && rx < wn.ob.rn[0];
  // region rows of this chunk (empty where the strip has no region column)
  const bool any_col = ACC && __ballot(in_cols) != 0;
  const int reg0 = any_col ? (wn.ob.lo[1] > y0 ? wn.ob.lo[1] : y0) : 0;
  const int reg1 = any_col ? (wn.ob.lo[1] + wn.ob.rn[1] < y1 ? wn.ob.lo[1] + wn.ob.rn[1] : y1) : 0;
  // the terms' slots: lanes outside the region's columns read its nearest one and write nothing
  const uint32_t offr =
      lane_offset(8u * (uint32_t)(ACC >= 2 ? (rx < 0 ? 0 : (rx < wn.ob.rn[0] ? rx : wn.ob.rn[0] - 1)) : 0));
  auto term_slot = [&](const int row, const int m) {
    return lane_ptr<double>(uni64((uint64_t)(wn.obj + m * wn.ob.rplane +
                                             (int64_t)wn.ob.rn[0] * (int64_t)(row - wn.ob.lo[1]))), offr);
  };
  double wcur[NT], hold[NB][NT];
  auto load_sums = [&](const int row) {
    if (sums_on && row >= y0 && row < y1) {
#pragma unroll
      for (int a = 0; a < NW; ++a) wcur[a] = *lane_ptr<const double>(sums[a] + pw.base, off8);
    }
    if (ACC >= 2 && row >= reg0 && row < reg1) {
#pragma unroll
      for (int m = 0; m < NO; ++m) wcur[NT - NO + m] = *term_slot(row, m);
    }
    if (ACC) pw.next();
  };
  Wait<T> w[NB];
  T cur[9], dcur, d[K];
  auto step = [&](const int r, auto phase) {
    constexpr int PH = decltype(phase)::value;
    T s[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) s[k] = cur[k];
#pragma unroll
    for (int t = K - 1; t > 0; --t) d[t] = d[t - 1];
    d[0] = dcur;
    double sum[NT];
#pragma unroll
    for (int a = 0; a < NT; ++a) sum[a] = wcur[a];
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int row = r - t;
      if (t == 1) {  // level 0 has used the row: load the next one (past the last: in bounds, unused)
        __builtin_amdgcn_sched_barrier(0);
        load(cur, dcur);
        load_sums(r + 1);
      }
      if (EDGE == 2 || t == 1) __builtin_amdgcn_sched_barrier(0);  // EDGE 2: levels kept apart (registers)
      if (t == K - 1 && row < y0) return;
      T drho, jx, jy, jz, omega, taue, p2[6], o[3], ns[9];
      cell_moments<9, T>(s, drho, jx, jy, jz);
      const T rho = (T)1 + drho;
      const T ir = recip(rho);
      if (EDGE == 2 && probe_lane && row == pr.y) *pr.out[t] = (double)(jy * ir);
      relaxation<9, T, HRR>(c, SMAG == 2 ? c.smag != 0 : SMAG == 1, s, drho, jx, jy, jz, ir, omega, taue, p2);
      if (ACC) {
        sum[0] = sum[0] + (double)drho;
        sum[1] = sum[1] + (double)jx;
        sum[2] = sum[2] + (double)jy;
        if (SMAG) sum[NW - 1] = sum[NW - 1] + (double)taue;
        if (ACC >= 2 && row >= reg0 && row < reg1) {
          double sd[9], terms[NO], dr, ax, ay, az, P[6];
#pragma unroll
          for (int k = 0; k < 9; ++k) sd[k] = (double)s[k];
          cell_moments<9, double>(sd, dr, ax, ay, az);
          neq_flux<9, double>(sd, dr, ax, ay, az, 1.0 / (1.0 + dr), P);
          objective_terms<9>(wn.ob, (double)d[t], dr, ax, ay, az, P, terms);
#pragma unroll
          for (int m = 0; m < NO; ++m) sum[NT - NO + m] = sum[NT - NO + m] + terms[m];
          if (t == K - 1 && in_cols) {
#pragma unroll
            for (int m = 0; m < NO; ++m) *term_slot(row, m) = sum[NT - NO + m];
          }
        }
        if (t == K - 1) {
          if (adds) {
#pragma unroll
            for (int a = 0; a < NW; ++a)
              if (a < 3 || tau_on) *lane_ptr<double>(sums[a] + out_row, off8) = sum[a];
          }
          out_row += (uint64_t)g.nx * 8u;
        } else {  // to the next level, one row later
#pragma unroll
          for (int a = 0; a < NT; ++a) {
            const double v = hold[t % NB][a];
            hold[t % NB][a] = sum[a];
            sum[a] = v;
          }
        }
        if (ACC == 1 && EDGE == 2 && row >= reg0 && row < reg1) {
          if (in_cols && wn.rec[t])
            store_record<9, T>(wn.rec[t], (int64_t)rx + (int64_t)wn.ob.rn[0] * (int64_t)(row - wn.ob.lo[1]), s, d[t]);
        }
      }
      collide_cell<9, T, HRR>(c, s, drho, jx, jy, jz, rho, ir, d[t], omega, p2);
      if (EDGE == 1 || (EDGE == 2 && st.ends)) {
        const T ux = jx * ir, uy = jy * ir, uz = jz * ir;
        const T uu = ux * ux + uy * uy + uz * uz;
        int n = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k)
          if (L::cx[k] == -1) o[n++] = (T)to_store<S>(outlet_value<9, T>(k, ux, uy, uz, uu));
        const T a = lane_value(in1, row - r0), b = lane_value(in3, row - r0);
        s[1] = st.inlet ? a : s[1];
        s[3] = st.inlet ? b : s[3];
        s[8] = st.inlet ? b : s[8];
      }
      if (t == K - 1) {
        push_row<EDGE, true, S, T>(g, st, walls, row, below, offb, pstep, rowb, s, o);
        below += rowb;
      } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) s[k] = (T)to_store<S>(s[k]);
        const int at_wall = row == row_first ? -1 : (row == row_last ? 1 : (row == row_last + 1 ? 2 : 0));
        hand_on<EDGE, T>((PH + t) & 1, st, at_wall, s, o, w[t % NB], ns);
#pragma unroll
        for (int k = 0; k < 9; ++k) s[k] = ns[k];
      }
    }
  };

  load(cur, dcur);
  load_sums(r0);
  for (int r = r0;; r += 2) {
    step(r, std::integral_constant<int, 0>{});
    if (r + 1 > r_end) break;
    step(r + 1, std::integral_constant<int, 1>{});
    if (r + 2 > r_end) break;
  }
}

// Wavefronts per SIMD the register allocation aims at: at 3 the FP64 passes of
// four steps spill (1100 x 410: 11.2 us a step instead of 6.1).  As given, no
// FP64 or FP16 pass uses scratch; of the FP32 ones BGK with closure does, 10
// registers (44 bytes a lane) with four steps and 9 with two, without 1 and 3.
template <typename S, int K>
constexpr int march2d_waves() {
  return sizeof(S) == 8 ? (K > 2 ? 2 : 3) : (K > 2 ? 4 : 6);
}
// With window sums, which wait in registers as well.  Without a large region's
// terms nothing spills; with them the passes of four do (56 to 167 registers; they
// pay beyond the caches only), and FP64 with closure (31, 96 bytes a lane).
template <typename S, int K, bool LARGE>
constexpr int window2d_waves() {
  return LARGE || sizeof(S) == 8 || K > 2 ? 2 : 4;
}

// K primal steps (rows a3, a4).  HRR, SMAG: collision model, closure.
template <typename S, int K, bool HRR, bool SMAG>
__global__ __launch_bounds__(256, (march2d_waves<S, K>())) void k_march2d(const Geo g, const MarchColl mc, const March2 m,
                                                 const S* __restrict__ A, S* __restrict__ B,
                                                 const typename Prec<S>::Dd* __restrict__ dpor, const Probe pr) {
  const Coll c = mc.coll();
  const int id = sweep_tile((int)blockIdx.x, (int)gridDim.x) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  if (id >= m.strips * m.chunks) return;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<K>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  const bool at_walls = g.bcy != BC_PERIODIC && (y0 < K || y1 > g.ny - K);
  const bool probed = pr.out[0] != nullptr && pr.y >= y0 && pr.y < y1 && __ballot(st.own && st.gx == pr.x) != 0;
  const Window wn{};
  if (at_walls || probed)
    march2d<S, K, HRR, SMAG, 2, 0>(g, c, st, y0, y1, A, B, dpor, pr, wn);
  else if (st.ends)
    march2d<S, K, HRR, SMAG, 1, 0>(g, c, st, y0, y1, A, B, dpor, pr, wn);
  else
    march2d<S, K, HRR, SMAG, 0, 0>(g, c, st, y0, y1, A, B, dpor, pr, wn);
}

// K primal steps of a mean-flow window (BGK).  LARGE: the objective region is
// a sizeable part of the lattice, its terms are added by the sweep.
template <typename S, int K, bool SMAG, bool LARGE>
__global__ __launch_bounds__(256, (window2d_waves<S, K, LARGE>())) void k_window2d(
    const Geo g, const MarchColl mc, const March2 m, const S* __restrict__ A, S* __restrict__ B,
    const typename Prec<S>::Dd* __restrict__ dpor, const Probe pr, const Window wn) {
  const Coll c = mc.coll();
  const int id = sweep_tile((int)blockIdx.x, (int)gridDim.x) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  if (id >= m.strips * m.chunks) return;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<K>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  const bool at_walls = g.bcy != BC_PERIODIC && (y0 < K || y1 > g.ny - K);
  const bool probed = pr.out[0] != nullptr && pr.y >= y0 && pr.y < y1 && __ballot(st.own && st.gx == pr.x) != 0;
  const ObjBox& ob = wn.ob;
  const bool recorded = !LARGE && ob.active && y0 < ob.lo[1] + ob.rn[1] && y1 > ob.lo[1] &&
                        __ballot(st.own && st.gx >= ob.lo[0] && st.gx < ob.lo[0] + ob.rn[0]) != 0;
  constexpr int ACC = LARGE ? 2 : 1;
  if (at_walls || probed || recorded)
    march2d<S, K, false, SMAG, 2, ACC>(g, c, st, y0, y1, A, B, dpor, pr, wn);
  else if (st.ends)
    march2d<S, K, false, SMAG, 1, ACC>(g, c, st, y0, y1, A, B, dpor, pr, wn);
  else
    march2d<S, K, false, SMAG, 0, ACC>(g, c, st, y0, y1, A, B, dpor, pr, wn);
}

// =========================================================================
// adjoint: K iterations (row a8) of the BGK adjoint with a frozen relaxation
// time, moment-form objectives.  phihat streams like the primal populations;
// the frozen data of a row waits for the later levels beside it.  Nothing
// arrives at the outlet from beyond; what leaves through it arrives on the
// lane beyond the outlet and enters the next level's virtual-column term from
// there (level 0 and the last level: the pv buffers).
// =========================================================================

struct MarchAdj {
  int les;  // per-cell omega
  double omega0;
};

template <typename T, int K, bool SRC, int EDGE>
__device__ __forceinline__ void march2d_adjoint(const Geo& g, const ObjBox& ob, const MarchAdj& ac, const Strip& st,
                                                const int y0, const int y1, const T* __restrict__ A,
                                                T* __restrict__ B, const T* __restrict__ prep,
                                                const double* __restrict__ src, const double* __restrict__ oprep,
                                                const T* __restrict__ pv_in, T* __restrict__ pv_out) {
  using L = Lat<9>;
  constexpr int NB = K > 1 ? K - 1 : 1;
  const bool walls = g.bcy != BC_PERIODIC;
  const int none = -0x40000000;
  const int row_first = walls ? 0 : none, row_last = walls ? g.ny - 1 : none;
  const int r0 = y0 - (K - 1), r_end = y1 + K - 2;
  const uint64_t pstep = uni64((uint64_t)g.plane * sizeof(T));
  RowPtr pa(A, r0, g.nx, g.ny, (int)sizeof(T)), pp(prep, r0, g.nx, g.ny, (int)sizeof(T));
  const uint32_t off = lane_offset((uint32_t)st.x * (uint32_t)sizeof(T));
  const uint32_t offb[3] = {lane_offset((uint32_t)st.xm * (uint32_t)sizeof(T)), off,
                            lane_offset((uint32_t)st.xp * (uint32_t)sizeof(T))};
  const uint32_t rowb = (uint32_t)g.nx * (uint32_t)sizeof(T);
  uint64_t below = uni64((uint64_t)B + (uint64_t)rowb * (uint64_t)(int64_t)(y0 - 1));
  struct Frozen {
    T tx, ty, d, om;
  };
  const bool reg_lane = SRC && st.x >= ob.lo[0] && st.x < ob.lo[0] + ob.rn[0];
  const uint32_t reg_x = lane_offset(8 * (uint32_t)(st.x - ob.lo[0]));
  // The source waits in registers beside the frozen data where these suffice;
  // the FP64 passes of four steps read it again at each level (from L2).
  constexpr bool QREG = SRC && (K == 2 || sizeof(T) == 4);
  double qcur[6];  // of the row loaded last
  T q[QREG ? K : 1][6];
  // the objective's source on row y, zero outside its region
  auto load_source = [&](int y, double (&a)[6]) {
    uint64_t base[6];  // formed ahead of the masked loads
    base[0] = uni64((uint64_t)src + 8 * (uint64_t)(Coef<9>::A0 * ob.rplane + (int64_t)ob.rn[0] * (y - ob.lo[1])));
#pragma unroll
    for (int m = 1; m < 6; ++m) {
      base[m] = base[m - 1] + 8 * (uint64_t)ob.rplane;
      asm("" : "+s"(base[m]));
    }
#pragma unroll
    for (int m = 0; m < 6; ++m) a[m] = 0.0;
    if (reg_lane && y >= ob.lo[1] && y < ob.lo[1] + ob.rn[1]) {
#pragma unroll
      for (int m = 0; m < 6; ++m) a[m] = *lane_ptr<const double>(base[m], reg_x);
    }
  };
  auto load = [&](T (&s)[9], Frozen& f) {
    uint64_t pb = pa.base;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      s[k] = *lane_ptr<const T>(pb, off);
      pb += pstep;
      asm("" : "+s"(pb));
    }
    f.tx = *lane_ptr<const T>(pp.base, off);
    f.ty = *lane_ptr<const T>(pp.base + pstep, off);
    f.d = *lane_ptr<const T>(pp.base + 2 * pstep, off);
    f.om = *lane_ptr<const T>(pp.base + (ac.les ? 3 : 2) * pstep, off);
    if (QREG) load_source(pa.y, qcur);
    pa.next();
    pp.next();
  };
  // outlet rows r0 + lane: 1/rho, u, and the adjoint on the virtual column
  T iro = (T)0, uox = (T)0, uoy = (T)0, pv0[3] = {(T)0, (T)0, (T)0};
  if (EDGE && st.any_outlet) {
    const int row = wrap_row(r0 + (int)(threadIdx.x & 63), g.ny);
    iro = (T)1 / (T)oprep[row];
    uox = (T)oprep[g.gplane + row];
    uoy = (T)oprep[2 * g.gplane + row];
    int n = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k)
      if (L::cx[k] == -1) pv0[n++] = pv_in[k * g.gplane + row];
  }
  Wait<T> w[NB];
  T cur[9];
  Frozen fcur, f[K];
  auto step = [&](const int r, auto phase) {
    constexpr int PH = decltype(phase)::value;
    T s[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) s[k] = cur[k];
#pragma unroll
    for (int t = K - 1; t > 0; --t) f[t] = f[t - 1];
    f[0] = fcur;
    if (QREG) {
#pragma unroll
      for (int t = K - 1; t > 0; --t)
#pragma unroll
        for (int m = 0; m < 6; ++m) q[QREG ? t : 0][m] = q[QREG ? t - 1 : 0][m];
#pragma unroll
      for (int m = 0; m < 6; ++m) q[0][m] = (T)qcur[m];
    }
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int row = r - t;
      if (t == 1) {
        __builtin_amdgcn_sched_barrier(0);
        load(cur, fcur);
      }
      if (EDGE == 2 || t == 1) __builtin_amdgcn_sched_barrier(0);
      if (t == K - 1 && row < y0) return;
      const int y = row < 0 || row >= g.ny ? wave_uniform(wrap_row(row, g.ny)) : row;
      if (SRC && !QREG) load_source(y, qcur);
      T pv[9];
      if (EDGE && st.any_outlet) {
        int n = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          if (L::cx[k] != -1) continue;
          if (t == 0) {
            pv[k] = lane_value(pv0[n], row - r0);
            // beyond the outlet: no adjoint inflow (a wall's bounce-back stays)
            const bool kept = walls && ((L::cy[k] > 0 && y == 0) || (L::cy[k] < 0 && y == g.ny - 1));
            s[k] = st.outlet && !kept ? (T)0 : s[k];
          } else {
            pv[k] = lane_shift(s[L::opp[k]], -1);
            const bool beyond = walls && ((L::cy[k] < 0 && y == 0) || (L::cy[k] > 0 && y == g.ny - 1));
            pv[k] = beyond ? (T)0 : pv[k];
          }
          ++n;
        }
      }
      T lam[9], c[9];
      adjoint_bgk<9, T>(s, f[t].tx, f[t].ty, (T)0, f[t].d, ac.les ? f[t].om : (T)ac.omega0, lam);
      if (EDGE && st.any_outlet) {
        T lo[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) lo[k] = lam[k];
        const int i = row - r0;
        adjoint_outlet<9, T>(pv, lane_value(iro, i), lane_value(uox, i), lane_value(uoy, i), (T)0, lo);
#pragma unroll
        for (int k = 0; k < 9; ++k) lam[k] = st.outlet ? lo[k] : lam[k];
      }
      if (SRC) {  // zero outside the objective's region
#pragma unroll
        for (int m = 0; m < 6; ++m)
          if (!QREG) q[0][m] = (T)qcur[m];
#pragma unroll
        for (int i = 0; i < 9; ++i) lam[i] -= quad_eval<9, T>(q[QREG ? t : 0], i);
      }
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        c[k] = lam[L::opp[k]];
        if (EDGE && L::cx[k] == 1) c[k] = st.inlet ? (T)0 : c[k];  // lambda = 0 at the pinned inlet
      }
      const T o[3] = {(T)0, (T)0, (T)0};
      if (t == K - 1) {
        push_row<EDGE, false, T, T>(g, st, walls, row, below, offb, pstep, rowb, c, o);
        below += rowb;
        if (EDGE && st.any_outlet) {
          const bool put = st.own && st.outlet;
#pragma unroll
          for (int k = 0; k < 9; ++k) {
            if (L::cx[k] != -1) continue;
            int vy = y - L::cy[k];
            const bool cell = !walls || (vy >= 0 && vy < g.ny);
            vy = vy < 0 ? vy + g.ny : (vy >= g.ny ? vy - g.ny : vy);
            if (put && cell) pv_out[k * g.gplane + vy] = lam[k];
          }
        }
      } else {
        const int at_wall = row == row_first ? -1 : (row == row_last ? 1 : (row == row_last + 1 ? 2 : 0));
        hand_on<EDGE, T>((PH + t) & 1, st, at_wall, c, o, w[t % NB], s);
      }
    }
  };

  load(cur, fcur);
  for (int r = r0;; r += 2) {
    step(r, std::integral_constant<int, 0>{});
    if (r + 1 > r_end) break;
    step(r + 1, std::integral_constant<int, 1>{});
    if (r + 2 > r_end) break;
  }
}

// Per iteration, single sweep -> pass: 8192 x 4096, drag plane, FP64 982 -> 329
// us, FP32 480 -> 174; dissipation box over 6/11 of it (48 bytes of FP64
// source a cell beside the 52 or 104 of phi and the frozen data) 1169 -> 449 and
// 653 -> 250; 1100 x 410 FP32 7.4 -> 6.6 and 7.6 -> 6.8, 220 x 41 FP64
// 4.1 -> 3.7.  On the small ones the strips that hold the outlet column set the
// time: its virtual-column term doubles the instructions of a level.
// With a third wavefront per SIMD the passes of four spill (FP32 1100 x 410
// 6.6 -> 8.1 us).
template <typename T, int K>
__global__ __launch_bounds__(256, (sizeof(T) == 8 || K > 2 ? 2 : 4)) void k_march2d_adjoint(
    const Geo g, const ObjBox ob, const MarchAdj ac, const March2 m, const T* __restrict__ A, T* __restrict__ B,
    const T* __restrict__ prep, const double* __restrict__ src, const double* __restrict__ oprep,
    const T* __restrict__ pv_in, T* __restrict__ pv_out) {
  const int id = sweep_tile((int)blockIdx.x, (int)gridDim.x) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  if (id >= m.strips * m.chunks) return;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<K>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  const bool walls = g.bcy != BC_PERIODIC;
  const bool at_walls = walls && (y0 < K || y1 > g.ny - K);
  // whether any row of the march (halo included) can hold region cells
  const bool rows = !walls || (y1 + K - 2 >= ob.lo[1] && y0 - (K - 1) < ob.lo[1] + ob.rn[1]);
  const bool src_here =
      ob.active && rows && __ballot(st.x >= ob.lo[0] && st.x < ob.lo[0] + ob.rn[0]) != 0;
  if (at_walls)
    march2d_adjoint<T, K, true, 2>(g, ob, ac, st, y0, y1, A, B, prep, src, oprep, pv_in, pv_out);
  else if (st.ends)
    march2d_adjoint<T, K, true, 1>(g, ob, ac, st, y0, y1, A, B, prep, src, oprep, pv_in, pv_out);
  else if (src_here)
    march2d_adjoint<T, K, true, 0>(g, ob, ac, st, y0, y1, A, B, prep, src, oprep, pv_in, pv_out);
  else
    march2d_adjoint<T, K, false, 0>(g, ob, ac, st, y0, y1, A, B, prep, src, oprep, pv_in, pv_out);
}

}  // namespace hlbm
