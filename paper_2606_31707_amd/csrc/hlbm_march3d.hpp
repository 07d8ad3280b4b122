// hlbm_march3d.hpp -- D3Q19 sweeps that take two steps in one pass over memory.
//
// A workgroup of R wavefronts holds R rows of 64 columns and marches along z.
// Level 0 collides plane z as it comes from memory; its post-collision values
// move along x by lane shifts, along y through LDS (the ten directions with a
// y component, one barrier a plane) and along z by waiting in registers; level
// 1 then collides plane z - 1 and pushes the result to the second array.  62
// columns and R - 2 rows of a tile and the planes of its chunk are its own, the
// rest is recomputed by the neighbours.  Input and output are the canonical
// layout in two arrays; every cell runs the per-cell code of the single steps
// and is rounded to the storage type between the levels, so that the results
// are bitwise those of two single steps.
//
// What bounds it: memory requests.  A single step moves every population twice
// and is bound by that; a pass moves each 62 x (R - 2) tile once in two steps
// and reads 1.24 (FP32) or 1.38 times (FP64) what it needs because of the rows
// and columns that neighbours recompute.  Its stores of whole rows shifted by
// one cell do not fill 128-byte lines; with stores aligned to lines the FP32
// pass takes 684 instead of 840 us, but no layout of 64 own columns was found
// whose halo loads did not cost that again (816 us at best).  The plane bases of
// loads and stores do not all fit the scalar registers: 90 of them spill to
// vector lanes in FP32 with closure, 201 with the window's, 109 to 225 in FP64
// (there a window with closure also spills 4 vector registers).  us a step, single
// steps / passes: 768x384x128 FP32 1104 / 845, FP64 2262 / 1558; 756x168x84
// with walls FP32 301 / 204, FP64 612 / 431; 192x96x64 with walls FP32 31.4 /
// 31.4 (periodic 26.0), FP64 56.4 / 54.4.
#pragma once

#include "hlbm_march2d.hpp"

namespace hlbm {

template <typename T>
constexpr int march3d_rows() {
  return march3d_rows_of(sizeof(T) == 8);
}

// LDS slot of a direction with cy != 0.
__device__ constexpr int yslot(int k) {
  int n = 0;
  for (int i = 0; i < k; ++i)
    if (Lat<19>::cy[i] != 0) ++n;
  return n;
}
// The i-th direction with cz = CZ.
template <int CZ>
__device__ constexpr int dir19(int i) {
  int n = 0;
  for (int k = 0; k < 19; ++k)
    if (Lat<19>::cz[k] == CZ && n++ == i) return k;
  return -1;
}
__device__ constexpr int zslot(int k) {  // place of k among the directions of its cz
  int n = 0;
  for (int i = 0; i < k; ++i)
    if (Lat<19>::cz[i] == Lat<19>::cz[k]) ++n;
  return n;
}

// One lane's place in a tile.
struct Tile3 {
  int wave, lane;
  int gx, gy;       // column and row (may lie outside the lattice)
  int xm, x, xp;    // columns, wrapped or clamped into [0, nx)
  int y;            // row, wrapped into [0, ny)
  bool own;         // column and row are the tile's own
  bool own_row;     // the row is (uniform)
  bool inlet, outlet, beyond;  // lane on the inlet column, on the outlet column, one past it
};
template <int R>
__device__ __forceinline__ Tile3 make_tile3(const Geo& g, int tx, int ty) {
  Tile3 t;
  t.lane = threadIdx.x & 63;
  t.wave = wave_uniform((int)(threadIdx.x >> 6));
  t.gx = tx * 62 - 1 + t.lane;
  t.gy = ty * (R - 2) - 1 + t.wave;
  const bool per = g.bcx == BC_PERIODIC;
  auto col = [&](int x) {
    if (per) {
      x %= g.nx;
      return x < 0 ? x + g.nx : x;
    }
    return x < 0 ? 0 : (x >= g.nx ? g.nx - 1 : x);
  };
  t.x = col(t.gx);
  t.xm = col(t.gx - 1);
  t.xp = col(t.gx + 1);
  t.y = wave_uniform(wrap_row(t.gy, g.ny));
  t.own_row = t.wave >= 1 && t.wave <= R - 2 && t.gy < g.ny;
  t.own = t.own_row && t.lane >= 1 && t.lane <= 62 && t.gx < g.nx;
  t.inlet = g.bcx == BC_INOUT && t.gx == 0;
  t.outlet = g.bcx == BC_INOUT && t.gx == g.nx - 1;
  t.beyond = g.bcx == BC_INOUT && t.gx == g.nx;
  return t;
}

// What level 1 waits for: the values moving up (cz = +1) from the last two
// planes and those staying on the last plane; at y walls also what the last
// plane's row beside the wall bounces into the direction with cz = -1.
template <typename T>
struct Wait3 {
  T up2[5], up1[5], mid[9], save;
};

// Hands the post-collision values c of plane z to level 1: s becomes the state
// of plane z - 1, w the rest.  lds: this plane's buffer.  Every wavefront
// writes its row's values and passes the barrier; rows that are not the
// tile's own stop there.
template <int R, bool WALLS, typename T>
__device__ __forceinline__ void hand_on3(const Geo& g, const Tile3& t, const int z, T* __restrict__ lds,
                                         const T (&c)[19], Wait3<T>& w, T (&s)[19]) {
  using L = Lat<19>;
  T* mine = lds + 1 + t.wave * 64 + t.lane;
#pragma unroll
  for (int k = 0; k < 19; ++k)
    if (L::cy[k] != 0) mine[yslot(k) * R * 64] = c[k];
  __syncthreads();
  if (!t.own_row) return;
  T sh[19];
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    if (L::cy[k] == 0)
      sh[k] = lane_shift(c[k], L::cx[k]);
    else
      sh[k] = mine[yslot(k) * R * 64 - L::cy[k] * 64 - L::cx[k]];
  }
  const bool low = WALLS && g.bcy != BC_PERIODIC && t.gy == 0, high = WALLS && g.bcy != BC_PERIODIC && t.gy == g.ny - 1;
  T keep = (T)0;
  if (WALLS && (low || high)) {
    // halfway bounce-back: the value stays on its cell; in the plane at once,
    // for cz = -1 when level 1 comes to this plane
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      if (!((L::cy[k] > 0 && low) || (L::cy[k] < 0 && high))) continue;
      if (L::cz[k] == 0) sh[k] = c[L::opp[k]];
      // (beyond a wall on z, up1 keeps the last plane's values)
      if (L::cz[k] > 0 && !(g.bcz != BC_PERIODIC && z == g.nz)) w.up1[zslot(k)] = c[L::opp[k]];
      if (L::cz[k] < 0) keep = c[L::opp[k]];
    }
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    s[dir19<1>(i)] = w.up2[i];
    s[dir19<-1>(i)] = sh[dir19<-1>(i)];
    w.up2[i] = w.up1[i];
    w.up1[i] = sh[dir19<1>(i)];
  }
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    s[dir19<0>(i)] = w.mid[i];
    w.mid[i] = sh[dir19<0>(i)];
  }
  if (WALLS && (low || high)) {
#pragma unroll
    for (int k = 0; k < 19; ++k)
      if (L::cz[k] < 0 && ((L::cy[k] > 0 && low) || (L::cy[k] < 0 && high))) s[k] = w.save;
    w.save = keep;
  }
  if (WALLS && g.bcz != BC_PERIODIC) {
    if (z == 0) {  // what goes down from the first plane is its upward arrival
#pragma unroll
      for (int i = 0; i < 5; ++i) w.up2[i] = c[L::opp[dir19<1>(i)]];
    }
    if (z == g.nz) {  // the plane beyond the last: what went up from it bounced
#pragma unroll
      for (int i = 0; i < 5; ++i) s[dir19<-1>(i)] = w.up2[zslot(L::opp[dir19<-1>(i)])];
    }
    if (z == g.nz - 1) {  // kept as it is for that
#pragma unroll
      for (int i = 0; i < 5; ++i) w.up1[i] = c[dir19<1>(i)];
    }
  }
}

// Row offsets in bytes of the planes z - 1, z, z + 1 and rows y - 1, y, y + 1
// (wrapped; a bounce takes the place of one that would leave through a wall).
struct Offsets3 {
  int64_t z[3], y[3];
};
__device__ __forceinline__ Offsets3 offsets3(const Geo& g, int z, int y, int size) {
  const int64_t rowb = (int64_t)g.nx * size, planeb = rowb * g.ny;
  Offsets3 o;
  o.z[0] = planeb * (z > 0 ? z - 1 : g.nz - 1);
  o.z[1] = planeb * z;
  o.z[2] = planeb * (z < g.nz - 1 ? z + 1 : 0);
  o.y[0] = rowb * (y > 0 ? y - 1 : g.ny - 1);
  o.y[1] = rowb * y;
  o.y[2] = rowb * (y < g.ny - 1 ? y + 1 : 0);
  return o;
}

// Stores the post-collision values c of an own cell (row y, plane z) to the
// slots they move to (B).  VIRT, o: the virtual column's values on the outlet
// lane (cx = -1 directions, in order).
template <bool ENDS, bool WALLS, bool VIRT, typename S, typename T>
__device__ __forceinline__ void push3(const Geo& g, const Tile3& t, const int z, S* __restrict__ B,
                                      const uint32_t (&v)[3], const T (&c)[19], const T (&o)[5]) {
  using L = Lat<19>;
  const Offsets3 of = offsets3(g, z, t.y, (int)sizeof(S));
  const uint64_t pstep = uni64((uint64_t)g.plane * sizeof(S));
  const uint32_t here = v[1];
  const uint64_t own = of.z[1] + of.y[1];
  const bool ylo = g.bcy != BC_PERIODIC && t.y == 0, yhi = g.bcy != BC_PERIODIC && t.y == g.ny - 1;
  const bool zlo = g.bcz != BC_PERIODIC && z == 0, zhi = g.bcz != BC_PERIODIC && z == g.nz - 1;
  uint64_t base[19];  // formed ahead of the masked stores
  base[0] = uni64((uint64_t)B);
#pragma unroll
  for (int k = 1; k < 19; ++k) {
    base[k] = base[k - 1] + pstep;
    asm("" : "+s"(base[k]));
  }
  if (!t.own) return;
#pragma unroll
  for (int m = 0; m < 3; ++m) {  // directions along x: 0, then 1, then -1
    const int cx = m == 2 ? -1 : m;
    int n = 0;
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      if (L::cx[k] != cx) continue;
      // a bounced value goes to the opposite slot of the own cell
      const bool bounce = WALLS && ((L::cy[k] < 0 && ylo) || (L::cy[k] > 0 && yhi) || (L::cz[k] < 0 && zlo) ||
                                    (L::cz[k] > 0 && zhi));  // uniform
      uint64_t row = base[k] + of.z[L::cz[k] + 1] + of.y[L::cy[k] + 1];
      uint32_t col = v[cx + 1];
      if (WALLS) {
        const uint64_t back = base[L::opp[k]] + own;
        row = bounce ? back : row;
        col = bounce ? here : col;
      }
      // what leaves through the inlet or outlet end is dropped
      if (!ENDS || cx == 0 || bounce || (cx > 0 ? !t.outlet : !t.inlet)) *lane_ptr<S>(row, col) = to_store<S>(c[k]);
      if (ENDS && VIRT && cx == -1 && t.outlet && !bounce) *lane_ptr<S>(row, v[1]) = to_store<S>(o[n]);
      if (cx == -1) ++n;
    }
  }
}

template <typename S, bool HRR, bool SMAG, bool ENDS, bool WALLS, bool ACC>
__device__ __forceinline__ void march3d(const Geo& g, const Coll& c, const March3& m, const int tx, const int ty,
                                        const int z0, const int z1, const S* __restrict__ A, S* __restrict__ B,
                                        const typename Prec<S>::Dd* __restrict__ dpor, const Probe& pr,
                                        const Window& wn, typename Prec<S>::T* __restrict__ lds) {
  using L = Lat<19>;
  using T = typename Prec<S>::T;
  using Dd = typename Prec<S>::Dd;
  constexpr int R = march3d_rows<T>();
  const Tile3 t = make_tile3<R>(g, tx, ty);
  const uint64_t pstep = uni64((uint64_t)g.plane * sizeof(S));
  const uint32_t off = lane_offset((uint32_t)t.x * (uint32_t)sizeof(S));
  const uint32_t offd = lane_offset((uint32_t)t.x * (uint32_t)sizeof(Dd));
  const uint32_t offb[3] = {lane_offset((uint32_t)t.xm * (uint32_t)sizeof(S)), off,
                            lane_offset((uint32_t)t.xp * (uint32_t)sizeof(S))};
  RowPtr pa(A, z0 - 1, g.nx * g.ny, g.nz, (int)sizeof(S)), pd(dpor, z0 - 1, g.nx * g.ny, g.nz, (int)sizeof(Dd));
  pa.base += (uint64_t)t.y * (uint64_t)g.nx * sizeof(S);
  pd.base += (uint64_t)t.y * (uint64_t)g.nx * sizeof(Dd);
  auto load = [&](T (&s)[19], T& dd) {
    uint64_t pb = pa.base;
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      s[k] = (T)*lane_ptr<const S>(pb, off);
      pb += pstep;
      asm("" : "+s"(pb));
    }
    dd = (T)*lane_ptr<const Dd>(pd.base, offd);
    pa.next();
    pd.next();
  };
  // what the pinned inlet column sends into the lattice from this row
  T in1 = (T)0, in4 = (T)0;
  if (ENDS) {
    const T ui = inlet_velocity<T>(g, t.y);
    in1 = (T)to_store<S>(inlet_value<19, T>(1, ui));
    in4 = (T)to_store<S>(inlet_value<19, T>(4, ui));
  }
  const bool probe_lane = pr.out[0] != nullptr && t.own && !t.inlet && t.gx == pr.x && t.gy == pr.y;
  const int probe_z = __ballot(probe_lane) != 0 ? pr.z : -0x40000000;
  // window: sums drho, j, tau_eff and, where the wavefront holds region cells, their planes
  constexpr int NW = SMAG ? 5 : 4;
  const uint64_t sums[5] = {uni64((uint64_t)wn.rho), uni64((uint64_t)wn.j), uni64((uint64_t)(wn.j + g.plane)),
                            uni64((uint64_t)(wn.j + 2 * g.plane)), uni64((uint64_t)wn.tau)};
  const uint32_t off8 = lane_offset((uint32_t)t.x * 8u);
  const bool adds = ACC && t.own && !t.inlet;
  const ObjBox& ob = wn.ob;
  const bool in_region = ACC && ob.active && adds && t.gx >= ob.lo[0] && t.gx < ob.lo[0] + ob.rn[0] &&
                         t.gy >= ob.lo[1] && t.gy < ob.lo[1] + ob.rn[1];
  const bool any_region = ACC && __ballot(in_region) != 0;
  const int reg0 = any_region ? (ob.lo[2] > z0 ? ob.lo[2] : z0) : 0;
  const int reg1 = any_region ? (ob.lo[2] + ob.rn[2] < z1 ? ob.lo[2] + ob.rn[2] : z1) : 0;
  T v0[NW], v1[NW];  // this level's values
  // one cell of either level: collision, ends
  auto collide = [&](const int lv, const int z, T (&s)[19], const T d, T (&o)[5], T (&val)[NW]) {
    T drho, jx, jy, jz, omega, taue, p2[6];
    cell_moments<19, T>(s, drho, jx, jy, jz);
    const T rho = (T)1 + drho;
    const T ir = recip(rho);
    if (z == probe_z && z >= z0 && z < z1 && probe_lane) *pr.out[lv] = (double)(jy * ir);
    relaxation<19, T, HRR>(c, SMAG, s, drho, jx, jy, jz, ir, omega, taue, p2);
    if (ACC) {
      val[0] = drho;
      val[1] = jx;
      val[2] = jy;
      val[3] = jz;
      if (SMAG) val[NW - 1] = taue;
      if (__builtin_expect(z >= reg0 && z < reg1, 0) && wn.rec[lv] != nullptr && in_region)
        store_record<19, T>(wn.rec[lv],
                            (int64_t)(t.gx - ob.lo[0]) +
                                (int64_t)ob.rn[0] * ((t.gy - ob.lo[1]) + (int64_t)ob.rn[1] * (z - ob.lo[2])),
                            s, d);
    }
    collide_cell<19, T, HRR>(c, s, drho, jx, jy, jz, rho, ir, d, omega, p2);
    if (ENDS) {
      const T ux = jx * ir, uy = jy * ir, uz = jz * ir;
      const T uu = ux * ux + uy * uy + uz * uz;
      int n = 0;
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        if (L::cx[k] == -1) o[n++] = (T)to_store<S>(outlet_value<19, T>(k, ux, uy, uz, uu));
        if (L::cx[k] == 1) s[k] = t.inlet ? (k == 1 ? in1 : in4) : s[k];
      }
    }
  };
  Wait3<T> w;
  T cur[19], dcur, d1 = (T)0, wait[NW];  // wait: level 0's values of the last plane
  load(cur, dcur);
  int buf = 0;
  for (int z = z0 - 1; z <= z1; ++z) {
    T s[19], o[5];
#pragma unroll
    for (int k = 0; k < 19; ++k) s[k] = cur[k];
    T d0 = dcur;
    collide(0, z, s, d0, o, v0);
    __builtin_amdgcn_sched_barrier(0);
    load(cur, dcur);  // the next plane (past the last: in bounds, unused)
    double sum[NW];
    const uint64_t at8 = (uint64_t)g.nx * 8u * ((uint64_t)t.y + (uint64_t)g.ny * (uint64_t)(int64_t)(z - 1));
    if (ACC && z > z0 && t.own_row) {
#pragma unroll
      for (int a = 0; a < NW; ++a) sum[a] = *lane_ptr<const double>(sums[a] + at8, off8);
    }
    __builtin_amdgcn_sched_barrier(0);
    int n = 0;
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      s[k] = (T)to_store<S>(s[k]);
      // the lane beyond the outlet stands for the virtual column
      if (ENDS && L::cx[k] == -1) {
        const T v = lane_shift(o[n++], 1);
        s[k] = t.beyond ? v : s[k];
      }
    }
    T s1[19];
    hand_on3<R, WALLS, T>(g, t, z, lds + buf * (10 * R * 64), s, w, s1);
    buf ^= 1;
    if (z > z0 && t.own_row) {
      collide(1, z - 1, s1, d1, o, v1);
      if (ACC && adds) {
#pragma unroll
        for (int a = 0; a < NW; ++a)
          *lane_ptr<double>(sums[a] + at8, off8) = (sum[a] + (double)wait[a]) + (double)v1[a];
      }
      push3<ENDS, WALLS, true, S, T>(g, t, z - 1, B, offb, s1, o);
    }
    d1 = d0;
#pragma unroll
    for (int a = 0; a < NW; ++a) wait[a] = v0[a];
  }
}

// The tile and planes of a workgroup, and whether they hold an inlet or outlet
// column, a row or a plane beside a wall.
struct Tile3Id {
  int tx, ty, z0, z1;
  bool ends, walls;
};
template <int R>
__device__ __forceinline__ Tile3Id tile3_id(const Geo& g, const March3& m) {
  Tile3Id t;
  const int id = sweep_tile((int)blockIdx.x, (int)gridDim.x);
  const int per = m.tx * m.ty;
  const int chunk = wave_uniform(id / per), r = id - chunk * per;
  t.ty = wave_uniform(r / m.tx);
  t.tx = r - t.ty * m.tx;
  t.z0 = chunk * m.planes;
  t.z1 = t.z0 + m.planes < g.nz ? t.z0 + m.planes : g.nz;
  t.ends = g.bcx == BC_INOUT && (t.tx == 0 || t.tx * 62 + 62 >= g.nx - 1);
  t.walls = (g.bcy != BC_PERIODIC && (t.ty == 0 || (t.ty + 1) * (R - 2) >= g.ny)) ||
            (g.bcz != BC_PERIODIC && (t.z0 == 0 || t.z1 == g.nz));
  return t;
}

template <typename S, bool HRR, bool SMAG, bool ACC>
__device__ __forceinline__ void march3d_tile(const Geo& g, const MarchColl& mc, const March3& m,
                                             const S* __restrict__ A, S* __restrict__ B,
                                             const typename Prec<S>::Dd* __restrict__ dpor, const Probe& pr,
                                             const Window& wn) {
  using T = typename Prec<S>::T;
  constexpr int R = march3d_rows<T>();
  __shared__ T lds[2 * 10 * R * 64 + 2];
  const Coll c = mc.coll();
  const Tile3Id id = tile3_id<R>(g, m);
  const int tx = id.tx, ty = id.ty, z0 = id.z0, z1 = id.z1;
  if (id.walls) {
    if (id.ends)
      march3d<S, HRR, SMAG, true, true, ACC>(g, c, m, tx, ty, z0, z1, A, B, dpor, pr, wn, lds);
    else
      march3d<S, HRR, SMAG, false, true, ACC>(g, c, m, tx, ty, z0, z1, A, B, dpor, pr, wn, lds);
  } else {
    if (id.ends)
      march3d<S, HRR, SMAG, true, false, ACC>(g, c, m, tx, ty, z0, z1, A, B, dpor, pr, wn, lds);
    else
      march3d<S, HRR, SMAG, false, false, ACC>(g, c, m, tx, ty, z0, z1, A, B, dpor, pr, wn, lds);
  }
}

template <typename S, bool HRR, bool SMAG>
__global__ __launch_bounds__(64 * march3d_rows<typename Prec<S>::T>()) void k_march3d(
    const Geo g, const MarchColl mc, const March3 m, const S* __restrict__ A, S* __restrict__ B,
    const typename Prec<S>::Dd* __restrict__ dpor, const Probe pr) {
  const Window wn{};
  march3d_tile<S, HRR, SMAG, false>(g, mc, m, A, B, dpor, pr, wn);
}

// The same with the sums of a mean-flow window (BGK).
template <typename S, bool SMAG>
__global__ __launch_bounds__(64 * march3d_rows<typename Prec<S>::T>()) void k_window3d(
    const Geo g, const MarchColl mc, const March3 m, const S* __restrict__ A, S* __restrict__ B,
    const typename Prec<S>::Dd* __restrict__ dpor, const Probe pr, const Window wn) {
  march3d_tile<S, false, SMAG, true>(g, mc, m, A, B, dpor, pr, wn);
}

}  // namespace hlbm
