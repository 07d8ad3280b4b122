// hlbm_march3d_adjoint.hip -- D3Q19 adjoint: two iterations in one pass over memory
// (BGK, frozen relaxation time, moment-form objectives).
//
// What bounds it: instructions (a level of the adjoint and its share of the
// scalar registers' spills, 362 in FP64, take 600 in FP32, twice the primal's), so
// that it pays only where single iterations are bound by FP64 traffic from HBM.
// The tiles of the primal passes (hlbm_march3d.hpp): phihat streams as the
// populations do.  The frozen data of a plane waits one plane in registers for
// level 1; the source of the objective's region is read at each level.  Nothing
// arrives at the outlet from beyond; what leaves through it arrives on the lane
// beyond and enters level 1's virtual-column term from there (level 0 and the
// last level: the pv buffers).
#include <cmath>
#include <utility>

#include "hlbm_march3d.hpp"

namespace hlbm {

namespace {
template <typename T>
struct Frozen3 {
  T tx, ty, tz, d, om;
};

template <typename T, bool ENDS, bool WALLS>
__device__ __forceinline__ void march3d_adjoint(const Geo& g, const ObjBox& ob, const MarchAdj& ac, const int tx,
                                                const int ty, const int z0, const int z1, const T* __restrict__ A,
                                                T* __restrict__ B, const T* __restrict__ prep,
                                                const double* __restrict__ src, const double* __restrict__ oprep,
                                                const T* __restrict__ pv_in, T* __restrict__ pv_out,
                                                T* __restrict__ lds) {
  using L = Lat<19>;
  constexpr int R = march3d_rows<T>();
  const Tile3 t = make_tile3<R>(g, tx, ty);
  const uint64_t pstep = uni64((uint64_t)g.plane * sizeof(T));
  const uint32_t off = lane_offset((uint32_t)t.x * (uint32_t)sizeof(T));
  const uint32_t offb[3] = {lane_offset((uint32_t)t.xm * (uint32_t)sizeof(T)), off,
                            lane_offset((uint32_t)t.xp * (uint32_t)sizeof(T))};
  RowPtr pa(A, z0 - 1, g.nx * g.ny, g.nz, (int)sizeof(T)), pp(prep, z0 - 1, g.nx * g.ny, g.nz, (int)sizeof(T));
  pa.base += (uint64_t)t.y * (uint64_t)g.nx * sizeof(T);
  pp.base += (uint64_t)t.y * (uint64_t)g.nx * sizeof(T);
  auto load = [&](T (&s)[19], Frozen3<T>& f) {
    uint64_t pb = pa.base;
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      s[k] = *lane_ptr<const T>(pb, off);
      pb += pstep;
      asm("" : "+s"(pb));
    }
    f.tx = *lane_ptr<const T>(pp.base, off);
    f.ty = *lane_ptr<const T>(pp.base + pstep, off);
    f.tz = *lane_ptr<const T>(pp.base + 2 * pstep, off);
    f.d = *lane_ptr<const T>(pp.base + 3 * pstep, off);
    f.om = *lane_ptr<const T>(pp.base + (ac.les ? 4 : 3) * pstep, off);
    pa.next();
    pp.next();
  };
  // (also without WALLS: the halo may hold a row or plane beside a wall)
  const bool ywall = g.bcy != BC_PERIODIC, zwall = g.bcz != BC_PERIODIC;
  const bool in_region = ob.active && t.x >= ob.lo[0] && t.x < ob.lo[0] + ob.rn[0] && t.y >= ob.lo[1] &&
                         t.y < ob.lo[1] + ob.rn[1];
  const bool any_region = __ballot(in_region) != 0;
  // one iteration of the cells of plane z: c gets the post-collision values in
  // direction order, lam those of the outlet's virtual column
  auto level = [&](const int lv, const int z, T (&s)[19], const Frozen3<T>& f, T (&c)[19], T (&lam)[19]) {
    const int zz = z < 0 ? z + g.nz : (z >= g.nz ? z - g.nz : z);
    T pv[19];
    if (ENDS) {
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        if (L::cx[k] != -1) continue;
        if (lv == 0) {
          pv[k] = pv_in[k * g.gplane + t.y + (int64_t)g.ny * zz];
        } else {
          pv[k] = lane_shift(s[L::opp[k]], -1);
          const bool beyond = (ywall && ((L::cy[k] < 0 && t.y == 0) || (L::cy[k] > 0 && t.y == g.ny - 1))) ||
                              (zwall && ((L::cz[k] < 0 && zz == 0) || (L::cz[k] > 0 && zz == g.nz - 1)));
          pv[k] = beyond ? (T)0 : pv[k];
        }
      }
      // beyond the outlet: no adjoint inflow (a wall's bounce-back stays)
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        if (L::cx[k] != -1) continue;
        const bool kept = (ywall && ((L::cy[k] > 0 && t.y == 0) || (L::cy[k] < 0 && t.y == g.ny - 1))) ||
                          (zwall && ((L::cz[k] > 0 && zz == 0) || (L::cz[k] < 0 && zz == g.nz - 1)));
        s[k] = t.outlet && !kept ? (T)0 : s[k];
      }
    }
    adjoint_bgk<19, T>(s, f.tx, f.ty, f.tz, f.d, ac.les ? f.om : (T)ac.omega0, lam);
    if (ENDS) {
      const int64_t o = t.y + (int64_t)g.ny * zz;
      T lo[19];
#pragma unroll
      for (int k = 0; k < 19; ++k) lo[k] = lam[k];
      adjoint_outlet<19, T>(pv, (T)1 / (T)oprep[o], (T)oprep[g.gplane + o], (T)oprep[2 * g.gplane + o],
                            (T)oprep[3 * g.gplane + o], lo);
#pragma unroll
      for (int k = 0; k < 19; ++k) lam[k] = t.outlet ? lo[k] : lam[k];
    }
    if (any_region && zz >= ob.lo[2] && zz < ob.lo[2] + ob.rn[2]) {
      constexpr int N = 1 + L::D + L::NSYM;
      T q[N];
#pragma unroll
      for (int m = 0; m < N; ++m) q[m] = (T)0;
      if (in_region) {
        const int64_t r = (int64_t)(t.x - ob.lo[0]) +
                          (int64_t)ob.rn[0] * ((t.y - ob.lo[1]) + (int64_t)ob.rn[1] * (zz - ob.lo[2]));
#pragma unroll
        for (int m = 0; m < N; ++m) q[m] = (T)src[(Coef<19>::A0 + m) * ob.rplane + r];
      }
#pragma unroll
      for (int i = 0; i < 19; ++i) lam[i] -= quad_eval<19, T>(q, i);
    }
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      c[k] = lam[L::opp[k]];
      if (ENDS && L::cx[k] == 1) c[k] = t.inlet ? (T)0 : c[k];  // lambda = 0 at the pinned inlet
    }
  };
  Wait3<T> w;
  T cur[19];
  Frozen3<T> fcur, f1;
  load(cur, fcur);
  f1 = fcur;
  int buf = 0;
  for (int z = z0 - 1; z <= z1; ++z) {
    T s[19], c[19], lam[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) s[k] = cur[k];
    const Frozen3<T> f0 = fcur;
    level(0, z, s, f0, c, lam);
    __builtin_amdgcn_sched_barrier(0);
    load(cur, fcur);  // the next plane (past the last: in bounds, unused)
    __builtin_amdgcn_sched_barrier(0);
    T s1[19];
    hand_on3<R, WALLS, T>(g, t, z, lds + buf * (10 * R * 64), c, w, s1);
    buf ^= 1;
    if (z > z0 && t.own_row) {
      level(1, z - 1, s1, f1, c, lam);
      const T o[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
      push3<ENDS, WALLS, false, T, T>(g, t, z - 1, B, offb, c, o);
      if (ENDS && t.own && t.outlet) {
#pragma unroll
        for (int k = 0; k < 19; ++k) {
          if (L::cx[k] != -1) continue;
          int vy = t.y - L::cy[k], vz = z - 1 - L::cz[k];
          const bool cell = !((ywall && (vy < 0 || vy >= g.ny)) || (zwall && (vz < 0 || vz >= g.nz)));
          vy = vy < 0 ? vy + g.ny : (vy >= g.ny ? vy - g.ny : vy);
          vz = vz < 0 ? vz + g.nz : (vz >= g.nz ? vz - g.nz : vz);
          if (cell) pv_out[k * g.gplane + vy + (int64_t)g.ny * vz] = lam[k];
        }
      }
    }
    f1 = f0;
  }
}

template <typename T>
__global__ __launch_bounds__(64 * march3d_rows<T>()) void k_march3d_adjoint(
    const Geo g, const ObjBox ob, const MarchAdj ac, const March3 m, const T* __restrict__ A, T* __restrict__ B,
    const T* __restrict__ prep, const double* __restrict__ src, const double* __restrict__ oprep,
    const T* __restrict__ pv_in, T* __restrict__ pv_out) {
  constexpr int R = march3d_rows<T>();
  __shared__ T lds[2 * 10 * R * 64 + 2];
  const Tile3Id id = tile3_id<R>(g, m);
  if (id.walls) {
    if (id.ends)
      march3d_adjoint<T, true, true>(g, ob, ac, id.tx, id.ty, id.z0, id.z1, A, B, prep, src, oprep, pv_in, pv_out, lds);
    else
      march3d_adjoint<T, false, true>(g, ob, ac, id.tx, id.ty, id.z0, id.z1, A, B, prep, src, oprep, pv_in, pv_out, lds);
  } else {
    if (id.ends)
      march3d_adjoint<T, true, false>(g, ob, ac, id.tx, id.ty, id.z0, id.z1, A, B, prep, src, oprep, pv_in, pv_out, lds);
    else
      march3d_adjoint<T, false, false>(g, ob, ac, id.tx, id.ty, id.z0, id.z1, A, B, prep, src, oprep, pv_in, pv_out, lds);
  }
}

}  // namespace

hipError_t launch_march3d_adjoint(hlbm_lattice_s* L) {
  constexpr int R = march3d_rows<double>();
  const March3 m = L->march3;
  const MarchAdj ac{L->adj_les, L->adj_omega};
  k_march3d_adjoint<double><<<dim3((unsigned)(m.tx * m.ty * m.chunks)), dim3(64 * R), 0, L->stream>>>(
      make_geo(L), make_obj(L), ac, m, (const double*)L->phi, (double*)L->phi2, (const double*)L->prep, L->src,
      L->oprep, (const double*)L->pv[L->pvcur], (double*)L->pv[L->pvcur ^ 1]);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) std::swap(L->phi, L->phi2);
  return e;
}

}  // namespace hlbm
