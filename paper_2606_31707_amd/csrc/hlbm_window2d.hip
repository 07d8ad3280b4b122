// hlbm_window2d.hip -- mean-flow windows in multi-step passes: which steps take
// them, the D2Q9 launcher, the objective terms of a small region.
#include <cmath>
#include <utility>

#include "hlbm_march2d.hpp"

namespace hlbm {

// Window steps of a pass (pass_limit).  Single steps remain for the HRR
// collision and tracked mean populations (q more sums per cell, more than the
// pass saves), J_MEA (terms of its own) and large regions in 3D, whose FP64
// terms do not fit beside two levels' state.
// us a step, single steps / passes: 1100 x 410 FP32 9.5 / 5.0, with a drag plane
// 13.0 / 7.0, with a dissipation box 12.2 / 9.1, FP64 15.1 / 9.6; 8192 x 4096
// FP32 608 / 248, FP16S 413 / 199; 768x384x128 FP32 with closure 1462 / 1390;
// 756x168x84 FP64 881 / 523.
int window_pass_limit(const hlbm_lattice_s* L) {
  const hlbm_desc& d = L->desc;
  if (d.collision != HLBM_COLL_BGK || d.track_mean_populations) return 1;
  PassKind kind = PASS_WINDOW;
  if (L->obj_set) {
    if (L->obj_kind == HLBM_OBJ_MEA) return 1;
    if (!L->rcopy) {
      if (d.stencil == HLBM_D3Q19) return 1;
      kind = PASS_WINDOW_LARGE;
    } else {
      // the pending slots hold the records of the later levels
      if (d.precision != HLBM_FP64 && L->rplane * region_copy_stride(L->q, (int)L->asize) > pend_slot_elems(L)) return 1;
      kind = PASS_WINDOW_REGION;
    }
  }
  return pass_limit(d, kind, L->march3);
}

// Level 0's records go to the region copy, those of the later levels to the
// pending slots of the grouped accumulation, which are empty between groups.
// FP64 lattices have no such slots: the first step's records of a region of
// up to one cross-section go to rcopy2 (192x96x64 with a drag plane 67 us a
// step, 81 without), a larger region's terms of that step are taken from the
// state the pass starts from.
Window make_window(const hlbm_lattice_s* L) {
  Window w{};
  w.rho = L->acc_rho;
  w.j = L->acc_j;
  w.tau = L->acc_tau;
  w.ob = make_obj(L);
  w.obj = L->acc_obj;
  if (L->obj_set && L->rcopy) {
    if (L->desc.precision == HLBM_FP64) {
      w.rec[1] = L->rcopy;
      if (L->rplane <= L->gplane) w.rec[0] = L->rcopy2;
    } else {
      w.rec[0] = L->rcopy;
      for (int t = 1; t < PEND_GROUP; ++t) w.rec[t] = L->acc_pend + (t - 1) * pend_slot_elems(L);
    }
  }
  return w;
}

namespace {
template <typename S, int K, bool LARGE>
void window2d(hlbm_lattice_s* L) {
  const Geo g = make_geo(L);
  const double cs = L->desc.smagorinsky_cs;
  const MarchColl c{L->desc.tau, 1.0 / L->desc.tau, 18.0 * sqrt(2.0) * cs * cs};
  const March2 m = march2d_plan(L->desc, K);
  const Probe pr = make_probe(L, K);
  const Window wn = make_window(L);
  const dim3 grid((unsigned)((m.strips * m.chunks + 3) / 4));
  const S* A = (const S*)L->f;
  S* B = (S*)L->f2;
  const auto* dp = (const typename Prec<S>::Dd*)L->dpor;
  if (cs > 0.0)
    k_window2d<S, K, true, LARGE><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr, wn);
  else
    k_window2d<S, K, false, LARGE><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr, wn);
}
}  // namespace

hipError_t launch_window2d(hlbm_lattice_s* L, int K) {
  const bool large = L->obj_set && !L->rcopy;
  switch ((L->desc.precision * 8 + K) * 2 + (large ? 1 : 0)) {
    case 2 * 2: window2d<double, 2, false>(L); break;
    case 2 * 2 + 1: window2d<double, 2, true>(L); break;
    case 10 * 2: window2d<float, 2, false>(L); break;
    case 10 * 2 + 1: window2d<float, 2, true>(L); break;
    case 12 * 2: window2d<float, 4, false>(L); break;
    case 12 * 2 + 1: window2d<float, 4, true>(L); break;
    case 20 * 2 + 1: window2d<_Float16, 4, true>(L); break;
    case 18 * 2: window2d<_Float16, 2, false>(L); break;
    case 18 * 2 + 1: window2d<_Float16, 2, true>(L); break;
    case 20 * 2: window2d<_Float16, 4, false>(L); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_window_pass(hlbm_lattice_s* L, int K) {
  const bool small = L->obj_set && L->rcopy;
  hipError_t e = hipSuccess;
  const Window w = make_window(L);
  if (small && w.rec[0] == nullptr && (e = launch_region_state(L)) != hipSuccess) return e;
  e = L->desc.stencil == HLBM_D3Q19 ? launch_march3d(L, true) : launch_window2d(L, K);
  if (e != hipSuccess) return e;
  std::swap(L->f, L->f2);
  if (!small) return e;
  Records rc{};
  for (int t = 0; t < K; ++t)
    if (w.rec[t]) rc.rec[rc.n++] = w.rec[t];
  return launch_region_records(L, rc);
}

}  // namespace hlbm
