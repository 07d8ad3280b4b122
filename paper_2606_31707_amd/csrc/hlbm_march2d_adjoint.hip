// hlbm_march2d_adjoint.hip -- launcher of the D2Q9 multi-iteration adjoint
// passes.
#include <cmath>
#include <utility>

#include "hlbm_march2d.hpp"

namespace hlbm {

namespace {
template <typename T, int K>
void march2d_adjoint_pass(hlbm_lattice_s* L) {
  const March2 m = march2d_plan(L->desc, K);
  const MarchAdj ac{L->adj_les, L->adj_omega};
  const dim3 grid((unsigned)((m.strips * m.chunks + 3) / 4));
  k_march2d_adjoint<T, K><<<grid, 256, 0, L->stream>>>(make_geo(L), make_obj(L), ac, m, (const T*)L->phi,
                                                       (T*)L->phi2, (const T*)L->prep, L->src, L->oprep,
                                                       (const T*)L->pv[L->pvcur], (T*)L->pv[L->pvcur ^ 1]);
}
}  // namespace

int adjoint_pass_limit(const hlbm_lattice_s* L) {
  const bool small = region_copy_used((int64_t)L->rn[0] * L->rn[1] * L->rn[2], L->n, L->obj_kind);
  return pass_limit(L->desc, small ? PASS_ADJOINT : PASS_ADJOINT_LARGE, L->march3);
}

hipError_t launch_adjoint_pass(hlbm_lattice_s* L, int K) {
  if (L->desc.stencil == HLBM_D3Q19) return K == 2 ? launch_march3d_adjoint(L) : hipErrorInvalidValue;
  const bool f64 = L->desc.precision == HLBM_FP64;
  if (K == 4) {
    if (f64) march2d_adjoint_pass<double, 4>(L); else march2d_adjoint_pass<float, 4>(L);
  } else if (K == 2) {
    if (f64) march2d_adjoint_pass<double, 2>(L); else march2d_adjoint_pass<float, 2>(L);
  } else {
    return hipErrorInvalidValue;
  }
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) std::swap(L->phi, L->phi2);
  return e;
}

}  // namespace hlbm
