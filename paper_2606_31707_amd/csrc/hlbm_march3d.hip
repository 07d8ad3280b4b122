// hlbm_march3d.hip -- launcher of the D3Q19 two-step passes.
#include <cmath>

#include "hlbm_march3d.hpp"

namespace hlbm {

namespace {
template <typename S>
void march3d_pass(hlbm_lattice_s* L, bool window) {
  constexpr int R = march3d_rows<typename Prec<S>::T>();
  const double cs = L->desc.smagorinsky_cs;
  const MarchColl c{L->desc.tau, 1.0 / L->desc.tau, 18.0 * sqrt(2.0) * cs * cs};
  const March3 m = L->march3;
  const Probe pr = make_probe(L, 2);
  const Geo g = make_geo(L);
  const dim3 grid((unsigned)(m.tx * m.ty * m.chunks)), block(64 * R);
  const S* A = (const S*)L->f;
  S* B = (S*)L->f2;
  const auto* dp = (const typename Prec<S>::Dd*)L->dpor;
  if (window) {
    const Window wn = make_window(L);
    if (cs > 0.0)
      k_window3d<S, true><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr, wn);
    else
      k_window3d<S, false><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr, wn);
  } else if (L->desc.collision == HLBM_COLL_HRR) {
    if (cs > 0.0)
      k_march3d<S, true, true><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr);
    else
      k_march3d<S, true, false><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr);
  } else {
    if (cs > 0.0)
      k_march3d<S, false, true><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr);
    else
      k_march3d<S, false, false><<<grid, block, 0, L->stream>>>(g, c, m, A, B, dp, pr);
  }
}
}  // namespace

hipError_t launch_march3d(hlbm_lattice_s* L, bool window) {
  if (L->desc.precision == HLBM_FP64)
    march3d_pass<double>(L, window);
  else
    march3d_pass<float>(L, window);
  return hipGetLastError();
}

}  // namespace hlbm
