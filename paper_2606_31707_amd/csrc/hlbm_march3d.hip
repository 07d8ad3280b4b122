// hlbm_march3d.hip -- launcher of the D3Q19 two-step passes.
#include <cmath>

#include "hlbm_march3d.hpp"

namespace hlbm {

March3 march3d_plan(const hlbm_lattice_s* L, int R) {
  March3 m;
  m.tx = (L->desc.nx + 61) / 62;
  m.ty = (L->desc.ny + R - 3) / (R - 2);
  const int tiles = m.tx * m.ty, nz = L->desc.nz;
  double best = 0.0;
  for (int chunks = 1; chunks <= nz; ++chunks) {
    const int planes = (nz + chunks - 1) / chunks;
    const int64_t rounds = ((int64_t)tiles * ((nz + planes - 1) / planes) + 255) / 256;
    const double cost = (double)rounds * (planes + 3.0);
    if (chunks == 1 || cost < best) {
      best = cost;
      m.planes = planes;
    }
  }
  m.chunks = (nz + m.planes - 1) / m.planes;
  return m;
}

namespace {
template <typename S>
void march3d_pass(hlbm_lattice_s* L, bool window) {
  constexpr int R = march3d_rows<typename Prec<S>::T>();
  const double cs = L->desc.smagorinsky_cs;
  const MarchColl c{L->desc.tau, 1.0 / L->desc.tau, 18.0 * sqrt(2.0) * cs * cs};
  const March3 m = march3d_plan(L, R);
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
