// hlbm_march2d.hip -- launchers of the D2Q9 multi-step passes.
#include <cmath>
#include <utility>

#include "hlbm_march2d.hpp"

namespace hlbm {

Probe make_probe(const hlbm_lattice_s* L, int K) {
  Probe pr{{nullptr, nullptr, nullptr, nullptr}, 0, 0, 0};
  if (L->probe_buf != nullptr && L->probe_cap > 0) {
    const int64_t nx = L->desc.nx, ny = L->desc.ny;
    for (int i = 0; i < K; ++i) pr.out[i] = L->probe_buf + (L->probe_n + i) % L->probe_cap;
    pr.x = (int)(L->probe_cell % nx);
    pr.y = (int)(L->probe_cell / nx % ny);
    pr.z = (int)(L->probe_cell / (nx * ny));
  }
  return pr;
}

namespace {
template <typename S, int K>
void march2d(hlbm_lattice_s* L) {
  const Geo g = make_geo(L);
  const double cs = L->desc.smagorinsky_cs;
  const MarchColl c{L->desc.tau, 1.0 / L->desc.tau, 18.0 * sqrt(2.0) * cs * cs};
  const March2 m = march2d_plan(L->desc, K);
  const Probe pr = make_probe(L, K);
  const dim3 grid((unsigned)((m.strips * m.chunks + 3) / 4));
  const S* A = (const S*)L->f;
  S* B = (S*)L->f2;
  const auto* dp = (const typename Prec<S>::Dd*)L->dpor;
  const bool hrr = L->desc.collision == HLBM_COLL_HRR, smag = cs > 0.0;
  if (hrr) {
    if (smag)
      k_march2d<S, K, true, true><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr);
    else
      k_march2d<S, K, true, false><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr);
  } else {
    if (smag)
      k_march2d<S, K, false, true><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr);
    else
      k_march2d<S, K, false, false><<<grid, 256, 0, L->stream>>>(g, c, m, A, B, dp, pr);
  }
}
}  // namespace

int primal_pass_limit(const hlbm_lattice_s* L, int accumulate) {
  return accumulate ? window_pass_limit(L) : pass_limit(L->desc, PASS_PLAIN, L->march3);
}

hipError_t launch_primal_pass(hlbm_lattice_s* L, int accumulate, int K) {
  if (accumulate) return launch_window_pass(L, K);
  hipError_t e = hipSuccess;
  if (L->desc.stencil == HLBM_D3Q19) {
    if (K != 2) return hipErrorInvalidValue;
    e = launch_march3d(L, false);
    if (e == hipSuccess) std::swap(L->f, L->f2);
    return e;
  }
  switch (L->desc.precision * 8 + K) {
    case 0 + 2: march2d<double, 2>(L); break;
    case 0 + 4: march2d<double, 4>(L); break;
    case 8 + 2: march2d<float, 2>(L); break;
    case 8 + 4: march2d<float, 4>(L); break;
    case 16 + 2: march2d<_Float16, 2>(L); break;
    case 16 + 4: march2d<_Float16, 4>(L); break;
    default: return hipErrorInvalidValue;
  }
  e = hipGetLastError();
  if (e == hipSuccess) std::swap(L->f, L->f2);
  return e;
}

}  // namespace hlbm
