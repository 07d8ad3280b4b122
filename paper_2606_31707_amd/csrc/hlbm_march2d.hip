// hlbm_march2d.hip -- launchers of the D2Q9 multi-step passes.
#include <cmath>
#include <utility>

#include "hlbm_march2d.hpp"

namespace hlbm {

// Rows per chunk: the number of iterations (rows plus the halo of the levels)
// times what an iteration costs with m workgroups on a compute unit.  Measured
// on 1100 x 410: a second wavefront on a SIMD adds 45 % to an iteration in
// FP64 and 9 % in FP32 (latency left by one is filled by the other), each
// further one 40 %.  Long chunks stop paying on lattices larger than the
// caches, where neighbouring chunks share their halo rows in L2
// (8192 x 4096 FP32: 8 rows 167 us, 16 rows 169, 58 rows 184; FP16S, whose
// rows are half as long, 150, 117 and 110).
March2 march2d_plan(const hlbm_lattice_s* L, int K, bool f64) {
  const int W = 64 - 2 * (K - 1), ny = L->desc.ny;
  March2 m;
  m.strips = (L->desc.nx + W - 1) / W;
  const int most = L->desc.precision == HLBM_FP16S ? 24 : 12;
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
  const March2 m = march2d_plan(L, K, sizeof(S) == 8);
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

// Four steps a pass; two for FP16 lattices that stay in the caches, whose
// loads and conversions rather than bytes bound a pass (1100 x 410: 4.6 us a
// step with two, 5.0 with four; 8192 x 4096: 172 and 110).
int primal_pass_limit(const hlbm_lattice_s* L, int accumulate) {
  if (accumulate) return window_pass_limit(L);
  if (L->desc.stencil == HLBM_D3Q19) return passes_pay_3d(L->desc, PASS_PLAIN, L->march3) ? 2 : 1;
  return HLBM_PASS_RULES && L->desc.precision == HLBM_FP16S && !L->large ? 2 : 4;
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
