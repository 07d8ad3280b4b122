// hlbm_packed2d.hip -- packed launches that take two steps (or adjoint iterations)
// of every member in one pass over memory (D2Q9, BGK).
//
// A tick of small lattices is bound by latency: every launch waits for its
// slowest wavefront's chain of loads, collisions and stores.  One pass does
// two steps with one such chain, of the rows of a chunk; the rows are chosen
// for the wavefronts of all members together.  One kernel body serves plain
// and window members (closure, sums and objective terms by runtime flags): the
// strips that hold an inlet, an outlet or walls take longest in lattices of a
// few strips, so that faster bodies for the others would save nothing.
#include <cmath>
#include <vector>

#include "hlbm_march2d.hpp"

namespace hlbm {

namespace {
template <typename S>
__global__ __launch_bounds__(256, 2) void k_primal_packed2d(const PackedPrimal* __restrict__ tab,
                                                            const int* __restrict__ first, int nm, int flip) {
  const int b = (int)blockIdx.x;
  const PackedPrimal& P = tab[packed_member(first, nm, b)];
  const int id = (b - P.first_pass) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  const March2 m = P.march;
  if (id >= m.strips * m.chunks) return;
  const Geo g = P.g;
  const Coll c = P.c;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<2>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  Window wn{};
  if (P.accumulate) {
    wn.rho = P.acc.rho;
    wn.j = P.acc.j;
    wn.tau = P.acc.tau;
    wn.ob = P.ob;
    wn.obj = P.acc.obj;
  }
  const Probe pr{{nullptr, nullptr, nullptr, nullptr}, 0, 0, 0};
  march2d<S, 2, false, 2, 2, 3>(g, c, st, y0, y1, (const S*)P.A[flip], (S*)P.A[flip ^ 1],
                                (const typename Prec<S>::Dd*)P.dpor, pr, wn);
}

template <typename T>
__global__ __launch_bounds__(256, 2) void k_adjoint_packed2d(const PackedAdjoint* __restrict__ tab,
                                                             const int* __restrict__ first, int nm, int flip,
                                                             int pv) {
  const int b = (int)blockIdx.x;
  const PackedAdjoint& P = tab[packed_member(first, nm, b)];
  const int id = (b - P.first_pass) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  const March2 m = P.march;
  if (id >= m.strips * m.chunks) return;
  const Geo g = P.g;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<2>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  const MarchAdj ac{P.ac.les, P.ac.omega0};
  const int cur = (P.pvcur0 + pv) & 1;
  march2d_adjoint<T, 2, true, 2>(g, P.ob, ac, st, y0, y1, (const T*)P.A[flip], (T*)P.A[flip ^ 1],
                                 (const T*)P.prep, P.src, P.oprep, (const T*)P.pv[cur], (T*)P.pv[cur ^ 1]);
}
}  // namespace

bool packed_pass_member(const hlbm_lattice_s* L, int mode) {
  if (L->desc.stencil != HLBM_D2Q9 || L->desc.collision != HLBM_COLL_BGK) return false;
  const bool mea = L->obj_set && L->obj_kind == HLBM_OBJ_MEA;
  if (mode == HLBM_GROUP_ADJOINT) return L->phi2 != nullptr && !L->adj_diff && !mea;
  return L->f2 != nullptr && (mode == HLBM_GROUP_PRIMAL || (!L->desc.track_mean_populations && !mea));
}

int packed_pass_plan(hlbm_lattice_s* const* L, int count, March2* m) {
  if (count == 0) return 0;
  std::vector<int> strips(count), ny(count);
  for (int i = 0; i < count; ++i) {
    strips[i] = (L[i]->desc.nx + 61) / 62;
    ny[i] = L[i]->desc.ny;
  }
  const int rows = march2d_rows(strips.data(), ny.data(), count, 2, L[0]->desc.precision == HLBM_FP64, 12);
  int blocks = 0;
  for (int i = 0; i < count; ++i) {
    m[i].strips = strips[i];
    m[i].rows = rows;
    m[i].chunks = (ny[i] + rows - 1) / rows;
    blocks += (m[i].strips * m[i].chunks + 3) / 4;
  }
  return blocks;
}

hipError_t launch_primal_packed_pass(hipStream_t st, int precision, const void* tab, const int* first, int nm,
                                     int blocks, int flip) {
  const PackedPrimal* t = (const PackedPrimal*)tab;
  const dim3 grid((unsigned)blocks);
  switch (precision) {
    case HLBM_FP64: k_primal_packed2d<double><<<grid, 256, 0, st>>>(t, first, nm, flip); break;
    case HLBM_FP32: k_primal_packed2d<float><<<grid, 256, 0, st>>>(t, first, nm, flip); break;
    default: k_primal_packed2d<_Float16><<<grid, 256, 0, st>>>(t, first, nm, flip); break;
  }
  return hipGetLastError();
}

hipError_t launch_adjoint_packed_pass(hipStream_t st, int precision, const void* tab, const int* first, int nm,
                                      int blocks, int flip, int pv) {
  const PackedAdjoint* t = (const PackedAdjoint*)tab;
  const dim3 grid((unsigned)blocks);
  if (precision == HLBM_FP64)
    k_adjoint_packed2d<double><<<grid, 256, 0, st>>>(t, first, nm, flip, pv);
  else
    k_adjoint_packed2d<float><<<grid, 256, 0, st>>>(t, first, nm, flip, pv);
  return hipGetLastError();
}

}  // namespace hlbm
