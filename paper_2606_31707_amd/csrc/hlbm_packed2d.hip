// hlbm_packed2d.hip -- packed launches that take two steps (or adjoint iterations)
// of every member in one pass over memory (D2Q9, BGK).
//
// A tick of small lattices is bound by the instructions of its slowest wavefronts
// (one to three a SIMD; loads two rows ahead changed nothing).  A pass takes two
// steps with one read and one write, and one launch holds the primal and the
// adjoint members.  One body serves all window members (closure, sums and
// objective terms by runtime flags), one the plain ones: bodies for strips
// without ends or walls as well outgrow the instruction cache and the registers
// (19.7 us a step instead of 16.5).  The three bodies fill 256 registers and spill
// (FP64 57, 216 bytes a lane; FP32 and FP16S 10, 44 bytes).  12 members of 128 x 64 to 512 x 256, FP32: single
// steps 27.1 us a step, passes 15.8.

#include "hlbm_march2d.hpp"

namespace hlbm {

namespace {
template <typename S>
__device__ __forceinline__ void packed_primal(const PackedPasses& p, const int b) {
  const PackedPrimal& P = ((const PackedPrimal*)p.primal.tab)[packed_member(p.primal.first, p.primal.nm, b)];
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
  const int flip = p.primal.flip;
  const S* A = (const S*)P.A[flip];
  S* B = (S*)P.A[flip ^ 1];
  const auto* dp = (const typename Prec<S>::Dd*)P.dpor;
  if (P.accumulate)
    march2d<S, 2, false, 2, 2, 3>(g, c, st, y0, y1, A, B, dp, pr, wn);
  else
    march2d<S, 2, false, 2, 2, 0>(g, c, st, y0, y1, A, B, dp, pr, wn);
}

template <typename T>
__device__ __forceinline__ void packed_adjoint(const PackedPasses& p, const int b) {
  const PackedAdjoint& P = ((const PackedAdjoint*)p.adjoint.tab)[packed_member(p.adjoint.first, p.adjoint.nm, b)];
  const int id = (b - P.first_pass) * 4 + wave_uniform((int)(threadIdx.x >> 6));
  const March2 m = P.march;
  if (id >= m.strips * m.chunks) return;
  const Geo g = P.g;
  const int chunk = wave_uniform(id / m.strips);
  const Strip st = make_strip<2>(g, id - chunk * m.strips);
  const int y0 = chunk * m.rows, y1 = y0 + m.rows < g.ny ? y0 + m.rows : g.ny;
  const MarchAdj ac{P.ac.les, P.ac.omega0};
  const int cur = (P.pvcur0 + p.pv) & 1, flip = p.adjoint.flip;
  march2d_adjoint<T, 2, true, 2>(g, P.ob, ac, st, y0, y1, (const T*)P.A[flip], (T*)P.A[flip ^ 1], (const T*)P.prep,
                                 P.src, P.oprep, (const T*)P.pv[cur], (T*)P.pv[cur ^ 1]);
}

template <typename S>
__global__ __launch_bounds__(256, 2) void k_packed2d(const PackedPasses p) {
  const int b = (int)blockIdx.x;
  if (b < p.primal.blocks)
    packed_primal<S>(p, b);
  else
    packed_adjoint<typename Prec<S>::T>(p, b - p.primal.blocks);
}
}  // namespace

bool packed_pass_member(const hlbm_lattice_s* L, int mode) {
  if (L->desc.stencil != HLBM_D2Q9 || L->desc.collision != HLBM_COLL_BGK) return false;
  const bool mea = L->obj_set && L->obj_kind == HLBM_OBJ_MEA;
  if (mode == HLBM_GROUP_ADJOINT) return L->phi2 != nullptr && !L->adj_diff && !mea;
  return L->f2 != nullptr && (mode == HLBM_GROUP_PRIMAL || (!L->desc.track_mean_populations && !mea));
}

// Rows per chunk: 4, or 3 where the wavefronts of all members are few (at most
// two workgroups a CU), so that each has less to do.  us a step with 3, 4, 7 and 12
// rows: 12 members of 128 x 64 to 512 x 256, FP32 16.5, 15.8, 15.9, 22.4, FP64 23.2, 21.8,
// 25.4, 35.4; 4 of them, FP32, 7.6, 8.6, 10.9, 16.0; 12 up to 200 x 100 7.0, 7.7, 10.6, 15.8.
void packed_pass_plan(hlbm_lattice_s* const* L, int count, March2* m) {
  int groups = 0;
  for (int i = 0; i < count; ++i) {
    m[i].strips = (L[i]->desc.nx + 61) / 62;
    groups += (m[i].strips * ((L[i]->desc.ny + 3) / 4) + 3) / 4;
  }
  for (int i = 0; i < count; ++i) {
    m[i].rows = groups > 512 ? 4 : 3;
    m[i].chunks = (L[i]->desc.ny + m[i].rows - 1) / m[i].rows;
  }
}

hipError_t launch_packed_pass(hipStream_t st, int precision, const PackedPasses& p) {
  const dim3 grid((unsigned)(p.primal.blocks + p.adjoint.blocks));
  switch (precision) {
    case HLBM_FP64: k_packed2d<double><<<grid, 256, 0, st>>>(p); break;
    case HLBM_FP32: k_packed2d<float><<<grid, 256, 0, st>>>(p); break;
    default: k_packed2d<_Float16><<<grid, 256, 0, st>>>(p); break;
  }
  return hipGetLastError();
}

}  // namespace hlbm
