// Answers for lattices on standard input, one a line, whether they take multi-step passes
// (csrc/hlbm_pass_rules.hpp): stencil precision nx ny nz bc_x bc_y bc_z collision closure kind
// -> bytes of optional arrays, steps that a pass of that kind (PassKind) takes at most (1: none).
// A line with nz = 0 asks for a packed list: precision, kind, nx = with_other, ny = blocks.
#include <cstdio>
#include <cstring>

#include "hlbm_pass_rules.hpp"

int main() {
  using namespace hlbm;
  hlbm_desc d;
  int kind;
  std::memset(&d, 0, sizeof d);
  d.struct_size = sizeof d;
  d.tau = 0.56;
  d.inlet_profile = HLBM_INLET_PARABOLIC;
  d.u_in = 0.04;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %lf %d", &d.stencil, &d.precision, &d.nx, &d.ny, &d.nz, &d.bc_x, &d.bc_y,
                    &d.bc_z, &d.collision, &d.smagorinsky_cs, &kind) == 11) {
    if (d.nz == 0) {
      std::printf("0 %d\n", (int)packed_passes_pay(d.precision, (PassKind)kind, d.nx != 0, d.ny));
      continue;
    }
    if (desc_problem(&d)) return std::printf("bad descriptor: %s\n", desc_problem(&d)), 1;
    const March3 m = march3d_plan(d, march3d_rows_of(d.precision == HLBM_FP64));
    const bool adjoint = kind == PASS_ADJOINT || kind == PASS_ADJOINT_LARGE;
    std::printf("%llu %d\n", (unsigned long long)(adjoint ? pass_bytes_adjoint(&d) : pass_bytes_primal(&d)),
                pass_limit(d, (PassKind)kind, m));
  }
  return 0;
}
