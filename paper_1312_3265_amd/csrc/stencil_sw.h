// The staggered Wilson corner stencil's launches: groups of three and the split
// kernel.  Its instantiations, 24 unrolled terms each, are compiled one
// precision per file (k_stencil_sw_*.hip: 161 s in one file).
#pragma once

#include "stencil_dispatch.h"
#include "stencil_swsplit.h"

namespace lq {

// (16-bit, nine systems, 16^3 x 32, t = M p and the CG update: 70 + 79 us in
// pairs, 64 + 77 in threes)
template <class P, int NL, bool DAG>
constexpr bool kThirds<SWCornerOp<P, NL, DAG>> = true;

// Lattices of one-wavefront site blocks take the split kernel, with one system
// per thread.  The choice depends on the lattice alone, so a system's result
// depends neither on its batch nor on the launch configuration.
template <class P, int NL, bool DAG, int EPI>
struct OtherKernel<SWCornerOp<P, NL, DAG>, EPI> {
  using Op = SWCornerOp<P, NL, DAG>;
  static bool launch(const OpArgs& oa, const void* in, const EpiArgs& ea, int nrhs,
                     hipStream_t s) {
    if (block_of(oa.g.V) != 64 || nrhs < 1) return false;
    hipLaunchKernelGGL((sw_split_kernel<Op, EPI>), dim3(ea.nbp * nrhs), dim3(64 * Op::kGroups), 0,
                       s, oa, (const typename Op::S*)in, ea, nrhs);
    return true;
  }
};

void launch_stencil_sw_f64(int nl, bool dag, int epi, const OpArgs& oa, const void* in,
                           const EpiArgs& ea, int nrhs, hipStream_t s);
void launch_stencil_sw_f32(int nl, bool dag, int epi, const OpArgs& oa, const void* in,
                           const EpiArgs& ea, int nrhs, hipStream_t s);
void launch_stencil_sw_q16(int nl, bool dag, int epi, const OpArgs& oa, const void* in,
                           const EpiArgs& ea, int nrhs, hipStream_t s);

}  // namespace lq
