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

// The split kernel (one system per thread) where sw_split_fits the systems that
// are active (a pool of nine on 8^2 x 16^2, 16-bit, one slot running: 5.3 ms per
// solve, 6.4 by the number of slots).
template <class P, int NL, bool DAG, int EPI>
struct OtherKernel<SWCornerOp<P, NL, DAG>, EPI> {
  using Op = SWCornerOp<P, NL, DAG>;
  static bool launch(const OpArgs& oa, const void* in, const EpiArgs& ea, int nrhs,
                     hipStream_t s) {
    const int active = ea.active > 0 && ea.active < nrhs ? ea.active : nrhs;
    if (nrhs < 1 || !sw_split_fits(P::id, oa.g.V, active)) return false;
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
