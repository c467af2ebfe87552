// Stencil kernel instantiations for SWCornerOp, FP64.
#include "stencil_sw.h"

namespace lq {
void launch_stencil_sw_f64(int nl, bool dag, int epi, const OpArgs& oa, const void* in,
                           const EpiArgs& ea, int nrhs, hipStream_t s) {
  dispatch_links<SWCornerOp, F64>(nl, dag, epi, oa, in, ea, nrhs, s);
}
}  // namespace lq
