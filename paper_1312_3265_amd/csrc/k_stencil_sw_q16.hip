// Stencil kernel instantiations for SWCornerOp, 16-bit.
#include "stencil_sw.h"

namespace lq {
void launch_stencil_sw_q16(int nl, bool dag, int epi, const OpArgs& oa, const void* in,
                           const EpiArgs& ea, int nrhs, hipStream_t s) {
  dispatch_links<SWCornerOp, Q16>(nl, dag, epi, oa, in, ea, nrhs, s);
}
}  // namespace lq
