// The staggered Wilson corner stencil: its precisions are in k_stencil_sw_*.hip.
#include "stencil_sw.h"

namespace lq {
void launch_stencil_sw(int prec, int nl, bool dag, int epi, const OpArgs& oa, const void* in,
          const EpiArgs& ea, int nrhs, hipStream_t s) {
  if (prec == P64) return launch_stencil_sw_f64(nl, dag, epi, oa, in, ea, nrhs, s);
  if (prec == P32) return launch_stencil_sw_f32(nl, dag, epi, oa, in, ea, nrhs, s);
  if (prec == P16) return launch_stencil_sw_q16(nl, dag, epi, oa, in, ea, nrhs, s);
  unsupported_storage(prec, nl);
}
}  // namespace lq
