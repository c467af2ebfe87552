// Staggered Wilson stencil (corner form) with a site's 24 terms split over the
// wavefronts of a block: eight wavefronts cover the same 64 sites, wavefront r
// taking the three terms of group r of SWCornerOp.  The terms meet in LDS and
// are added there in the order of the one-thread form, so the result is the
// same to the bit; wavefront 0 runs the epilogue.
//
// For launches that leave the chip idle (sw_split_fits): with one thread per
// site a system of 8^3 x 16 has 128 wavefronts on 1024 SIMDs, and each waits
// for its 24 matrices one after another.  FP64 t = M p, one system, against
// the one-thread kernel in blocks of 256 before its loads were grouped: 4^4
// 19 -> 6 us, 8^3 x 16 22 -> 6, 8^2 x 16^2 27 -> 7.
#pragma once

#include "stencil.h"

namespace lq {

template <class Op, int EPI>
__global__ void __launch_bounds__(64 * Op::kGroups)
__attribute__((amdgpu_waves_per_eu(4, 8)))
sw_split_kernel(const OpArgs oa, const typename Op::S* __restrict__ in, const EpiArgs ea,
                int nrhs) {
  using C = typename Op::C;
  __shared__ C terms[3 * Op::kGroups][3][64];
  int sb, kl;
  map_block(ea.nbp, nrhs, ea.window < -2 ? 0 : ea.window, sb, kl);
  const int k = ea.k0 + kl;
  if (ea.st && !slot_active(ea.st, k, ea.state_mode, ea.par, ea.ru_mask)) return;   // uniform
  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = sb * 64 + lane;
  const bool valid = i < oa.g.V;
  const typename Op::S* f = in + (size_t)k * field_planes<typename Op::Pol>(3) * oa.g.Vp;

  double alpha = 0.0;
  if constexpr (EPI == EPI_CG_UPDATE) {
    if (r == 0) {
      const double tt = wave_partials(ea.part_in + (size_t)k * ea.nbp, ea.nbp, 4);
      const double rho = ea.st[k].rho[ea.par];
      alpha = (tt > 0.0 && isfinite(tt) && isfinite(rho)) ? rho / tt : 0.0;
      if (sb == 0 && lane == 0) {
        if (!(tt > 0.0 && isfinite(tt))) ea.st[k].flags |= 1;
        ea.st[k].alpha[ea.q4] = alpha;   // read on the group's last iteration
      }
    }
  }

  if (valid) {
    const SWSite n = sw_site(oa.g, i);
    C y[3][3];
    Op::group_terms(oa, f, n, i, r, y);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int q = 0; q < 3; ++q) terms[3 * r + t][q][lane] = y[t][q];
  }
  __syncthreads();
  // one colour per wavefront, into the slots of the first two terms
  if (r < 3) {
    C h = czero<C>(), c = czero<C>();
#pragma unroll
    for (int gr = 0; gr < Op::kGroups; ++gr) {
      h = cadd(h, terms[3 * gr][r][lane]);
      c = cadd(cadd(c, terms[3 * gr + 1][r][lane]), terms[3 * gr + 2][r][lane]);
    }
    terms[0][r][lane] = h;
    terms[1][r][lane] = c;
  }
  __syncthreads();
  if (r != 0) return;
  double acc = 0.0;
  if (valid) {
    typename Op::Sums s;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      s.hop[q] = terms[0][q][lane];
      s.corner[q] = terms[1][q][lane];
    }
    C o[3];
    Op::finish(oa, f, i, k, s, o);
    acc = site_finish<Op, EPI, 0>(oa, ea, k, i, o, alpha);
  }
  if constexpr (EPI != EPI_STORE && EPI != EPI_CHEB) {
    acc = wave_sum(acc);
    if (lane == 0) ea.part[(size_t)k * ea.nbp + sb] = acc;
  }
}

}  // namespace lq
