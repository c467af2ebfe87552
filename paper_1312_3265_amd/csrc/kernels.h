// Host-side launch interface of the kernels (one translation unit per group).
#pragma once

#include <algorithm>

#include <hip/hip_runtime.h>

#include "common.h"
#include "lq_types.h"

namespace lq {

struct OpArgs;
struct EpiArgs;

// The search-direction buffers of a CG solve, used in turn: iteration q of a
// group of G reads p[q] and writes p_{k+1} into p[(q + 1) % G] (G = 4, or 2
// for FP64; x takes the group's steps on its last iteration).
struct PRing {
  void* p[4];
};

// Whether the staggered corner stencil splits a site's terms over the
// wavefronts of its block (stencil_swsplit.h) for nrhs systems of V sites:
// fields of one-wavefront blocks, where the launch's blocks are resident
// together -- two a compute unit in FP64 (their LDS) and FP32 (registers),
// four in 16 bits.  Past that the one-thread form (with systems sharing the
// matrices of a thread) is ahead.  M p and the CG update together, split
// against the best one-thread form, in us: FP64 8^4 eight systems (512 blocks)
// 16 and 20, nine 22 and 20, 16^2 x 8^2 one (256) 20 and 30, two 32 and 31,
// nine 121 and 64, 36 457 and 306; FP32 12^2 x 8^2 three (432) 13 and 14, four
// 17 and 15, 16^2 x 8^2 36 systems 154 and 97; 16 bits 8^4 eighteen (1152) 21
// and 23, 24 (1536) 24 and 23, 16^2 x 8^2 three (768) 16 and 17, 36 115 and 70.
// The two forms add the terms in the same order, so the choice does not change
// a system's bits.
inline bool sw_split_fits(int prec, int V, int nrhs) {
  return block_of(V) == 64 && (long long)nbp_of(V) * nrhs <= (prec == P16 ? 1024 : 512);
}

// Bytes per site of the widest array that a stencil addresses from one base:
// a vector field, one direction's links or one corner's matrices.
inline int widest_record(int op, int prec, int nl) {
  const int z = prec == P64 ? 16 : prec == P32 ? 8 : 4;   // a complex number
  const int nc = op == OP_SW_CORNERS || op == OP_SW_OTF ? 3 : 12;
  const int vec = (nc + (prec == P16)) * z, link = nl / 2 * z;
  const int corner = op == OP_SW_CORNERS ? 9 * z : 0;
  return std::max(std::max(vec, link), corner);
}

// ---- stencils: op = OpKind, prec = Prec, nl = 18/12 link reals
void launch_stencil(int op, int prec, int nl, bool dag, int epi, const OpArgs& oa,
                    const void* in, const EpiArgs& ea, int nrhs, hipStream_t s);

// Bytes of the intermediate fields of the on-the-fly Gamma_55 for one system
// (OpArgs::g55w; 14 fields of three complex numbers, FP64 or FP32).
size_t g55_bytes_per_system(const Geom& g, int prec);

// ---- CG vector kernels (templated on precision and components)
void launch_p_update(int prec, int nc, const Geom& g, SlotState* st, int par, int pend_next,
                     const double* part, int nbp, const void* p, void* pout, const void* r, int k0,
                     int nrhs, hipStream_t s);
// Reliable-update kernels act on running slots k with mask[k] != 0 (mask may be null).
void launch_ru_accumulate(int prec, int nc, const Geom& g, const SlotState* st, const int* mask,
                          double* xhi, void* xlo, const PRing& ring, int nbp, int k0, int nrhs,
                          hipStream_t s);
// part_f, part_g: the even-odd norms (null otherwise), see ru_finish_kernel;
// per: partials_per of the fields
void launch_ru_finish(SlotState* st, const int* mask, const double* part, const double* part_f,
                      const double* part_g, int nbp, int per, int k0, int nrhs, double ncomp,
                      int rescale, int max_cand, int init, int par, hipStream_t s);
void launch_ru_convert(int prec, int nc, const Geom& g, const SlotState* st, const int* mask,
                       const double* rhi, void* rlo, const PRing& ring, double* part, int nbp,
                       int init, int k0, int nrhs, hipStream_t s);
void launch_ru_commit(SlotState* st, const int* mask, const double* part, int nbp, int per,
                      int k0, int nrhs, hipStream_t s);
void launch_load_prepare(int prec, int nc, const Geom& g, double* xhi, void* xlo, double* rhi,
                         const double* b, int nbp, int k0, int nrhs, hipStream_t s);

// ---- layout / conversion
// canonical (V, nc) complex (c128 if src_f64 else c64) -> SoA field (prec) for rhs k0..
// par >= 0: g is a half-lattice geometry and the SoA field holds the sites of
// that parity of the canonical (2 g.V, nc) field (even-odd blocks)
void launch_field_in(int prec, int nc, const Geom& g, const void* canon, int canon_f64, void* soa,
                     int nbp, int k0, int nrhs, hipStream_t s, int par = -1);
void launch_field_out(int prec, int nc, const Geom& g, const void* soa, void* canon, int canon_f64,
                      int nbp, int k0, int nrhs, hipStream_t s, int par = -1);
// The link copies of a gauge field (null: not kept); dev: the largest deviation
// from SU(3), as the bits of a double, zero before the first call.
struct GaugeOut {
  double2* u64;
  float2 *u32_18, *u32_12;
  short2 *u16_12, *u16_18;
  double2* eo64;               // even-odd copies: per parity, Vhp sites a slab
  float2 *eo32_18, *eo32_12;
  short2 *eo16_12, *eo16_18;
  unsigned long long* dev;
};
// sites [i0, i0 + n) of a canonical gauge field whose site i0 is at `canon`
void launch_gauge_in(const Geom& g, int Vhp, const void* canon, int i0, int n, const GaugeOut& o,
                     hipStream_t s);
// c32, c16 may be null
void launch_corners(const Geom& g, const double2* u64, double2* c64, float2* c32, short2* c16,
                    hipStream_t s);
void launch_plaquette(const Geom& g, const double2* u64, double* part, int nbp, double* out,
                      hipStream_t s);
void launch_fill_zero(void* p, size_t bytes, hipStream_t s);
// nrhs vector fields of nc components in precision prec, every component
// uniform in [-1, 1) from a hash of (seed, system, site, component)
void launch_fill_test(int prec, int nc, const Geom& g, void* soa, int nrhs, uint32_t seed,
                      hipStream_t s);

// ---- pion correlator (Wilson point-source propagators, canonical complex128)
int pion_blocks_per_slice(int L4);
// part: L4 * pion_blocks_per_slice(L4) doubles; corr: L4 doubles (device)
void launch_pion_correlator(const Geom& g, int nsrc, const double2* props, double* part,
                            double* corr, hipStream_t s);

// ---- Gram-Schmidt of Lanczos and Arnoldi (FP64, vectors of nc planes)
// Upper limit of the blocks along the vector elements, and so of the partials
// per sum: part_h holds kLzBlocks complex numbers per vector, part_n kLzBlocks
// doubles.
constexpr int kLzBlocks = 512;
// partials of h = V^H w
void launch_lz_dots(const Geom& g, int nc, const double2* V, int nvec, double2* w, double* part_h,
                    hipStream_t s);
// h from its partials; alpha = the sum of alpha_part (may be null)
void launch_lz_reduce(const Geom& g, int nc, const double* part_h, int nvec, double2* h,
                      const double* alpha_part, int nbp_alpha, double* alpha_out, hipStream_t s);
// w -= V h, with partials of ||w||^2 when part_n is not null
void launch_lz_update(const Geom& g, int nc, const double2* V, int nvec, const double2* h,
                      double2* w, double* part_n, hipStream_t s);
// w -= V h, then the partials of V^H w
void launch_lz_update_dots(const Geom& g, int nc, const double2* V, int nvec, const double2* h,
                           double2* w, double* part_h, hipStream_t s);
// beta = sqrt(sum of part_n)
void launch_lz_finish(const Geom& g, int nc, const double* part_n, double* beta_out, hipStream_t s);
// the same, and vnext = w / beta
void launch_lz_normalize(const Geom& g, int nc, const double2* w, const double* part_n,
                         double* beta_out, double2* vnext, hipStream_t s);

}  // namespace lq
