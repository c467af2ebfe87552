// Layout kernels: canonical <-> SoA repacking, link compression to 12 reals
// (K6), the staggered Wilson corner matrices (K3) and the mean plaquette.
#include <algorithm>
#include <stdexcept>
#include <type_traits>

#include "kernels.h"
#include "stencil.h"

namespace lq {

// ------------------------------------------------------------ fermions
// Canonical site of field site i: i itself, or for a half-lattice field of
// parity par (EO) the lexicographic site of that parity in the pair (2i, 2i+1).
template <bool EO>
__device__ __forceinline__ size_t canon_site(const Geom& g, int i, int par, int kl) {
  if constexpr (EO) {
    const Coord c = site_coords(g, 2 * i);
    return (size_t)kl * 2 * g.V + 2 * i + ((c.x[1] + c.x[2] + c.x[3] + par) & 1);
  } else {
    return (size_t)kl * g.V + i;
  }
}

template <class P, int NC, bool F64SRC, bool EO>
__global__ void __launch_bounds__(256)
field_in_kernel(const Geom g, const void* __restrict__ canon, typename P::S* __restrict__ soa,
                int par, int nbp, int k0, int nrhs) {
  using C = typename P::C;
  using R = typename P::R;
  int sb, kl;
  map_block(nbp, nrhs, 1, sb, kl);
  const int k = k0 + kl;
  const int i = sb * blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  const size_t cbase = canon_site<EO>(g, i, par, kl) * NC;
  C v[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    if constexpr (F64SRC) {
      const double2 z = ((const double2*)canon)[cbase + q];
      v[q].x = (R)z.x; v[q].y = (R)z.y;
    } else {
      const float2 z = ((const float2*)canon)[cbase + q];
      v[q].x = (R)z.x; v[q].y = (R)z.y;
    }
  }
  st_site<P, NC>(soa + (size_t)k * field_planes<P>(NC) * g.Vp, g.Vp, i, v);
}

// The canonical field is written in storage order through LDS: a lane writing
// its own site's record would touch 64 lines with every store.  Bound by
// memory; FP64 Wilson on 16^3 x 32 (50 MB) 13.8 us directly, 8.2 so (6.1 TB/s
// from the caches).  The half-lattice forms, whose sites are every other one,
// write directly, and field_in_kernel reads directly: the lines of its reads
// stay in L1 until used (9.5 us; 10.5 through LDS).
template <class P, int NC, bool F64DST, bool EO>
__global__ void __launch_bounds__(256)
field_out_kernel(const Geom g, const typename P::S* __restrict__ soa, void* __restrict__ canon,
                 int par, int nbp, int k0, int nrhs) {
  using C = typename P::C;
  using Z = typename std::conditional<F64DST, double2, float2>::type;
  using ZR = typename std::conditional<F64DST, double, float>::type;
  int sb, kl;
  map_block(nbp, nrhs, 1, sb, kl);
  const int k = k0 + kl;
  const int i = sb * blockDim.x + threadIdx.x;
  Z z[NC];
  if (i < g.V) {
    C v[NC];
    ld_site<P, NC>(soa + (size_t)k * field_planes<P>(NC) * g.Vp, g.Vp, i, v);
#pragma unroll
    for (int q = 0; q < NC; ++q) { z[q].x = (ZR)v[q].x; z[q].y = (ZR)v[q].y; }
  }
  if constexpr (EO) {
    if (i >= g.V) return;
    const size_t cbase = canon_site<EO>(g, i, par, kl) * NC;
#pragma unroll
    for (int q = 0; q < NC; ++q) ((Z*)canon)[cbase + q] = z[q];
  } else {
    __shared__ Z rec[256 * (NC | 1)];
    const int i0 = sb * blockDim.x;
    if (i < g.V) {
#pragma unroll
      for (int q = 0; q < NC; ++q) rec[threadIdx.x * (NC | 1) + q] = z[q];
    }
    __syncthreads();
    const int n = min((int)blockDim.x, g.V - i0) * NC;
    Z* dst = (Z*)canon + ((size_t)kl * g.V + i0) * NC;
    for (int e = threadIdx.x; e < n; e += blockDim.x) dst[e] = rec[e / NC * (NC | 1) + e % NC];
  }
}

#define LQ_PNC(prec, nc, CALL)                                                        \
  do {                                                                                \
    if (prec == P64 && nc == 12) { using PP = F64; constexpr int NCC = 12; CALL; }    \
    else if (prec == P64 && nc == 3) { using PP = F64; constexpr int NCC = 3; CALL; }  \
    else if (prec == P32 && nc == 12) { using PP = F32; constexpr int NCC = 12; CALL; } \
    else if (prec == P32 && nc == 3) { using PP = F32; constexpr int NCC = 3; CALL; }  \
    else if (prec == P16 && nc == 12) { using PP = Q16; constexpr int NCC = 12; CALL; } \
    else if (prec == P16 && nc == 3) { using PP = Q16; constexpr int NCC = 3; CALL; }  \
    else throw std::runtime_error("unsupported precision/components");                \
  } while (0)

#define LQ_FIELD_LAUNCH(KERNEL, F64FLAG, SRC, DST)                                          \
  do {                                                                                    \
    if (par < 0)                                                                          \
      LQ_PNC(prec, nc, hipLaunchKernelGGL((KERNEL<PP, NCC, F64FLAG, false>),              \
                                          dim3(nbp * nrhs), dim3(block_of(g.V)), 0, s, g, SRC, DST, \
                                          par, nbp, k0, nrhs));                           \
    else                                                                                  \
      LQ_PNC(prec, nc, hipLaunchKernelGGL((KERNEL<PP, NCC, F64FLAG, true>),               \
                                          dim3(nbp * nrhs), dim3(block_of(g.V)), 0, s, g, SRC, DST, \
                                          par, nbp, k0, nrhs));                           \
  } while (0)

void launch_field_in(int prec, int nc, const Geom& g, const void* canon, int canon_f64, void* soa,
                     int nbp, int k0, int nrhs, hipStream_t s, int par) {
  if (nbp * nrhs == 0) return;
  if (canon_f64) LQ_FIELD_LAUNCH(field_in_kernel, true, canon, (typename PP::S*)soa);
  else LQ_FIELD_LAUNCH(field_in_kernel, false, canon, (typename PP::S*)soa);
}

void launch_field_out(int prec, int nc, const Geom& g, const void* soa, void* canon, int canon_f64,
                      int nbp, int k0, int nrhs, hipStream_t s, int par) {
  if (nbp * nrhs == 0) return;
  if (canon_f64) LQ_FIELD_LAUNCH(field_out_kernel, true, (const typename PP::S*)soa, canon);
  else LQ_FIELD_LAUNCH(field_out_kernel, false, (const typename PP::S*)soa, canon);
}

// --------------------------------------------------------------- links
// Sites [i0, i0 + n) of the canonical field (canon points at site i0) into
// every link copy the gauge field keeps, in one pass: FP64 with 18 reals, the
// 32-bit and 16-bit copies, the per-parity half-lattice copies of the even-odd
// blocks (link mu of site i at half site i / 2 of its parity's array), and the
// largest deviation of a row 2 from conj(row0 x row1): zero up to rounding for
// SU(3) links, which is what the 12-real storage relies on.  The last sites'
// call also zeroes the padding of every slab, so the buffer needs no clearing.
//
// Bound by memory: 75 MB in and 170 MB out for FP32 and 16-bit copies on
// 16^3 x 32.  The 64 sites of a block are read in storage order through LDS
// (a lane reading its own site would touch 64 lines of 576-byte records), one
// direction per wavefront.  Clearing, repacking, four conversions and the
// check took 170 us as separate kernels, this one 50 (4.9 TB/s).
__global__ void __launch_bounds__(256)
gauge_in_kernel(const Geom g, int Vhp, const double2* __restrict__ canon, int i0, int n,
                const GaugeOut o) {
  __shared__ double2 rec[64][37];   // a site's 36 entries; 37: off the bank period
  __shared__ double red[4];
  const int j0 = blockIdx.x * 64;
  const int cnt = max(0, min(64, n - j0));
  for (int e = threadIdx.x; e < cnt * 36; e += 256)
    rec[e / 36][e % 36] = canon[(size_t)j0 * 36 + e];
  __syncthreads();
  const int mu = threadIdx.x >> 6, sl = threadIdx.x & 63;
  const int i = i0 + j0 + sl;
  const bool site = sl < cnt;
  double2 m[9];
  float2 f[9];
  double dev = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    m[k] = site ? rec[sl][mu * 9 + k] : make_double2(0.0, 0.0);
    f[k] = make_float2((float)m[k].x, (float)m[k].y);
  }
  if (site) {
    const double2 r[3] = {cconj(csub(cmul(m[1], m[5]), cmul(m[2], m[4]))),
                          cconj(csub(cmul(m[2], m[3]), cmul(m[0], m[5]))),
                          cconj(csub(cmul(m[0], m[4]), cmul(m[1], m[3])))};
#pragma unroll
    for (int k = 0; k < 3; ++k)
      dev = fmax(dev, fmax(fabs(r[k].x - m[6 + k].x), fabs(r[k].y - m[6 + k].y)));
  }
  // past the sites of a call only the padding that follows the last site
  if (site || (i >= g.V && i < g.Vp)) {
    store_link<F64, 18>(o.u64, g.Vp, mu, i, m);
    if (o.u32_18) store_link<F32, 18>(o.u32_18, g.Vp, mu, i, f);
    if (o.u32_12) store_link<F32, 12>(o.u32_12, g.Vp, mu, i, f);
    if (o.u16_12) store_link<Q16L, 12>(o.u16_12, g.Vp, mu, i, f);
    if (o.u16_18) store_link<Q16L, 18>(o.u16_18, g.Vp, mu, i, f);
  }
  if (o.eo64 && (site || (i >= g.V && i < 2 * Vhp))) {
    int par = i & 1;
    if (site) {
      const Coord c = site_coords(g, i);
      par = (c.x[0] + c.x[1] + c.x[2] + c.x[3]) & 1;
    }
    const int h = i >> 1;
    const size_t p18 = (size_t)par * 36 * Vhp, p12 = (size_t)par * 24 * Vhp;
    store_link<F64, 18>(o.eo64 + p18, Vhp, mu, h, m);
    if (o.eo32_18) store_link<F32, 18>(o.eo32_18 + p18, Vhp, mu, h, f);
    if (o.eo32_12) store_link<F32, 12>(o.eo32_12 + p12, Vhp, mu, h, f);
    if (o.eo16_12) store_link<Q16L, 12>(o.eo16_12 + p12, Vhp, mu, h, f);
    if (o.eo16_18) store_link<Q16L, 18>(o.eo16_18 + p18, Vhp, mu, h, f);
  }
  for (int off = 32; off >= 1; off >>= 1) dev = fmax(dev, __shfl_xor(dev, off, 64));
  if (sl == 0) red[mu] = dev;
  __syncthreads();
  // non-negative doubles order as their bits do
  if (threadIdx.x == 0)
    atomicMax(o.dev, (unsigned long long)__double_as_longlong(
                         fmax(fmax(red[0], red[1]), fmax(red[2], red[3]))));
}

void launch_gauge_in(const Geom& g, int Vhp, const void* canon, int i0, int n, const GaugeOut& o,
                     hipStream_t s) {
  if (n <= 0) return;
  int end = i0 + n;
  if (end == g.V) end = o.eo64 ? std::max(g.Vp, 2 * Vhp) : g.Vp;
  hipLaunchKernelGGL(gauge_in_kernel, dim3((end - i0 + 63) / 64), dim3(256), 0, s, g, Vhp,
                     (const double2*)canon, i0, n, o);
}

// ---------------------------------------------------------- corners (K3)
// W_s(x) = (1/24) sum over the 24 orderings of the path products from x to
// x + s taking one link per direction.  With pt(T) = x + sum_{nu in T} s_nu nu
// and P(T) = sum of the products along all orderings of the directions in T,
//   P(T) = sum_{mu in T} P(T \ mu) L(pt(T \ mu), s_mu mu),   P({}) = 1,
// where L(y, +mu) = U_mu(y) and L(y, -mu) = U_mu(y - mu)^dag.
//
// P(T) depends on the signs of T's directions only, so the eight stored
// corners of a site (s4 = +1) share 18 matrices of level 2 and 20 of level 3:
// 128 products and 164 links a site instead of 320 and 512 with every corner
// on its own, which was bound by those loads (9.7 GB through L2 on 16^3 x 32,
// 849 us, and 65 for the 32-bit and 16-bit copies; now 271 with the copies).
// A block takes 16 sites, one matrix of the level per thread row (16 lanes),
// and the levels meet in LDS (46 KB: three blocks per CU).  Each corner's
// sums run in the same order as on its own.
struct M3 { double2 e[9]; };

__device__ __forceinline__ void m3_load(const double2* __restrict__ u, int Vp, int mu, int site,
                                        bool dag, M3& m) {
  if (!dag) {
#pragma unroll
    for (int k = 0; k < 9; ++k) m.e[k] = u[(size_t)(mu * 9 + k) * Vp + site];
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) m.e[a * 3 + b] = cconj(u[(size_t)(mu * 9 + b * 3 + a) * Vp + site]);
  }
}

__device__ __forceinline__ void m3_mul_acc(const M3& a, const M3& b, M3& acc) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = acc.e[i * 3 + j];
#pragma unroll
      for (int k = 0; k < 3; ++k) s = cfma(a.e[i * 3 + k], b.e[k * 3 + j], s);
      acc.e[i * 3 + j] = s;
    }
}

__device__ __forceinline__ void m3_zero(M3& m) {
#pragma unroll
  for (int k = 0; k < 9; ++k) m.e[k] = make_double2(0.0, 0.0);
}

constexpr int kCornerSites = 16, kCornerRows = 20;

// Index steps of a site to x + nu and x - nu.
struct Steps { int f[4], b[4]; };

// the link L(y, -+mu) (neg: the step is -mu), y = site `at`, whose coordinate
// along mu is that of x
__device__ __forceinline__ void path_link(const double2* __restrict__ u, int Vp, const Steps& st,
                                          int at, int mu, bool neg, M3& m) {
  int back = 0;
#pragma unroll
  for (int nu = 0; nu < 4; ++nu) back = nu == mu ? st.b[nu] : back;
  const double2* p = u + (size_t)(mu * 9) * Vp + (neg ? at + back : at);
  M3 l;
#pragma unroll
  for (int k = 0; k < 9; ++k) l.e[k] = p[(size_t)k * Vp];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double2 t = cconj(l.e[b * 3 + a]), v = l.e[a * 3 + b];
      m.e[a * 3 + b] = make_double2(neg ? t.x : v.x, neg ? t.y : v.y);
    }
}
// index step of direction nu with the sign of bit nu of neg
__device__ __forceinline__ int step_of(const Steps& st, int nu, int neg) {
  int d = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) d = k == nu ? ((neg >> k) & 1 ? st.b[k] : st.f[k]) : d;
  return d;
}
// places of the level-2 matrix of directions a < b and of the level-3 matrix
// without direction m, for the signs neg (bits of the directions < 3)
__device__ __forceinline__ int place2(int a, int b, int neg) {
  const int sa = (neg >> a) & 1, sb = (neg >> b) & 1;
  return b == 3 ? 12 + 2 * a + sa : 4 * (a + b - 1) + sa + 2 * sb;
}
__device__ __forceinline__ int place3(int m, int neg) {
  if (m == 3) return neg & 7;
  const int lo = m == 0 ? 1 : 0, hi = m == 2 ? 1 : 2;
  return 8 + 4 * m + ((neg >> lo) & 1) + 2 * ((neg >> hi) & 1);
}

__global__ void __launch_bounds__(kCornerSites * kCornerRows)
__attribute__((amdgpu_waves_per_eu(4, 4)))
corners_kernel(const Geom g, const double2* __restrict__ u, double2* __restrict__ w64,
               float2* __restrict__ w32, short2* __restrict__ w16) {
  __shared__ double2 lv[kCornerRows][9][kCornerSites];
  const int sl = threadIdx.x % kCornerSites, row = threadIdx.x / kCornerSites;
  const int i = blockIdx.x * kCornerSites + sl;
  const int x = min(i, g.V - 1);   // blocks past the last site: its padding, stored as zero
  const Coord c = site_coords(g, x);
  Steps st;
#pragma unroll
  for (int nu = 0; nu < 4; ++nu) {
    st.f[nu] = c.x[nu] == g.L[nu] - 1 ? (1 - g.L[nu]) * g.stride[nu] : g.stride[nu];
    st.b[nu] = c.x[nu] == 0 ? (g.L[nu] - 1) * g.stride[nu] : -g.stride[nu];
  }
  M3 p, l1, l2;
  // level 2, a < b: L(x, a) L(x + a, b) + L(x, b) L(x + b, a)
  if (row < 18) {
    int a, b, neg;
    if (row >= 12) {
      a = (row - 12) >> 1; b = 3; neg = ((row - 12) & 1) << a;
    } else {
      const int q = row >> 2;
      a = q == 2 ? 1 : 0; b = q == 0 ? 1 : 2;
      neg = ((row & 1) << a) | (((row >> 1) & 1) << b);
    }
    const bool na = (neg >> a) & 1, nb = (neg >> b) & 1;
    m3_zero(p);
    path_link(u, g.Vp, st, x, a, na, l1);
    path_link(u, g.Vp, st, x + step_of(st, a, neg), b, nb, l2);
    m3_mul_acc(l1, l2, p);
    path_link(u, g.Vp, st, x, b, nb, l1);
    path_link(u, g.Vp, st, x + step_of(st, b, neg), a, na, l2);
    m3_mul_acc(l1, l2, p);
#pragma unroll
    for (int k = 0; k < 9; ++k) lv[row][k][sl] = p.e[k];
  }
  __syncthreads();
  // level 3 without direction m: sum over its directions mu, ascending
  {
    int m = 3, neg = row;
    if (row >= 8) {
      m = (row - 8) >> 2;
      const int lo = m == 0 ? 1 : 0, hi = m == 2 ? 1 : 2;
      neg = ((row & 1) << lo) | (((row >> 1) & 1) << hi);
    }
    m3_zero(p);
#pragma unroll 1
    for (int q = 0; q < 3; ++q) {
      const int mu = q + (q >= m);                     // the q-th direction of the three
      const int q0 = q == 0 ? 1 : 0, q1 = q == 2 ? 1 : 2;
      const int a = q0 + (q0 >= m), b = q1 + (q1 >= m);
      const int at = place2(a, b, neg);
#pragma unroll
      for (int k = 0; k < 9; ++k) l1.e[k] = lv[at][k][sl];
      path_link(u, g.Vp, st, x + step_of(st, a, neg) + step_of(st, b, neg), mu, (neg >> mu) & 1, l2);
      m3_mul_acc(l1, l2, p);
    }
  }
  __syncthreads();   // level 3 takes level 2's place
#pragma unroll
  for (int k = 0; k < 9; ++k) lv[row][k][sl] = p.e[k];
  __syncthreads();
  // the corner with the signs of row's bits
  if (row >= 8) return;
  m3_zero(p);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    const int at = place3(mu, row);
    int y = x;
#pragma unroll
    for (int nu = 0; nu < 4; ++nu) y += nu == mu ? 0 : ((row >> nu) & 1) ? st.b[nu] : st.f[nu];
#pragma unroll
    for (int k = 0; k < 9; ++k) l1.e[k] = lv[at][k][sl];
    path_link(u, g.Vp, st, y, mu, (row >> mu) & 1, l2);
    m3_mul_acc(l1, l2, p);
  }
  const bool pad = i >= g.V;
  float2 f[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    p.e[k] = pad ? make_double2(0.0, 0.0) : make_double2(p.e[k].x / 24.0, p.e[k].y / 24.0);
    f[k] = make_float2((float)p.e[k].x, (float)p.e[k].y);
  }
  store_corner<F64>(w64, g.Vp, row, i, p.e);
  if (w32) store_corner<F32>(w32, g.Vp, row, i, f);
  if (w16) store_corner<Q16L>(w16, g.Vp, row, i, f);
}

void launch_corners(const Geom& g, const double2* u64, double2* c64, float2* c32, short2* c16,
                    hipStream_t s) {
  // Vp is a multiple of the block's sites
  hipLaunchKernelGGL(corners_kernel, dim3(g.Vp / kCornerSites), dim3(kCornerSites * kCornerRows), 0,
                     s, g, u64, c64, c32, c16);
}

// ------------------------------------------------------------ plaquette
// (1/3) Re tr U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag summed over mu < nu.
__global__ void __launch_bounds__(256)
plaquette_kernel(const Geom g, const double2* __restrict__ u, double* __restrict__ part) {
  __shared__ double red[16];
  // XCD b % 8 takes a contiguous range, so that neighbouring sites' links are
  // shared in its L2 (16^3 x 32: 54 us dealt out in turn, 48 so)
  const int sb = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int i = sb * blockDim.x + threadIdx.x;
  double acc = 0.0;
  if (i < g.V) {
    const Coord c = site_coords(g, i);
    for (int mu = 0; mu < 4; ++mu)
      for (int nu = mu + 1; nu < 4; ++nu) {
        bool w;
        const int xm = nb_fwd(g, c, i, mu, w);
        const int xn = nb_fwd(g, c, i, nu, w);
        M3 a, b, cc, d, ab, abc;
        m3_load(u, g.Vp, mu, i, false, a);
        m3_load(u, g.Vp, nu, xm, false, b);
        m3_load(u, g.Vp, mu, xn, true, cc);
        m3_load(u, g.Vp, nu, i, true, d);
        m3_zero(ab);
        m3_mul_acc(a, b, ab);
        m3_zero(abc);
        m3_mul_acc(ab, cc, abc);
        double tr = 0.0;
        for (int p = 0; p < 3; ++p)
          for (int k = 0; k < 3; ++k) tr += abc.e[p * 3 + k].x * d.e[k * 3 + p].x - abc.e[p * 3 + k].y * d.e[k * 3 + p].y;
        acc += tr / 3.0;
      }
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0 && i < g.V) part[sb] = s;
}

__global__ void plaquette_finish_kernel(const double* __restrict__ part, int n, double V,
                                        double* out) {
  __shared__ double red[16];
  const double s = sum_partials(part, n, red, 1);
  if (threadIdx.x == 0) *out = s / (6.0 * V);
}

void launch_plaquette(const Geom& g, const double2* u64, double* part, int nbp, double* out,
                      hipStream_t s) {
  const int nb = (g.V + 255) / 256;
  (void)nbp;
  hipLaunchKernelGGL(plaquette_kernel, dim3((nb + 7) / 8 * 8), dim3(256), 0, s, g, u64, part);
  hipLaunchKernelGGL(plaquette_finish_kernel, dim3(1), dim3(64), 0, s, part, nb, (double)g.V, out);
}

// ------------------------------------------------------------- filling
__global__ void fill_zero_kernel(uint4* __restrict__ p, size_t n16) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n16;
       e += (size_t)gridDim.x * blockDim.x)
    p[e] = make_uint4(0, 0, 0, 0);
}

void launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  // callers pass 16-byte aligned, 16-byte multiple regions
  const size_t n16 = bytes / 16;
  if (n16 == 0) return;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)p, n16);
}

// Deterministic test data for timing: every component of nrhs vector fields
// uniform in [-1, 1) from a counter-based hash of (seed, system, site,
// component) (the 32-bit finaliser of MurmurHash3), stored in the field's
// precision.
__device__ __forceinline__ uint32_t mix32(uint32_t h) {
  h ^= h >> 16; h *= 0x85ebca6bu;
  h ^= h >> 13; h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}
template <class P, int NC>
__global__ void __launch_bounds__(256)
fill_test_kernel(const Geom g, typename P::S* __restrict__ f, int nbp, int nrhs, uint32_t seed) {
  using C = typename P::C;
  using R = typename P::R;
  int sb, k;
  map_block(nbp, nrhs, 1, sb, k);
  const int i = sb * blockDim.x + threadIdx.x;
  if (i >= g.V) return;
  C v[NC];
  uint32_t h = mix32(seed ^ mix32((uint32_t)k * 0x9e3779b9u ^ mix32((uint32_t)i)));
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    h = mix32(h + 0x632be5abu);
    const uint32_t h2 = mix32(h ^ 0x5bd1e995u);
    v[q].x = (R)((int32_t)h * (1.0 / 2147483648.0));
    v[q].y = (R)((int32_t)h2 * (1.0 / 2147483648.0));
  }
  st_site<P, NC>(f + (size_t)k * field_planes<P>(NC) * g.Vp, g.Vp, i, v);
}

void launch_fill_test(int prec, int nc, const Geom& g, void* soa, int nrhs, uint32_t seed,
                      hipStream_t s) {
  const int nbp = nbp_of(g.V);
  if (nbp * nrhs == 0) return;
  LQ_PNC(prec, nc, hipLaunchKernelGGL((fill_test_kernel<PP, NCC>), dim3(nbp * nrhs), dim3(block_of(g.V)), 0,
                                      s, g, (typename PP::S*)soa, nbp, nrhs, seed));
}

}  // namespace lq
