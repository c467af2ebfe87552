// Gram-Schmidt kernels of the Lanczos and Arnoldi drivers.
//
// Basis V (nvec vectors of n = nc * Vp complex doubles, back to back), work
// vector w.  One classical Gram-Schmidt pass is h = V^H w (dots + reduce),
// w -= V h (update); the drivers make two.  Each pass streams the basis, by
// far the largest operand (200 Wilson vectors on 16^3 x 32 are 5 GB), so these
// kernels are bound by HBM and every pass over the basis counts:
//   * a block takes tiles of 64 consecutive elements and its eight waves split
//     the vectors (wave g takes vectors g, g + 8, ...): every load of a wave is
//     1 KB of one vector, KT of them in flight per wave, which covers the
//     latency with one or two blocks on a CU;
//   * the first pass's update and the second pass's dots are one kernel: the
//     tile of V stays in registers between them, so the two passes read the
//     basis three times instead of four.
// Measured on MI355X, Wilson 16^3 x 32 (25 MB per vector), averages over a
// 200-step run (100 vectors, 2.5 GB): dots 456 us, update 454 us, 5.5 TB/s
// (one block of 256 threads per CU, each chunk of eight vectors reduced over
// the block: 1250 us; a one-block reduction of the partials: 37 us, here one
// wave per vector: 5 us).  A run of 200 steps: 729 -> 301 ms.
//
// Every sum runs in a fixed order (waves in order, tiles in order, the
// partials of a launch in lane-strided order), so results do not depend on
// scheduling.
#include "kernels.h"

namespace lq {

constexpr int kLzWaves = 8;              // waves per block
constexpr int kLzThreads = 64 * kLzWaves;

// Sums of M values per lane (M a power of two <= EW) over groups of EW lanes:
// each step halves the values a lane keeps, so all M sums take about M
// exchanges instead of M log2(EW).  Returns the sum of value
// lz_sum_index<M, EW>(lane).
template <int M, int EW>
__device__ __forceinline__ double wave_sum_many(double (&a)[M]) {
  int off = EW / 2;
#pragma unroll
  for (int m = M / 2; m >= 1; m >>= 1, off >>= 1) {
    const bool up = (threadIdx.x & off) != 0;
#pragma unroll
    for (int i = 0; i < m; ++i) {
      const double send = up ? a[i] : a[i + m];
      const double keep = up ? a[i + m] : a[i];
      a[i] = keep + __shfl_xor(send, off, 64);
    }
  }
  double v = a[0];
  for (; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
template <int M, int EW>
__device__ __forceinline__ int lz_sum_index(int lane) {
  int j = 0, off = EW / 2;
#pragma unroll
  for (int m = M / 2; m >= 1; m >>= 1, off >>= 1) j += (lane & off) ? m : 0;
  return j;
}
constexpr int pow2_at_least(int v) { int p = 1; while (p < v) p *= 2; return p; }

// h_k partials of this block for the vectors c0 .. c0 + KG KT - 1 (KG = 512 /
// EW, c0 = KG KT blockIdx.y): part_h[(k * nblk + block) * 2 + {0: re, 1: im}].
// A tile is EW consecutive elements; thread (kg, e) takes element e of vectors
// kg, kg + KG, ..., KT of them at once.  With UPDATE (gridDim.y = 1): first
// w -= V h, from the same registers.  Vectors past nvec are the last one read
// again (h = 0 for them, their sums dropped).
template <int EW, int KT, bool UPDATE>
__global__ void __launch_bounds__(kLzThreads) __attribute__((amdgpu_waves_per_eu(4, 8)))
lz_dots_kernel(const double2* __restrict__ V, size_t n, int nvec, const double2* __restrict__ h,
               double2* __restrict__ w, double* __restrict__ part_h, int nblk) {
  constexpr int KG = kLzThreads / EW;
  __shared__ double2 hs[UPDATE ? KG * KT : 1];
  __shared__ double2 red[UPDATE ? 2 : 1][UPDATE ? kLzWaves : 1][EW];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave * (64 / EW) + lane / EW;
  const int le = lane & (EW - 1);
  const int c0 = blockIdx.y * KG * KT;
  if constexpr (UPDATE) {
    for (int k = threadIdx.x; k < KG * KT; k += kLzThreads)
      hs[k] = k < nvec ? h[k] : make_double2(0.0, 0.0);
    __syncthreads();
  }
  constexpr int M = pow2_at_least(2 * KT);
  static_assert(M <= EW, "the block's sums are reduced over EW lanes");
  double acc[M];
#pragma unroll
  for (int j = 0; j < M; ++j) acc[j] = 0.0;
  const size_t ntiles = n / EW;
  int buf = 0;
  for (size_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const size_t e = tile * EW + le;
    double2 v[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const int k = min(c0 + t * KG + kg, nvec - 1);
      v[t] = V[(size_t)k * n + e];
    }
    double2 x = w[e];
    if constexpr (UPDATE) {
      double2 s = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const double2 c = hs[t * KG + kg];
        s.x += v[t].x * c.x - v[t].y * c.y;
        s.y += v[t].x * c.y + v[t].y * c.x;
      }
#pragma unroll
      for (int off = EW; off < 64; off <<= 1) {
        s.x += __shfl_xor(s.x, off, 64);
        s.y += __shfl_xor(s.y, off, 64);
      }
      // double-buffered: a wave writes this buffer again only after the next
      // tile's barrier, which every wave reaches after its reads below
      if (lane < EW) red[buf][wave][le] = s;
      __syncthreads();
      s = red[buf][0][le];
#pragma unroll
      for (int g = 1; g < kLzWaves; ++g) {
        s.x += red[buf][g][le].x;
        s.y += red[buf][g][le].y;
      }
      buf ^= 1;
      x.x -= s.x;
      x.y -= s.y;
      if (kg == 0) w[e] = x;   // every wave has read the tile's old w (barrier above)
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      acc[2 * t] += v[t].x * x.x + v[t].y * x.y;
      acc[2 * t + 1] += v[t].x * x.y - v[t].y * x.x;
    }
  }
  const double s = wave_sum_many<M, EW>(acc);
  const int j = lz_sum_index<M, EW>(le);
  const int k = c0 + (j >> 1) * KG + kg;
  // with M < EW several lanes hold the same sum: the first writes it
  if ((le & (EW / M - 1)) == 0 && (j >> 1) < KT && k < nvec)
    part_h[((size_t)k * nblk + blockIdx.x) * 2 + (j & 1)] = s;
}

// w -= V h for any number of vectors; block partials of ||w||^2 into part_n
// when it is not null.
template <int KT>
__global__ void __launch_bounds__(kLzThreads) __attribute__((amdgpu_waves_per_eu(4, 8)))
lz_update_kernel(const double2* __restrict__ V, size_t n, int nvec, const double2* __restrict__ h,
                 double2* __restrict__ w, double* __restrict__ part_n) {
  __shared__ double2 hs[1024];
  __shared__ double2 red[2][kLzWaves][64];
  const int lane = threadIdx.x & 63;
  const int kg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int k = threadIdx.x; k < nvec; k += kLzThreads) hs[k] = h[k];
  __syncthreads();
  const size_t ntiles = n / 64;
  double norm = 0.0;
  int buf = 0;
  for (size_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const size_t e = tile * 64 + lane;
    double2 s = make_double2(0.0, 0.0);
    for (int c0 = kg; c0 < nvec; c0 += kLzWaves * KT) {
      double2 v[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const int k = min(c0 + t * kLzWaves, nvec - 1);
        v[t] = V[(size_t)k * n + e];
      }
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const int k = c0 + t * kLzWaves;
        if (k < nvec) {
          const double2 c = hs[k];
          s.x += v[t].x * c.x - v[t].y * c.y;
          s.y += v[t].x * c.y + v[t].y * c.x;
        }
      }
    }
    red[buf][kg][lane] = s;   // double-buffered, as in lz_dots_kernel
    __syncthreads();
    if (kg == 0) {
      double2 x = w[e];
#pragma unroll
      for (int g = 0; g < kLzWaves; ++g) {
        x.x -= red[buf][g][lane].x;
        x.y -= red[buf][g][lane].y;
      }
      w[e] = x;
      norm += x.x * x.x + x.y * x.y;
    }
    buf ^= 1;
  }
  if (part_n && kg == 0) {
    norm = wave_sum(norm);
    if (lane == 0) part_n[blockIdx.x] = norm;
  }
}

// Block k < nvec: h_k from the block partials; block nvec (when alpha_part is
// not null): alpha = the sum of the Lanczos stencil's partials.
__global__ void __launch_bounds__(64)
lz_reduce_kernel(const double* __restrict__ part_h, int nvec, int nblk, double2* __restrict__ h,
                 const double* __restrict__ alpha_part, int nbp_alpha, int per_alpha,
                 double* alpha_out) {
  __shared__ double red[16];
  const int k = blockIdx.x;
  if (k == nvec) {
    const double a = sum_partials(alpha_part, nbp_alpha, red, per_alpha);
    if (threadIdx.x == 0) *alpha_out = a;
    return;
  }
  const double2* p = (const double2*)part_h + (size_t)k * nblk;
  double2 s = make_double2(0.0, 0.0);
  for (int b = threadIdx.x; b < nblk; b += 64) {
    s.x += p[b].x;
    s.y += p[b].y;
  }
  s.x = wave_sum(s.x);
  s.y = wave_sum(s.y);
  if (threadIdx.x == 0) h[k] = s;
}

__global__ void lz_finish_kernel(const double* __restrict__ part_n, int nblk, double* beta_out) {
  __shared__ double red[16];
  const double s = sum_partials(part_n, nblk, red, 1);
  if (threadIdx.x == 0) *beta_out = sqrt(s);
}

// vnext = w / beta, beta = sqrt(sum of the nblk partials part_n), also written
// to beta_out (one launch instead of a one-block kernel and this one)
__global__ void __launch_bounds__(256)
lz_normalize_kernel(size_t n, const double2* __restrict__ w, const double* __restrict__ part_n,
                    int nblk, double* beta_out, double2* __restrict__ vnext) {
  __shared__ double red[16];
  const double bt = sqrt(sum_partials(part_n, nblk, red, 1));
  if (blockIdx.x == 0 && threadIdx.x == 0) *beta_out = bt;
  const double inv = (bt > 1e-300 && isfinite(bt)) ? 1.0 / bt : 0.0;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (size_t)gridDim.x * blockDim.x) {
    const double2 x = w[e];
    vnext[e] = make_double2(x.x * inv, x.y * inv);
  }
}

// Blocks along the elements: two per CU, fewer where the vector has fewer tiles.
static int lz_blocks(size_t n) {
  const size_t tiles = n / 64;
  return (int)(tiles < (size_t)kLzBlocks ? tiles : (size_t)kLzBlocks);
}

template <int KT>
static void dots_launch(const double2* V, size_t n, int nvec, double2* w, double* part_h,
                        hipStream_t s) {
  const int nb = lz_blocks(n), per = kLzWaves * KT;
  hipLaunchKernelGGL((lz_dots_kernel<64, KT, false>), dim3(nb, (nvec + per - 1) / per),
                     dim3(kLzThreads), 0, s, V, n, nvec, (const double2*)nullptr, w, part_h, nb);
}

void launch_lz_dots(const Geom& g, int nc, const double2* V, int nvec, double2* w, double* part_h,
                    hipStream_t s) {
  const size_t n = (size_t)nc * g.Vp;
  // 64 vectors per block row where that still fills the GPU, else 16
  if ((size_t)lz_blocks(n) * ((nvec + 63) / 64) >= 256) dots_launch<8>(V, n, nvec, w, part_h, s);
  else dots_launch<2>(V, n, nvec, w, part_h, s);
}

void launch_lz_reduce(const Geom& g, int nc, const double* part_h, int nvec, double2* h,
                      const double* alpha_part, int nbp_alpha, double* alpha_out, hipStream_t s) {
  const int nb = lz_blocks((size_t)nc * g.Vp);
  hipLaunchKernelGGL(lz_reduce_kernel, dim3(nvec + (alpha_part ? 1 : 0)), dim3(64), 0, s, part_h,
                     nvec, nb, h, alpha_part, nbp_alpha, partials_per(g.V), alpha_out);
}

void launch_lz_update(const Geom& g, int nc, const double2* V, int nvec, const double2* h,
                      double2* w, double* part_n, hipStream_t s) {
  const size_t n = (size_t)nc * g.Vp;
  hipLaunchKernelGGL(lz_update_kernel<8>, dim3(lz_blocks(n)), dim3(kLzThreads), 0, s, V, n, nvec, h,
                     w, part_n);
}

template <int EW, int KT>
static bool fused_launch(const double2* V, size_t n, int nvec, const double2* h, double2* w,
                         double* part_h, hipStream_t s) {
  if (nvec > kLzThreads / EW * KT) return false;
  const int nb = lz_blocks(n);
  hipLaunchKernelGGL((lz_dots_kernel<EW, KT, true>), dim3(nb), dim3(kLzThreads), 0, s, V, n, nvec,
                     h, w, part_h, nb);
  return true;
}

void launch_lz_update_dots(const Geom& g, int nc, const double2* V, int nvec, const double2* h,
                           double2* w, double* part_h, hipStream_t s) {
  const size_t n = (size_t)nc * g.Vp;
  // The tile narrows as the vectors grow in number, so that a thread holds at
  // most eight of them and two blocks fit on a CU: one block's loads then run
  // under the other's barrier and arithmetic.  (With 64-element tiles
  // throughout and up to 26 vectors per thread one block filled the CU, and
  // the pass fell from 5.2 TB/s at 57 vectors to 3.3 TB/s at 168.)  Past 256
  // vectors update and dots are two launches.
  if (fused_launch<64, 1>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<64, 2>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<64, 4>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<64, 6>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<64, 8>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<32, 5>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<32, 6>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<32, 7>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<32, 8>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<16, 5>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<16, 6>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<16, 7>(V, n, nvec, h, w, part_h, s) ||
      fused_launch<16, 8>(V, n, nvec, h, w, part_h, s))
    return;
  launch_lz_update(g, nc, V, nvec, h, w, nullptr, s);
  launch_lz_dots(g, nc, V, nvec, w, part_h, s);
}

void launch_lz_finish(const Geom& g, int nc, const double* part_n, double* beta_out, hipStream_t s) {
  hipLaunchKernelGGL(lz_finish_kernel, dim3(1), dim3(64), 0, s, part_n,
                     lz_blocks((size_t)nc * g.Vp), beta_out);
}

void launch_lz_normalize(const Geom& g, int nc, const double2* w, const double* part_n,
                         double* beta_out, double2* vnext, hipStream_t s) {
  const size_t n = (size_t)nc * g.Vp;
  const size_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(lz_normalize_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256),
                     0, s, n, w, part_n, lz_blocks(n), beta_out, vnext);
}

}  // namespace lq
