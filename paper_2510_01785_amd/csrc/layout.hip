// Conversion of the caller's coefficient layout alm[b][idx(l,m)] into the
// transposed internal layout of the synthesis Legendre kernels, ALMT[idx][b]
// per channel group (chan_group), with the per-coefficient scale factors of
// each entry point:
//
//   ALMT = s * f_m * c_lm * alm   (Im of m = 0 ignored)
//
// f_m is f0 for m = 0 and fm for m > 0; c_lm is the normalisation of the
// scaled recurrence (tables.hip) that the synthesis kernels expect folded in.
// (The analysis kernels write the caller's layout themselves.)
#include "common.h"

namespace shtx {

// A pass over HBM: 2 nalm B complex elements and the nalm factors.  A workgroup
// takes kLayoutThreads consecutive coefficient indices idx(l, m) (m = 0 exactly for
// idx <= lmax) of one slice of 16 channels through an LDS tile: the caller side
// alm[b][idx] is read along idx, all channels of the slice in flight together, and
// the internal side written as contiguous runs of each channel group (a loop over
// the channels, one slice after the other, waited for each load: FP32 us at L 767
// B 64 104 -> 77, L 1535 B 12 72 -> 60, L 2047 B 16 138 -> 134, 4.0 TB/s).
constexpr int kLayoutThreads = 256;
constexpr int kLayoutChannels = 16;

// Two adjacent channels of a row at once where they are aligned (16 bytes in FP32).
__device__ __forceinline__ void store_two(float2 *p, float2 a, float2 b) {
  *reinterpret_cast<float4 *>(p) = make_float4(a.x, a.y, b.x, b.y);
}
__device__ __forceinline__ void store_two(double2 *p, double2 a, double2 b) {
  p[0] = a;
  p[1] = b;
}

template <typename T>
__device__ __forceinline__ cplx<T> scaled(cplx<T> v, double g, bool m0) {
  cplx<T> o;
  o.x = (T)(g * (double)v.x);
  o.y = m0 ? (T)0 : (T)(g * (double)v.y);
  return o;
}

template <typename T>
__global__ void __launch_bounds__(kLayoutThreads)
    k_alm_in(int L, int B, int gmax, const cplx<T> *__restrict__ alm, const double *__restrict__ coefC,
             cplx<T> *__restrict__ ALMT, double s, double f0, double fm) {
  using C = cplx<T>;
  __shared__ C tile[kLayoutThreads][kLayoutChannels + 1];
  const size_t nalm = nalm_of(L);
  const unsigned ns = (unsigned)(B + kLayoutChannels - 1) / kLayoutChannels, blk = blockIdx.x / ns;
  const size_t i0 = (size_t)blk * kLayoutThreads;
  const int ni = (int)min((size_t)kLayoutThreads, nalm - i0);
  const int t = threadIdx.x;
  const size_t idx = i0 + t;
  const int b0 = (int)(blockIdx.x - blk * ns) * kLayoutChannels;
  const int nb = min(kLayoutChannels, B - b0);
  if (t < ni) {
    C v[kLayoutChannels];
#pragma unroll
    for (int b = 0; b < kLayoutChannels; ++b)
      if (b < nb) v[b] = alm[(size_t)(b0 + b) * nalm + idx];
    const bool m0 = idx <= (size_t)L;
    const double g = s * (m0 ? f0 : fm) * coefC[idx];
#pragma unroll
    for (int b = 0; b < kLayoutChannels; ++b)
      if (b < nb) tile[t][b] = scaled<T>(v[b], g, m0);
  }
  __syncthreads();
  const ChanGroup gr = chan_group(b0, B, gmax);
  if (b0 + nb <= gr.g0 + gr.w) {
    // the slice within one group: rows i0 + r of its [idx][w] layout
    C *dst = ALMT + (size_t)gr.g0 * (nalm + kCoefPad) + i0 * gr.w + (b0 - gr.g0);
    if (((nb | gr.w | (b0 - gr.g0) | gr.g0) & 1) == 0) {
      for (int q = t; q < ni * (kLayoutChannels / 2); q += kLayoutThreads) {
        const int r = q / (kLayoutChannels / 2), b = 2 * (q % (kLayoutChannels / 2));
        if (b < nb) store_two(dst + (size_t)r * gr.w + b, tile[r][b], tile[r][b + 1]);
      }
    } else {
      for (int q = t; q < ni * kLayoutChannels; q += kLayoutThreads) {
        const int r = q / kLayoutChannels, b = q % kLayoutChannels;
        if (b < nb) dst[(size_t)r * gr.w + b] = tile[r][b];
      }
    }
    return;
  }
  for (int q = t; q < ni * nb; q += kLayoutThreads) {
    const int r = q / nb, b = q - r * nb;
    const ChanGroup gq = chan_group(b0 + b, B, gmax);
    ALMT[(size_t)gq.g0 * (nalm + kCoefPad) + (i0 + r) * gq.w + (b0 + b - gq.g0)] = tile[r][b];
  }
}

// Up to 4 channels: no transpose worth an LDS tile, a thread keeps its index's
// channels, kLayoutRows / B indices in flight (FP64 L 4095 B 1 145 -> 51 us,
// 6.6 TB/s with part of it from the last-level cache).
constexpr int kLayoutRows = 4;

template <typename T, int B>
__global__ void __launch_bounds__(kLayoutThreads)
    k_alm_in_few(int L, int gmax, const cplx<T> *__restrict__ alm, const double *__restrict__ coefC,
                 cplx<T> *__restrict__ ALMT, double s, double f0, double fm) {
  constexpr int U = kLayoutRows / B;
  const size_t nalm = nalm_of(L);
  const size_t i0 = (size_t)blockIdx.x * (kLayoutThreads * U) + threadIdx.x;
  cplx<T> v[U][B];
  double c[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t idx = i0 + u * kLayoutThreads;
    if (idx < nalm) {
      c[u] = coefC[idx];
#pragma unroll
      for (int b = 0; b < B; ++b) v[u][b] = alm[b * nalm + idx];
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t idx = i0 + u * kLayoutThreads;
    if (idx < nalm) {
      const bool m0 = idx <= (size_t)L;
      const double g = s * (m0 ? f0 : fm) * c[u];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const ChanGroup gr = chan_group(b, B, gmax);
        ALMT[(size_t)gr.g0 * (nalm + kCoefPad) + idx * gr.w + (b - gr.g0)] = scaled<T>(v[u][b], g, m0);
      }
    }
  }
}

template <typename T>
hipError_t launch_alm_in(int L, int B, int gmax, const cplx<T> *alm, const double *coefC, cplx<T> *ALMT, double s,
                         double f0, double fm, hipStream_t st) {
  const size_t nalm = nalm_of(L);
  auto blocks = [&](size_t rows) { return (unsigned)((nalm + rows - 1) / rows); };
  auto few = [&](auto kern, int b) {
    hipLaunchKernelGGL(kern, dim3(blocks((size_t)kLayoutThreads * (kLayoutRows / b))), dim3(kLayoutThreads), 0, st, L,
                       gmax, alm, coefC, ALMT, s, f0, fm);
  };
  switch (B) {
    case 1: few(k_alm_in_few<T, 1>, 1); break;
    case 2: few(k_alm_in_few<T, 2>, 2); break;
    case 3: few(k_alm_in_few<T, 3>, 3); break;
    case 4: few(k_alm_in_few<T, 4>, 4); break;
    default:
      hipLaunchKernelGGL(k_alm_in<T>,
                         dim3(blocks(kLayoutThreads) * ((unsigned)(B + kLayoutChannels - 1) / kLayoutChannels)),
                         dim3(kLayoutThreads), 0, st, L, B, gmax, alm, coefC, ALMT, s, f0, fm);
  }
  return hipGetLastError();
}

template hipError_t launch_alm_in<double>(int, int, int, const double2 *, const double *, double2 *, double, double,
                                          double, hipStream_t);
template hipError_t launch_alm_in<float>(int, int, int, const float2 *, const double *, float2 *, double, double,
                                         double, hipStream_t);

}  // namespace shtx
