// |M|^2 of the processes with few flows (up to three gluons) in one launch.
//
// A lane evaluates one event for one mirror pair of helicities (flipping every helicity
// conjugates the amplitudes up to a sign, so both have the same colour form: it counts
// once per good helicity of the pair).  A workgroup holds 16 events with all their
// pairs, reads the caller's momenta as they are, and sums the pairs in order: no
// structure-of-arrays copy, no partial sums in memory, no second and third launch.  Bound
// by the latency of one lane's chain of FP64 operations (g g -> t t~ g: 512 registers,
// one wave a SIMD); 16 events a workgroup spread 8192 events over two rounds of the
// compute units, and the smallest calls over several of them.  On an MI355X, against the
// three launches of the one-lane kernel: 64 events of g g -> t t~ 4.5 us (11.8), 8192 of
// g g -> t t~ g with running coupling 16.2 us (47.8).
#pragma once
#include "me_device.h"
#include "me_pair_desc.h"

namespace me {

constexpr int kPairEvents = 16;

template <class P>
struct PairShape {
  static constexpr int PAIRS = 1 << (P::NPAR - 1);          // at most
  static constexpr int THREADS = kPairEvents * PAIRS;
};

template <class P>
__global__ void __launch_bounds__(PairShape<P>::THREADS)
pair_kernel(const double* __restrict__ mom, int64_t n, double g, double mt, const int* __restrict__ pairs, int npair,
            const double* __restrict__ alphas, double* __restrict__ out, double scale) {
  constexpr int EV = kPairEvents;
  __shared__ double form[PairShape<P>::PAIRS][EV];
  const int t = threadIdx.x, k = t / EV;
  const int64_t e = (int64_t)blockIdx.x * EV + t % EV;
  if (e < n && k < npair) {
    const int pr = pairs[k], h = pr & 0xffff;
    double p[P::NPAR][4];
    const double* m = mom + e * (P::NPAR * 4);
#pragma unroll
    for (int q = 0; q < P::NPAR; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u) p[q][u] = m[4 * q + u];
    if (alphas) g = sqrt(4.0 * 3.14159265358979323846 * alphas[e]);
    int lam[P::NPAR];
#pragma unroll
    for (int q = 0; q < P::NPAR; ++q) lam[q] = ((h >> (P::NPAR - 1 - q)) & 1) ? 1 : -1;
    cx jamp[P::NCOL];
#pragma unroll
    for (int i = 0; i < P::NCOL; ++i) jamp[i] = cx{0.0, 0.0};
    P::amplitudes(p, lam, g, mt, jamp);
    form[k][t % EV] = (double)(pr >> 16) * P::colour_sum(jamp);
  }
  __syncthreads();
  if (t < EV && e < n) {
    double sum = 0.0;
    for (int i = 0; i < npair; ++i) sum += form[i][t];   // fixed order
    out[e] = scale * sum;
  }
}

// A launch has fewer than 2^32 threads: larger batches take several (of 5.4e8 events of
// g g -> t t~, 2.7e8 of g g -> t t~ g).
template <class P>
hipError_t launch_pair(const PairArgs& a) {
  constexpr int64_t THREADS = PairShape<P>::THREADS, most = 0xffffffffll / THREADS * kPairEvents;
  if (a.npair < 0 || a.npair > PairShape<P>::PAIRS) return hipErrorInvalidValue;
  for (int64_t off = 0; off < a.n; off += most) {
    const int64_t n = a.n - off < most ? a.n - off : most;
    const dim3 grid((unsigned)((n + kPairEvents - 1) / kPairEvents));
    hipLaunchKernelGGL(pair_kernel<P>, grid, dim3((unsigned)THREADS), 0, a.stream, a.mom + off * (P::NPAR * 4), n, a.g, a.mt, a.pairs, a.npair,
                       a.alphas ? a.alphas + off : nullptr, a.out + off, a.scale);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace me
