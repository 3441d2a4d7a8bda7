// Two-sided colour-ordered recursion with helicity recycling: the dual amplitudes of
// one event, four to six gluons, by one workgroup (launch variants 4 and 5).  The
// recursion, vertices and conventions are those of me_bg.h and me_bgh.h; what is
// different is how much of it is formed, and where.
//
//  * Mirror images.  Flipping every helicity turns each dual amplitude into its
//    complex conjugate times a sign common to all orderings, so both helicities have
//    the same |M|^2 (and the same |J_c|^2 in every flow).  Gluon 0 keeps helicity -;
//    a row stands for itself and its mirror image.  This halves the variants of
//    everything that holds gluon 0, and the rows of the colour form.
//  * The orderings of a gluon current are not independent:
//    J(alpha, x, beta) = (-1)^|alpha| sum J(x, rho) over the shuffles rho of reversed
//    alpha with beta (Kleiss-Kuijf for currents).  Currents of length 4 and more are
//    formed only for the (L-1)! orderings with their lowest gluon first and expanded
//    where they are used (1 .. 3 terms for length 4, up to 6 for length 5).
//  * The quark line is cut at the block that holds position M = 2 (six gluons: 3):
//      A(sigma) = Q.J(sigma) + i g sum_{i <= M < j, (i,j) != (0,N)}
//                 R(sigma[:i]) gamma.J(sigma[i:j]) C(sigma[j:]),
//    R(p) the row spinor of the top end (me_bg.h), C(s) the column spinor of the
//    antitop end, C(()) = v, C(s) = S(p3 - P(rest)) sum_j i g gamma.J(s[:j]) C(s[j:]).
//    Only R and C of at most two gluons are stored; the sums over i belong to prefixes of
//    sigma, so a work item = (prefix of length N-1, its helicities) forms
//    X_j = sum_i R gamma.J(sigma[i:j]) for j < N once for both helicities of the last
//    gluon.
//  * Q.J(sigma) needs the currents of length N only contracted: they are formed for
//    the orderings that start with gluon 0, and their contractions with the four
//    Q = i g ubar gamma v expanded (1 .. 10 terms).
//
// FP64 operations per event with all helicities (flops.bgm_event; counted by running
// this code on a counting double): 3.47e6 for g g -> t t~ g g g against 19.1e6 of the
// one-sided kernel of me_bgh.h, 0.27e6 against 1.24e6 for g g -> t t~ g g, 59.5e6 for
// g g -> t t~ g g g g.  Bound by the issue of FP64 vector instructions: 40.4e3 vector
// instructions an event, four cycles each on one of a compute unit's four SIMDs, are 68 %
// of the 59.3e3 cycles that an event takes a compute unit (five gluons); the rest is
// latency of LDS and of the work-item records between barriers.  On an MI355X, FP64
// colour, against the one-sided kernel on the same card: 262144 g g -> t t~ g g g 27.7 ms
// (149.7), 524288 g g -> t t~ g g 5.5 ms (18.8), 1000 g g -> t t~ g g g 0.12 ms (0.63);
// split FP16 colour, 100003 g g -> t t~ g g g 11.5 ms (51.0); six gluons against the
// one-row kernel of me_bg.h, 4096 events 11.1 ms (284).  Cards differ: another took 30.3,
// 6.0, 0.13, 12.6 and 11.5 ms (152, 20.4, 0.63, 55.5 and 285).
//
// Frame of an event in LDS: slots of four complex numbers, component-major (component
// c of slot s is the 16-byte element c NS + s), so that the 16-byte reads of lanes on
// consecutive helicity variants fall on consecutive banks.
#pragma once
#include "me_bgh.h"
#include "me_bgm_shape.h"
#ifdef __HIPCC__
#include "colour_mfma.h"
#endif

namespace me {

struct alignas(16) cx16 {
  double r, i;
};

// A work item's record: word w of item i at t[w items + i], two 16-bit fields a word,
// held in registers.
template <int FIELDS>
struct BgmRec {
  static constexpr int W = (FIELDS + 1) / 2;
  uint32_t w[W];
  __device__ __forceinline__ BgmRec() {}
  __device__ __forceinline__ BgmRec(const uint32_t* t, int items, int i) { read(t, items, i); }
  __device__ __forceinline__ void read(const uint32_t* t, int items, int i) {
#pragma unroll
    for (int k = 0; k < W; ++k) w[k] = t[k * items + i];
  }
  __device__ __forceinline__ int operator()(int f) const {
    return (f & 1) ? (int)(w[f >> 1] >> 16) : (int)(w[f >> 1] & 0xffffu);
  }
};

// The vector at byte offset off, read where the program says so: an opaque copy of the
// offset keeps a vector that is used twice from being held in registers in between
// (the sums below would hold more vectors than there are registers).
template <int N>
__device__ __forceinline__ void bgm_load(const double* F, int off, cx* v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(off));
#endif
  const char* p = reinterpret_cast<const char*>(F) + off;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const cx16 x = *reinterpret_cast<const cx16*>(p + c * BgmShape<N>::NS * 16);
    v[c] = cx{x.r, x.i};
  }
}

template <int N>
__device__ __forceinline__ void bgm_store(double* F, int slot, const cx* v) {
  char* p = reinterpret_cast<char*>(F) + 16 * slot;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    *reinterpret_cast<cx16*>(p + c * BgmShape<N>::NS * 16) = cx16{v[c].r, v[c].i};
}

// A value that every lane of the wave holds, in scalar registers.
__device__ __forceinline__ double bgm_uniform(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readfirstlane((int)b), hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
#else
  return x;
#endif
}

template <int N>
__device__ __forceinline__ void bgm_load_uniform(const double* F, int slot, cx* v) {
  bgm_load<N>(F, 16 * slot, v);
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = cx{bgm_uniform(v[c].r), bgm_uniform(v[c].i)};
}

// q = p3 - P(mask), the top momentum after a row spinor has absorbed the subset
template <int N>
__device__ __forceinline__ void bgm_topmom(const double* F, int mask, double* q) {
#pragma unroll
  for (int u = 0; u < 4; ++u) q[u] = F[BgmShape<N>::MOFF + 8 + u] - F[BgmShape<N>::PSOFF + 4 * mask + u];
}

template <int N>
__device__ __forceinline__ void bgm_mom(const double* F, int mask, double* p) {
#pragma unroll
  for (int u = 0; u < 4; ++u) p[u] = F[BgmShape<N>::PSOFF + 4 * mask + u];
}

// Sum of stored currents with a common sign (an expansion of me_bgm_tables.h): off(t) the
// address of term t, info = their number (1 or 3 for length 4), bit 15 = negative.
template <int N, typename Off>
__device__ __forceinline__ void bgm_expand(const double* F, int info, Off off, cx* v) {
  const int cnt = info & 0x7fff;
  bgm_load<N>(F, off(0), v);
  if (cnt > 1) {
    cx a[4], b[4];
    bgm_load<N>(F, off(1), a);
    bgm_load<N>(F, off(2), b);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = (v[c] + a[c]) + b[c];
  }
  const double s = (info & 0x8000) ? -1.0 : 1.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = s * v[c];
}

// The same for currents of length 5, which six gluons keep in memory (1, 4 or 6 terms).
__device__ __forceinline__ void bgm_load5(const cx16* j5, int k, cx* v) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const cx16 x = j5[c * BgmShape<6>::CV(5) + k];
    v[c] = cx{x.r, x.i};
  }
}
template <typename Var>
__device__ __forceinline__ void bgm_expand5(const cx16* j5, int info, Var var, cx* v) {
  const int cnt = info & 0x7fff;
  // the terms in two steps, the loads of each in flight together
  bgm_load5(j5, var(0), v);
  if (cnt > 1) {
    cx a[3][4];
#pragma unroll
    for (int t = 0; t < 3; ++t) bgm_load5(j5, var(1 + t), a[t]);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = v[c] + a[t][c];
  }
  if (cnt > 4) {
    cx a[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) bgm_load5(j5, var(4 + t), a[t]);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = v[c] + a[t][c];
  }
  const double s = (info & 0x8000) ? -1.0 : 1.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = s * v[c];
}

// gamma.J in blocks (see bgh_rg_acc)
struct BgmSlash {
  cx jp, jm, js, jd;
};
__device__ __forceinline__ BgmSlash bgm_slash(const cx* j) {
  const cx ij2 = times_i(j[2]);
  return BgmSlash{j[0] + j[3], j[0] - j[3], j[1] + ij2, j[1] - ij2};
}
// acc = r . gamma.J, and accumulated
__device__ __forceinline__ void bgm_rg(const cx* r, const BgmSlash& s, cx* acc) {
  acc[0] = fma(r[2] * s.jp, r[3], s.js);
  acc[1] = fma(r[2] * s.jd, r[3], s.jm);
  acc[2] = fma(r[0] * s.jm, r[1], -s.js);
  acc[3] = fma(r[0] * (-s.jd), r[1], s.jp);
}
__device__ __forceinline__ void bgm_rg_acc(const cx* r, const BgmSlash& s, cx* acc) {
  acc[0] = fma(fma(acc[0], r[2], s.jp), r[3], s.js);
  acc[1] = fma(fma(acc[1], r[2], s.jd), r[3], s.jm);
  acc[2] = fma(fma(acc[2], r[0], s.jm), r[1], -s.js);
  acc[3] = fma(fma(acc[3], r[0], -s.jd), r[1], s.jp);
}
// acc += gamma.J c
__device__ __forceinline__ void bgm_gc_acc(const BgmSlash& s, const cx* c, cx* acc) {
  acc[0] = fma(fma(acc[0], s.jm, c[2]), -s.jd, c[3]);
  acc[1] = fma(fma(acc[1], -s.js, c[2]), s.jp, c[3]);
  acc[2] = fma(fma(acc[2], s.jp, c[0]), s.jd, c[1]);
  acc[3] = fma(fma(acc[3], s.js, c[0]), s.jm, c[1]);
}
// out = i (qslash + m) f . (i g acc), f = 1 / (q^2 - m^2): the column form of bgh_prop
__device__ __forceinline__ void bgm_prop_col(const cx* a, const double* q, double f, double m, double g, cx* out) {
  const double sc = -g * f;
  const double qp = q[0] + q[3], qm = q[0] - q[3];
  const cx o0 = cx{m * a[0].r + qm * a[2].r - q[1] * a[3].r - q[2] * a[3].i,
                   m * a[0].i + qm * a[2].i - q[1] * a[3].i + q[2] * a[3].r};
  const cx o1 = cx{m * a[1].r - q[1] * a[2].r + q[2] * a[2].i + qp * a[3].r,
                   m * a[1].i - q[1] * a[2].i - q[2] * a[2].r + qp * a[3].i};
  const cx o2 = cx{m * a[2].r + qp * a[0].r + q[1] * a[1].r + q[2] * a[1].i,
                   m * a[2].i + qp * a[0].i + q[1] * a[1].i - q[2] * a[1].r};
  const cx o3 = cx{m * a[3].r + q[1] * a[0].r - q[2] * a[0].i + qm * a[1].r,
                   m * a[3].i + q[1] * a[0].i + q[2] * a[0].r + qm * a[1].i};
  out[0] = sc * o0;
  out[1] = sc * o1;
  out[2] = sc * o2;
  out[3] = sc * o3;
}

// Set-up: momentum sums and propagators of gluon subset i,
template <int N>
__device__ __forceinline__ void bgm_setup_subset(double* F, double mt, int i) {
  using S = BgmShape<N>;
  const double(*p)[4] = reinterpret_cast<const double(*)[4]>(F + S::MOFF);
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = 0; b < N; ++b)
    if ((i >> b) & 1) {
      const int q = b < 2 ? b : b + 2;
      const double sg = b < 2 ? 1.0 : -1.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += sg * p[q][u];
    }
#pragma unroll
  for (int u = 0; u < 4; ++u) F[S::PSOFF + 4 * i + u] = s[u];
  F[S::GIOFF + i] = __builtin_popcount(i) >= 2 ? 1.0 / (s[0] * s[0] - s[1] * s[1] - s[2] * s[2] - s[3] * s[3])
                                                 : 0.0;
  const double* p3 = p[2];
  double q[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) q[u] = p3[u] - s[u];
  F[S::TFOFF + i] = 1.0 / (q[0] * q[0] - q[1] * q[1] - q[2] * q[2] - q[3] * q[3] - mt * mt);
}
// polarisation vector of variant j of length 1 (gluon 0: helicity - alone; then gluon,
// helicity),
template <int N>
__device__ __forceinline__ void bgm_setup_gluon(double* F, int j) {
  using S = BgmShape<N>;
  const int b = (j + 1) >> 1, bit = j == 0 ? 0 : (j + 1) & 1;
  const int q = b < 2 ? b : b + 2;
  cx e[4];
  ext_gluon(F + S::MOFF + 4 * q, bit ? 1 : -1, b >= 2, e);
  bgm_store<N>(F, S::cslot(1) + j, e);
}
// ubar (j = 0, 1) and v (j = 2, 3) of both helicities,
template <int N>
__device__ __forceinline__ void bgm_setup_spinor(double* F, double mt, int j) {
  using S = BgmShape<N>;
  cx w[4];
  if (j < 2) ext_ubar(F + S::MOFF + 8, j ? 1 : -1, mt, w);
  else ext_v(F + S::MOFF + 12, (j - 2) ? 1 : -1, mt, w);
  bgm_store<N>(F, S::UBS + j, w);
}
// and, once these are stored, Q of quark helicity pair uv.
template <int N>
__device__ __forceinline__ void bgm_setup_q(double* F, int uv) {
  using S = BgmShape<N>;
  cx ub[4], v[4], w[4];
  bgm_load<N>(F, 16 * (S::UBS + (uv >> 1)), ub);
  bgm_load<N>(F, 16 * (S::VS + (uv & 1)), v);
  line_current(ub, v, F[S::GOFF], w);
  bgm_store<N>(F, S::QS + uv, w);
}

// A point that the sums in v (four complex numbers) have to have reached before what
// follows is read: left alone, the compiler reads every vector of the unrolled sums
// below first and adds them up last, and spills.
__device__ __forceinline__ void bgm_pin(cx* v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(""
               : "+v"(v[0].r), "+v"(v[0].i), "+v"(v[1].r), "+v"(v[1].i), "+v"(v[2].r), "+v"(v[2].i), "+v"(v[3].r),
                 "+v"(v[3].i)
               :
               :);
#endif
}

// acc += V(a, pa, b, P - pa), the three-gluon vertex of bg_v3 with the sum P given.
__device__ __forceinline__ void bgm_v3(const cx* a, const double* pa, const cx* b, const double* P, cx* acc) {
  double kma[4], pbk[4], pamb[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    kma[u] = -(P[u] + pa[u]);
    pbk[u] = 2.0 * P[u] - pa[u];
    pamb[u] = 2.0 * pa[u] - P[u];
  }
  const cx c1 = rdot(kma, b);
  const cx c2 = vdot(a, b);
  const cx c3 = rdot(pbk, a);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    cx v = fma(acc[u], a[u], c1);
    v = fma(v, b[u], c3);
    acc[u] = cx{v.r + pamb[u] * c2.r, v.i + pamb[u] * c2.i};
  }
}

// The fields of a current's record list its sub-currents by length, then by start.
template <int L>
__device__ __forceinline__ constexpr int bgm_field(int start, int len) {
  int f = 0;
  for (int x = 1; x < len; ++x) f += L - x + 1;
  return f + start;
}

// Current of length L = 2 .. 6 over the subset pm[L] (pm[j]: its first j gluons):
// head(j, v) reads the sub-current of the first j gluons, mid(j, l, v) that of gluons
// j .. l - 1, tail(v) that of the last L - 1.  The tails that several splits share
// stay in registers, and each vector is asked for one vertex ahead of its use (two
// waves per SIMD do not hide the latency of LDS behind each other).
template <int N, int L, typename Head, typename Mid, typename Tail>
__device__ __forceinline__ void bgm_splits(const double* F, const int* pm, Head head, Mid mid, Tail tail, cx* out) {
  using S = BgmShape<N>;
  cx a3[4], a4[4], A[4], B[4], T[L][4];   // T[l]: gluons l .. L - 1, l >= 2
  double P[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) a3[c] = a4[c] = cx{0.0, 0.0};
  head(1, A);
  tail(B);
  bgm_mom<N>(F, pm[L], P);
#pragma unroll
  for (int l = 2; l < L; ++l) mid(l, L, T[l]);
#pragma unroll
  for (int j = 1; j < L; ++j) {
    cx M[4], X[4];
    double pa[4];
    bgm_mom<N>(F, pm[j], pa);
    if (j + 1 < L) mid(j, j + 1, M);
    bgm_v3(A, pa, j == 1 ? B : T[j], P, a3);
    bgm_pin(a3);
#pragma unroll
    for (int l = j + 1; l < L; ++l) {
      if (l + 1 < L) mid(j, l + 1, X);
      else head(j + 1, X);
      bg_v4(A, M, T[l], a4);
      bgm_pin(a4);
      bgh_copy(X, l + 1 < L ? M : A);
    }
  }
  const double g = F[S::GOFF], inv = F[S::GIOFF + pm[L]];
  const double f3 = -g * inv, f4 = -g * g * inv;
#pragma unroll
  for (int c = 0; c < 4; ++c) out[c] = L == 2 ? f3 * a3[c] : f3 * a3[c] + f4 * a4[c];
}

// Current of length L = 2 .. 4 from its record: field bgm_field<L>(a, len) the address
// of the sub-current of len gluons from a, then the prefix masks and its own.
template <int N, int L, typename Rec>
__device__ __forceinline__ void bgm_current(const double* F, const Rec& rec, cx* out) {
  constexpr int M = bgm_field<L>(0, L);
  int pm[L + 1];
#pragma unroll
  for (int j = 1; j <= L; ++j) {
    const int w = rec(M + (j - 1) / 2);
    pm[j] = ((j - 1) & 1) ? w >> 8 : w & 0xff;
  }
  bgm_splits<N, L>(
      F, pm, [&](int j, cx* v) { bgm_load<N>(F, rec(bgm_field<L>(0, j)), v); },
      [&](int j, int l, cx* v) { bgm_load<N>(F, rec(bgm_field<L>(j, l - j)), v); },
      [&](cx* v) { bgm_load<N>(F, rec(bgm_field<L>(1, L - 1)), v); }, out);
}

// Canonical current of length 5 from its record: as above for lengths 1 .. 3, then the
// prefix of length 4, the expansion of the last four gluons (three addresses, info), and
// the masks.
template <int N>
__device__ __forceinline__ void bgm_current5(const double* F, const BgmRec<BgmShape<N>::F5>& rec, cx* out) {
  constexpr int L = 5, K = bgm_field<L>(0, 4);
  const int w0 = rec(K + 5), w1 = rec(K + 6);
  const int pm[6] = {0, w0 & 0xff, w0 >> 8, w1 & 0xff, w1 >> 8, rec(K + 7)};
  bgm_splits<N, L>(
      F, pm, [&](int j, cx* v) { bgm_load<N>(F, rec(j < 4 ? bgm_field<L>(0, j) : K), v); },
      [&](int j, int l, cx* v) { bgm_load<N>(F, rec(bgm_field<L>(j, l - j)), v); },
      [&](cx* v) { bgm_expand<N>(F, rec(K + 4), [&](int t) { return rec(K + 1 + t); }, v); }, out);
}

// Current of six gluons, ordering that starts with gluon 0: lengths 1 .. 3, the prefix of
// length 4, the expansions of gluons 1 .. 4 and 2 .. 5, the prefix of length 5 and the
// expansion of the last five (variant numbers), the masks.
__device__ __forceinline__ void bgm_current6(const double* F, const cx16* j5, const BgmRec<BgmShape<6>::F6>& rec,
                                             cx* out) {
  constexpr int N = 6, L = 6, K = bgm_field<L>(0, 4);
  const int w0 = rec(K + 17), w1 = rec(K + 18);
  const int pm[7] = {0, w0 & 0xff, w0 >> 8, w1 & 0xff, w1 >> 8, rec(K + 19), (1 << N) - 1};
  bgm_splits<N, L>(
      F, pm,
      [&](int j, cx* v) {
        if (j < 5) bgm_load<N>(F, rec(j < 4 ? bgm_field<L>(0, j) : K), v);
        else bgm_load5(j5, rec(K + 9), v);
      },
      [&](int j, int l, cx* v) {
        if (l - j < 4) bgm_load<N>(F, rec(bgm_field<L>(j, l - j)), v);
        else bgm_expand<N>(F, rec(K + 4 * j), [&](int t) { return rec(K + 4 * j - 3 + t); }, v);
      },
      [&](cx* v) { bgm_expand5(j5, rec(K + 16), [&](int t) { return rec(K + 10 + t); }, v); }, out);
}

// Row spinors of one gluon (variant it, both top helicities) and column spinors of one
// gluon (both antitop helicities): the other end's momentum follows from all the rest.
template <int N>
__device__ __forceinline__ void bgm_row1_item(double* F, const uint32_t* tabs, double mt, int it, int u) {
  using S = BgmShape<N>;
  const int m = BgmRec<S::F1>(tabs + S::T1, S::V(1), it)(0);
  double q[4];
  bgm_topmom<N>(F, m, q);
  cx r[4], j[4], acc[4], out[4];
  bgm_load<N>(F, 16 * (S::UBS + u), r);
  bgm_load<N>(F, 16 * (S::cslot(1) + it), j);
  bgm_rg(r, bgm_slash(j), acc);
  bgh_prop(acc, q, F[S::TFOFF + m], mt, F[S::GOFF], out);
  bgm_store<N>(F, S::R1S + u * S::V(1) + it, out);
}
template <int N>
__device__ __forceinline__ void bgm_col1_item(double* F, const uint32_t* tabs, double mt, int it, int v) {
  using S = BgmShape<N>;
  const int m = ((1 << N) - 1) ^ BgmRec<S::F1>(tabs + S::T1, S::V(1), it)(0);
  double q[4];
  bgm_topmom<N>(F, m, q);
  cx c[4], j[4], acc[4], out[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = cx{0.0, 0.0};
  bgm_load<N>(F, 16 * (S::VS + v), c);
  bgm_load<N>(F, 16 * (S::cslot(1) + it), j);
  bgm_gc_acc(bgm_slash(j), c, acc);
  bgm_prop_col(acc, q, F[S::TFOFF + m], mt, F[S::GOFF], out);
  bgm_store<N>(F, S::C1S + v * S::V(1) + it, out);
}
// Row and column spinors of two gluons a, b (record: J(a), J(b), J(ab), R(a), C(b), mask).
template <int N>
__device__ __forceinline__ void bgm_row2_item(double* F, const uint32_t* tabs, double mt, int it, int u) {
  using S = BgmShape<N>;
  const BgmRec<S::FR2> rec(tabs + S::TR2, S::V(2), it);
  const int m = rec(5);
  double q[4];
  bgm_topmom<N>(F, m, q);
  cx r[4], j[4], acc[4], out[4];
  bgm_load<N>(F, 16 * (S::UBS + u), r);
  bgm_load<N>(F, rec(2), j);
  bgm_rg(r, bgm_slash(j), acc);
  bgm_load<N>(F, rec(3) + 16 * u * S::V(1), r);
  bgm_load<N>(F, rec(1), j);
  bgm_rg_acc(r, bgm_slash(j), acc);
  bgh_prop(acc, q, F[S::TFOFF + m], mt, F[S::GOFF], out);
  bgm_store<N>(F, S::R2S + u * S::V(2) + it, out);
}
template <int N>
__device__ __forceinline__ void bgm_col2_item(double* F, const uint32_t* tabs, double mt, int it, int v) {
  using S = BgmShape<N>;
  const BgmRec<S::FR2> rec(tabs + S::TR2, S::V(2), it);
  const int m = ((1 << N) - 1) ^ rec(5);
  double q[4];
  bgm_topmom<N>(F, m, q);
  cx c[4], j[4], acc[4], out[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = cx{0.0, 0.0};
  bgm_load<N>(F, 16 * (S::VS + v), c);
  bgm_load<N>(F, rec(2), j);
  bgm_gc_acc(bgm_slash(j), c, acc);
  bgm_load<N>(F, rec(4) + 16 * v * S::V(1), c);
  bgm_load<N>(F, rec(0), j);
  bgm_gc_acc(bgm_slash(j), c, acc);
  bgm_prop_col(acc, q, F[S::TFOFF + m], mt, F[S::GOFF], out);
  bgm_store<N>(F, S::C2S + v * S::V(2) + it, out);
}

// Q.J of canonical ordering it >> (N-1), gluon helicities it & (NGH - 1), for the four
// quark helicity pairs, from the item's record, to qj [ordering][2 u + v][gh] (j5: the
// currents of length 5 of six gluons).
template <int N>
__device__ __forceinline__ void bgm_qj_item(const double* F, const BgmRec<BgmShape<N>::FQ>& rec, const cx16* j5,
                                            cx16* qj, int it) {
  using S = BgmShape<N>;
  cx j[4];
  if constexpr (N == 5)
    bgm_current5<N>(F, rec, j);
  else if constexpr (N == 6)
    bgm_current6(F, j5, rec, j);
  else
    bgm_current<N, 4>(F, rec, j);
  cx16* dst = qj + (it >> (N - 1)) * S::NROW + (it & (S::NGH - 1));
#pragma unroll
  for (int uv = 0; uv < 4; ++uv) {
    cx q[4];
    bgm_load_uniform<N>(F, S::QS + uv, q);
    const cx x = vdot(q, j);
    dst[uv * S::NGH] = cx16{x.r, x.i};
  }
}

// The records of one prefix item.  An item with one leaf taken as one with two forms
// its leaf twice.
template <int N, int LEAVES>
struct BgmPrefix {
  using S = BgmShape<N>;
  BgmRec<S::FP> rec;
  BgmRec<S::FL> leaf[LEAVES];
  __device__ __forceinline__ void read(const uint32_t* tabs, int it) {
    rec.read(tabs + S::TP, S::VP, it);
    leaf[0].read(tabs + S::TL0, S::VP, it);
    if constexpr (LEAVES == 2) {
      const bool two = it < S::VP2;
      leaf[1].read(tabs + (two ? S::TL1 : S::TL0), two ? S::VP2 : S::VP, it);
    }
  }
};

// ubar and v of both helicities, uniform over the workgroup's event: scalar registers.
struct BgmEnds {
  cx ub[2][4], v[2][4];
};
template <int N>
__device__ __forceinline__ void bgm_ends(const double* F, BgmEnds& e) {
  using S = BgmShape<N>;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    bgm_load_uniform<N>(F, S::UBS + u, e.ub[u]);
    bgm_load_uniform<N>(F, S::VS + u, e.v[u]);
  }
}

// One prefix item: the amplitudes of its ordering for the LEAVES helicities of the last
// gluon and the four quark helicity pairs; row (2 u + v) NGH + gh of jt [2 NCOL][RS].
// Each row spinor is read once for all the sums it enters.
template <int N, int RS, int LEAVES, typename Note>
__device__ __forceinline__ void bgm_prefix_item(const double* F, const BgmPrefix<N, LEAVES>& p, const BgmEnds& ends,
                                                double* __restrict__ jt, Note note) {
  using S = BgmShape<N>;
  const BgmRec<S::FP>& rec = p.rec;
  const BgmRec<S::FL>* leaf = p.leaf;
  constexpr int FC = N == 5 ? 11 : 5;   // column field, then the expansion of Q.J
  const double g = F[S::GOFF];
  // X_3, X_4 (five gluons) and X_N of each leaf, both top helicities
  cx x3[2][4], x4[2][4], xn[LEAVES][2][4];
  {
    cx j[4];
    bgm_load<N>(F, rec(4), j);
    const BgmSlash s = bgm_slash(j);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bgm_rg(ends.ub[u], s, x3[u]);
      bgm_pin(x3[u]);
    }
  }
  if constexpr (N == 5) {
    cx j[4];
    bgm_expand<N>(F, rec(10), [&](int t) { return rec(7 + t); }, j);
    const BgmSlash s = bgm_slash(j);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bgm_rg(ends.ub[u], s, x4[u]);
      bgm_pin(x4[u]);
    }
  }
  // the terms of one stored row spinor: R of one gluon, then of two
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    cx j[4], r[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) bgm_load<N>(F, rec(k) + 16 * u * S::V(k + 1), r[u]);
    bgm_load<N>(F, rec(k ? 2 : 3), j);
    {
      const BgmSlash s = bgm_slash(j);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bgm_rg_acc(r[u], s, x3[u]);
        bgm_pin(x3[u]);
      }
    }
    if constexpr (N == 5) {
      bgm_load<N>(F, rec(k ? 5 : 6), j);
      const BgmSlash s = bgm_slash(j);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bgm_rg_acc(r[u], s, x4[u]);
        bgm_pin(x4[u]);
      }
    }
#pragma unroll
    for (int h = 0; h < LEAVES; ++h) {
      if (N == 5 && k == 0)
        bgm_expand<N>(F, leaf[h](3), [&](int t) { return leaf[h](t); }, j);
      else
        bgm_load<N>(F, leaf[h](N == 5 ? 4 : k), j);
      const BgmSlash s = bgm_slash(j);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (k == 0) bgm_rg(r[u], s, xn[h][u]);
        else bgm_rg_acc(r[u], s, xn[h][u]);
        bgm_pin(xn[h][u]);
      }
    }
  }
  const int col = rec(FC), qinfo = rec(FC + 1 + S::QKK);
  const int qn = qinfo & 0x7fff;
  const double qs = (qinfo & 0x8000) ? -1.0 : 1.0;
#pragma unroll
  for (int h = 0; h < LEAVES; ++h) {
    const int gh = leaf[h](N == 5 ? 7 : 3);
    // Q.J(sigma), expanded over the canonical orderings
    cx a[4];
    {
      const char* q = reinterpret_cast<const char*>(F + S::QJOFF) + 16 * gh;
#pragma unroll
      for (int uv = 0; uv < 4; ++uv) a[uv] = cx{0.0, 0.0};
#pragma unroll
      for (int t = 0; t < S::QKK; ++t) {
        if (t < qn) {
          const char* qt = q + rec(FC + 1 + t) * (16 * S::NROW);
#pragma unroll
          for (int uv = 0; uv < 4; ++uv) {
            const cx16 x = *reinterpret_cast<const cx16*>(qt + 16 * uv * S::NGH);
            a[uv] = a[uv] + cx{x.r, x.i};
          }
        }
      }
    }
    // i g times the sums over j: X_N v + X_{N-1} C(last) (+ X_{N-2} C(last two))
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      cx c[4], w[2];
      bgm_load<N>(F, leaf[h](N == 5 ? 6 : 2) + 16 * v * S::V(1), c);
#pragma unroll
      for (int u = 0; u < 2; ++u) w[u] = sdot(xn[h][u], ends.v[v]) + sdot(N == 5 ? x4[u] : x3[u], c);
      if constexpr (N == 5) {
        bgm_load<N>(F, leaf[h](5) + 16 * v * S::V(2), c);
#pragma unroll
        for (int u = 0; u < 2; ++u) w[u] = w[u] + sdot(x3[u], c);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const cx q = a[2 * u + v];
        const cx y = cx{qs * q.r - g * w[u].i, qs * q.i + g * w[u].r};   // Q.J + i g w
        const int row = (2 * u + v) * S::NGH + gh;
        jt[(int64_t)(2 * col) * RS + row] = y.r;
        jt[(int64_t)(2 * col + 1) * RS + row] = y.i;
        note(row, y.r, y.i);
      }
    }
  }
}

template <int K>
struct BgmInt {
  static constexpr int value = K;
};

// The same for six gluons, cut at position 3: the row spinor of three gluons is formed
// here, R(sigma[:3]) = S . i g X_3, currents of length 5 and Q.J come from memory, and
// each leaf is formed after the other (register space).  Two thirds of an event's time,
// bound by the latency of those loads at two waves a SIMD: the terms of an expansion are
// loaded in steps that the lanes of a wave mostly share, several in flight (4096 events
// 11.1 ms; one after the other, and the colour form's loads not ahead, 12.5).
template <int RS>
__device__ __forceinline__ void bgm_prefix6_item(const double* F, const uint32_t* tabs,
                                                 const BgmRec<BgmShape<6>::FP>& rec, const BgmEnds& ends, double mt,
                                                 const cx16* j5, const cx16* qj, double* __restrict__ jt, int it) {
  constexpr int N = 6;
  using S = BgmShape<N>;
  constexpr int FC = 26;
  const double g = F[S::GOFF];
  cx r3[2][4], x4[2][4], x5[2][4];
  auto add = [&](cx(*x)[4], const cx* j, const cx(*r)[4], bool first) {
    const BgmSlash s = bgm_slash(j);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (first) bgm_rg(r[u], s, x[u]);
      else bgm_rg_acc(r[u], s, x[u]);
      bgm_pin(x[u]);
    }
  };
  cx j[4], r[2][4];
  bgm_load<N>(F, rec(4), j);
  add(r3, j, ends.ub, true);
  bgm_expand<N>(F, rec(8), [&](int t) { return rec(5 + t); }, j);
  add(x4, j, ends.ub, true);
  bgm_expand5(j5, rec(18), [&](int t) { return rec(12 + t); }, j);
  add(x5, j, ends.ub, true);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int u = 0; u < 2; ++u) bgm_load<N>(F, rec(k) + 16 * u * S::V(k + 1), r[u]);
    bgm_load<N>(F, rec(3 - k), j);
    add(r3, j, r, false);
    bgm_load<N>(F, rec(9 + k), j);
    add(x4, j, r, false);
    if (k == 0) bgm_expand<N>(F, rec(22), [&](int t) { return rec(19 + t); }, j);
    else bgm_load<N>(F, rec(23), j);
    add(x5, j, r, false);
  }
  {
    const int m = rec(25);
    double q[4];
    bgm_topmom<N>(F, m, q);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      cx y[4];
      bgh_prop(r3[u], q, F[S::TFOFF + m], mt, g, y);
      bgh_copy(y, r3[u]);
      bgm_pin(r3[u]);
    }
  }
  bgm_load<N>(F, rec(11), j);
  add(x4, j, r3, false);
  bgm_load<N>(F, rec(24), j);
  add(x5, j, r3, false);
  const int qinfo = rec(FC + 1 + S::QKK), qn = qinfo & 0x7fff;
  const double qs = (qinfo & 0x8000) ? -1.0 : 1.0;
  const int nleaf = it < S::VP2 ? 2 : 1;
#pragma unroll 1
  for (int h = 0; h < nleaf; ++h) {
    const BgmRec<S::FL> leaf(tabs + (h ? S::TL1 : S::TL0), h ? S::VP2 : S::VP, it);
    const int gh = leaf(14);
    cx xn[2][4];
    bgm_expand5(j5, leaf(6), [&](int t) { return leaf(t); }, j);
#pragma unroll
    for (int u = 0; u < 2; ++u) bgm_load<N>(F, rec(0) + 16 * u * S::V(1), r[u]);
    add(xn, j, r, true);
    bgm_expand<N>(F, leaf(10), [&](int t) { return leaf(7 + t); }, j);
#pragma unroll
    for (int u = 0; u < 2; ++u) bgm_load<N>(F, rec(1) + 16 * u * S::V(2), r[u]);
    add(xn, j, r, false);
    bgm_load<N>(F, leaf(11), j);
    add(xn, j, r3, false);
    cx a[4];
#pragma unroll
    for (int uv = 0; uv < 4; ++uv) a[uv] = cx{0.0, 0.0};
    // 1, 5 or 10 terms, the loads of each step in flight together
    auto terms = [&](auto first, auto last) {
      constexpr int T0 = decltype(first)::value, T1 = decltype(last)::value;
#pragma unroll
      for (int half = 0; half < 4; half += 2) {
        cx16 x[T1 - T0][2];
#pragma unroll
        for (int t = T0; t < T1; ++t)
#pragma unroll
          for (int k = 0; k < 2; ++k) x[t - T0][k] = qj[rec(FC + 1 + t) * S::NROW + gh + (half + k) * S::NGH];
#pragma unroll
        for (int t = T0; t < T1; ++t)
#pragma unroll
          for (int k = 0; k < 2; ++k) a[half + k] = a[half + k] + cx{x[t - T0][k].r, x[t - T0][k].i};
      }
    };
    terms(BgmInt<0>{}, BgmInt<1>{});
    if (qn > 1) terms(BgmInt<1>{}, BgmInt<5>{});
    if (qn > 5) terms(BgmInt<5>{}, BgmInt<S::QKK>{});
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      cx c[4], w[2];
      bgm_load<N>(F, leaf(13) + 16 * v * S::V(1), c);
#pragma unroll
      for (int u = 0; u < 2; ++u) w[u] = sdot(xn[u], ends.v[v]) + sdot(x5[u], c);
      bgm_load<N>(F, leaf(12) + 16 * v * S::V(2), c);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const cx x = w[u] + sdot(x4[u], c), q = a[2 * u + v];
        const int row = (2 * u + v) * S::NGH + gh, col = rec(FC);
        jt[(int64_t)(2 * col) * RS + row] = qs * q.r - g * x.i;
        jt[(int64_t)(2 * col + 1) * RS + row] = qs * q.i + g * x.r;
      }
    }
  }
}

// Helicity index (bit npar-1-q set = particle q has helicity +) of a row.
template <int N>
__device__ __forceinline__ int bgm_helicity(int row) {
  constexpr int NPAR = N + 2;
  const int gh = row & (BgmShape<N>::NGH - 1), uv = row / BgmShape<N>::NGH;
  int h = ((uv >> 1) << (NPAR - 3)) | ((uv & 1) << (NPAR - 4));
#pragma unroll
  for (int b = 1; b < N; ++b) h |= ((gh >> (b - 1)) & 1) << (NPAR - 1 - (b < 2 ? b : b + 2));
  return h;
}

// Row of a helicity index: the one it shares with its mirror image.
template <int N>
__device__ __forceinline__ int bgm_row(int h) {
  constexpr int NPAR = N + 2;
  if ((h >> (NPAR - 1)) & 1) h ^= (1 << NPAR) - 1;
  int gh = 0;
#pragma unroll
  for (int b = 1; b < N; ++b) gh |= ((h >> (NPAR - 1 - (b < 2 ? b : b + 2))) & 1) << (b - 1);
  return ((h >> (NPAR - 3)) & 1) * 2 * BgmShape<N>::NGH + ((h >> (NPAR - 4)) & 1) * BgmShape<N>::NGH + gh;
}

// Lane's part of an inverse-CDF draw: of its K consecutive weights v, entries first ..
// first + K - 1 of n, the first whose running sum (cum before them) exceeds t, and the
// last that is positive (-1: none).  An entry that adds nothing is never the one at which
// the sum passes t; where cum, a tree's rounding of the weights before, is above the sum
// with which the lane before ended, t may lie between the two, and the next entry that
// adds something is the one.
template <int K>
__device__ __forceinline__ int bgm_pick(const double* v, int first, int n, double cum, double t, int* last) {
  int pick = -1;
  *last = -1;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    cum += v[i];
    if (v[i] > 0.0) *last = first + i;
    if (pick < 0 && first + i < n && t < cum && (v[i] > 0.0 || first + i == 0)) pick = first + i;
  }
  return pick;
}

#ifdef __HIPCC__
// Workgroup of the fused kernels: EV events of WPE waves each, W waves per SIMD.
// A five-gluon event (a frame of 79 KB) takes four waves, two workgroups to a compute
// unit (160 KB).  Six waves would divide its 384 currents of length 5 and 1152 prefix items
// evenly, but three waves a SIMD leave room for 168 registers each, and workgroups of
// six waves were seen to run one at a time on a compute unit (65 ms for 262144 events
// where four waves took 40, before later changes).  A four-gluon event (18 KB) is one
// wave's work; four share a workgroup so that the set-up, which differs from lane to lane,
// is shared by kind.  A six-gluon event (124 KB) has a compute unit to itself: eight waves, two a SIMD.
template <int N> struct BgmLaunchShape;
// LTAB: the work-item tables are copied to LDS first (four gluons: 7 KB, which leave two
// workgroups to a compute unit; a record is then an LDS read, not one through the vector
// cache in front of every item of the short phases: 524288 g g -> t t~ g g 5.51 ms
// instead of 5.72 on one card).
template <>
struct BgmLaunchShape<4> {
  static constexpr int EV = 4, WPE = 1, W = 2;
  static constexpr bool LTAB = true;
};
template <>
struct BgmLaunchShape<5> {
  static constexpr int EV = 1, WPE = 4, W = 2;
  static constexpr bool LTAB = false;
};
template <>
struct BgmLaunchShape<6> {
  static constexpr int EV = 1, WPE = 8, W = 2;
  static constexpr bool LTAB = false;
};

// The items of a level to the threads, whole waves: the items of the next kind start
// on a wave of their own.
constexpr int bgm_waves(int n) { return (n + 63) & ~63; }

// The tables as the phases read them: copied to LDS behind the frames (to be used after
// the next barrier), or where they are.
template <int N>
__device__ __forceinline__ const uint32_t* bgm_tables(double* lds, const uint32_t* __restrict__ tabs) {
  using B = BgmLaunchShape<N>;
  if constexpr (B::LTAB) {
    uint32_t* t = reinterpret_cast<uint32_t*>(lds + B::EV * BgmShape<N>::FRAME);
    for (int i = threadIdx.x; i < BgmShape<N>::TWORDS; i += 64 * B::EV * B::WPE) t[i] = tabs[i];
    return t;
  } else {
    return tabs;
  }
}

// All phases of nev <= EV events by the whole workgroup, barriers between them: momenta
// and couplings, set-up, currents of length 2 with the spinors of one gluon and Q, of
// length 3 with the spinors of two, of length 4 (five gluons), Q.J, the prefix items.
// The dual amplitudes are in jt [2 NCOL][EV NROW] (row = event NROW + row of the event)
// after the next barrier.
template <int N, typename Note>
__device__ __forceinline__ void bgm_events(double* lds, const uint32_t* tabs,
                                           const double* __restrict__ mom, const double* __restrict__ alphas,
                                           int nev, double g0, double mt, double* jt, int tid, Note note) {
  using S = BgmShape<N>;
  using B = BgmLaunchShape<N>;
  constexpr int EV = B::EV, TE = 64 * B::WPE, THREADS = EV * TE;
  // tables in memory (one event): the records of a phase are read a phase ahead (262144
  // g g -> t t~ g g g 27.7 ms, 28.4 with each read where it is used)
  constexpr bool AHEAD = !B::LTAB;
  static_assert(!AHEAD || (EV == 1 && S::V(2) <= THREADS && S::SV(3) <= THREADS), "one round of the short phases");
  auto read = [&](auto& rec, int table, int items, int i) {
    if (i < items) rec.read(tabs + table, items, i);
  };
  BgmRec<S::F2> r2;
  if constexpr (AHEAD) read(r2, S::T2, S::V(2), tid);
  for (int i = tid; i < nev * (N + 2) * 4; i += THREADS)
    lds[(i / ((N + 2) * 4)) * S::FRAME + S::MOFF + i % ((N + 2) * 4)] = mom[i];
  for (int i = tid; i < nev; i += THREADS)
    lds[i * S::FRAME + S::GOFF] = alphas ? sqrt(4.0 * 3.14159265358979323846 * alphas[i]) : g0;
  __syncthreads();
  {
    // the kinds of every event on waves of their own
    constexpr int NG = 2 * N - 1, A = bgm_waves(EV << N), G = A + bgm_waves(EV * NG), Z = G + 4 * EV;
    for (int i = tid; i < Z; i += THREADS) {
      if (i < A) {
        if (i < nev << N) bgm_setup_subset<N>(lds + (i >> N) * S::FRAME, mt, i & ((1 << N) - 1));
      } else if (i < G) {
        const int k = i - A;
        if (k < nev * NG) bgm_setup_gluon<N>(lds + (k / NG) * S::FRAME, k % NG);
      } else {
        const int k = i - G;
        if (k < 4 * nev) bgm_setup_spinor<N>(lds + (k >> 2) * S::FRAME, mt, k & 3);
      }
    }
  }
  __syncthreads();
  BgmRec<S::F3> r3;
  if constexpr (AHEAD) read(r3, S::T3, S::SV(3), tid);
  {
    constexpr int A = bgm_waves(EV * S::V(2)), R = A + bgm_waves(EV * 2 * S::V(1)), C = R + bgm_waves(EV * 2 * S::V(1)),
                  Z = C + 4 * EV;
    for (int i = tid; i < Z; i += THREADS) {
      if (i < A) {
        const int e = i / S::V(2), k = i % S::V(2);
        if (e < nev) {
          double* F = lds + e * S::FRAME;
          cx j[4];
          if constexpr (!AHEAD) r2.read(tabs + S::T2, S::V(2), k);
          bgm_current<N, 2>(F, r2, j);
          bgm_store<N>(F, S::cslot(2) + k, j);
        }
      } else if (i < C) {
        const bool row = i < R;
        const int k = row ? i - A : i - R, e = k / (2 * S::V(1)), m = k % (2 * S::V(1));
        if (e < nev) {
          if (row) bgm_row1_item<N>(lds + e * S::FRAME, tabs, mt, m % S::V(1), m / S::V(1));
          else bgm_col1_item<N>(lds + e * S::FRAME, tabs, mt, m % S::V(1), m / S::V(1));
        }
      } else {
        const int k = i - C;
        if (k < 4 * nev) bgm_setup_q<N>(lds + (k >> 2) * S::FRAME, k & 3);
      }
    }
  }
  __syncthreads();
  // the spinors of two gluons are wanted by the prefix items only: for five gluons they
  // go where a later round of the threads is not full
  auto pairs = [&](int i, int step) {
    constexpr int R = bgm_waves(EV * 2 * S::V(2)), Z = R + (S::TWO ? EV * 2 * S::V(2) : 0);
    for (; i < Z; i += step) {
      const bool row = i < R;
      const int k = row ? i : i - R, e = k / (2 * S::V(2)), m = k % (2 * S::V(2));
      if (e >= nev) continue;
      if (row) bgm_row2_item<N>(lds + e * S::FRAME, tabs, mt, m % S::V(2), m / S::V(2));
      else if constexpr (S::TWO) bgm_col2_item<N>(lds + e * S::FRAME, tabs, mt, m % S::V(2), m / S::V(2));
    }
  };
  BgmRec<S::F4> r4;
  if constexpr (AHEAD) read(r4, S::T4, S::CV(4), tid);
  {
    constexpr int A = bgm_waves(EV * S::SV(3));
    for (int i = tid; i < EV * S::SV(3); i += THREADS) {
      const int e = i / S::SV(3), k = i % S::SV(3);
      if (e >= nev) continue;
      double* F = lds + e * S::FRAME;
      cx j[4];
      if constexpr (!AHEAD) r3.read(tabs + S::T3, S::SV(3), k);
      bgm_current<N, 3>(F, r3, j);
      bgm_store<N>(F, S::cslot(3) + k, j);
    }
    if constexpr (N == 4) pairs((tid + THREADS - A % THREADS) % THREADS, THREADS);
  }
  __syncthreads();
  // from here on the waves of an event work on it alone
  const int ev = tid / TE, t = tid % TE;
  double* F = lds + ev * S::FRAME;
  double* je = jt + ev * S::NROW;
  const bool on = ev < nev;
  BgmRec<S::FQ> rq;
  if constexpr (N == 5) read(rq, S::TQ, S::CV(N), t);
  BgmRec<S::F5> r5;
  if constexpr (S::BIG) read(r5, S::T5, S::CV(5), t);
  if constexpr (N >= 5) {
    for (int i = t; i < S::CV(4); i += TE) {
      const BgmRec<S::F4> rec = r4;
      read(r4, S::T4, S::CV(4), i + TE);
      cx j[4];
      bgm_current<N, 4>(F, rec, j);
      bgm_store<N>(F, S::cslot(4) + i, j);
    }
    __syncthreads();
  }
  // currents of length 5 and Q.J of six gluons are in the event's scratch
  cx16* j5 = reinterpret_cast<cx16*>(je + S::XJOFF);
  cx16* qj = S::BIG ? reinterpret_cast<cx16*>(je + S::XQOFF) : reinterpret_cast<cx16*>(F + S::QJOFF);
  if constexpr (S::BIG) {
    for (int i = t; i < S::CV(5); i += TE) {
      const BgmRec<S::F5> rec = r5;
      read(r5, S::T5, S::CV(5), i + TE);
      cx j[4];
      bgm_current5<N>(F, rec, j);
#pragma unroll
      for (int c = 0; c < 4; ++c) j5[c * S::CV(5) + i] = cx16{j[c].r, j[c].i};
    }
    pairs(t, TE);
    read(rq, S::TQ, S::CV(N), t);
    __syncthreads();
  }
  if (on) {
    constexpr int NQ = S::NCAN * S::NGH;
    for (int i = t; i < NQ; i += TE) {
      if constexpr (!AHEAD) rq.read(tabs + S::TQ, NQ, i);
      const BgmRec<S::FQ> rec = rq;
      if constexpr (AHEAD) read(rq, S::TQ, NQ, i + TE);
      bgm_qj_item<N>(F, rec, j5, qj, i);
    }
    if (N == 5 && t >= NQ % TE) pairs(t - NQ % TE, TE - NQ % TE);   // the waves without a second current
  }
  // the prefixes with gluon 0 have two leaves, the others one (one wave's two rounds of
  // four gluons take all as having two); the records of the next item are read while
  // this one is worked on
  constexpr int V2 = N == 4 ? S::VP : S::VP2;
  BgmPrefix<N, 2> next;
  BgmRec<S::FP> r6;
  if constexpr (S::BIG) read(r6, S::TP, S::VP, t);
  else if (t < V2) next.read(tabs, t);
  __syncthreads();
  if constexpr (S::BIG) {
    BgmEnds ends;
    bgm_ends<N>(F, ends);
    for (int i = t; i < S::VP; i += TE) {
      const BgmRec<S::FP> rec = r6;
      read(r6, S::TP, S::VP, i + TE);
      bgm_prefix6_item<S::NROW>(F, tabs, rec, ends, mt, j5, qj, je, i);
    }
    return;
  }
  if (on) {
    BgmEnds ends;
    bgm_ends<N>(F, ends);
    auto observe = [&](int r, double re, double im) { note(ev * S::NROW + r, re, im); };
    for (int i = t; i < V2; i += TE) {
      const BgmPrefix<N, 2> p = next;
      if (i + TE < V2) next.read(tabs, i + TE);
      bgm_prefix_item<N, EV * S::NROW, 2>(F, p, ends, je, observe);
    }
    if constexpr (V2 < S::VP) {
      BgmPrefix<N, 1> single;
      if (V2 + t < S::VP) single.read(tabs, V2 + t);
      for (int i = V2 + t; i < S::VP; i += TE) {
        const BgmPrefix<N, 1> p = single;
        if (i + TE < S::VP) single.read(tabs, i + TE);
        bgm_prefix_item<N, EV * S::NROW, 1>(F, p, ends, je, observe);
      }
    }
  }
}

typedef double bgm_f64x4 __attribute__((ext_vector_type(4)));

// FP64 colour form in symmetry sectors.  Relabelling gluons (0 1) and (2 3), and
// reversing the ordering, each map orderings to orderings and leave the colour matrix
// unchanged, and they commute: in the sums and differences over their orbits the
// matrix falls into eight blocks (bgm_sectors), one row per orbit (4, 16).  Six gluons
// have the exchange of (4 5) too: sixteen blocks of 48.  An orbit's members are read once
// and combined by stages of butterflies in registers:
//   a_s[o] = sum_b (-1)^popcount(s & b) A(member b of orbit o).
template <int G>
__device__ __forceinline__ void bgm_butterfly(double* x) {
#pragma unroll
  for (int d = 1; d < G; d <<= 1)
#pragma unroll
    for (int b = 0; b < G; ++b)
      if (!(b & d)) {
        const double p = x[b], q = x[b | d];
        x[b] = p + q;
        x[b | d] = p - q;
      }
}

// Five gluons: the forms of the 64 rows, by every wave of the workgroup.  Four lanes of
// a wave (l % 16 equal) hold shares of a row's form; each hands its own to take(row,
// share), all lanes at the same time.  A wave takes 16 rows: their real and then their
// imaginary parts are the columns of v_mfma_f64_16x16x4f64, a sector's matrix its A
// operand (lane l: row l % 16, K index l / 16), the orbits the K index.  A lane's four orbits o = 4 q + l / 16 are those of
// its accumulator rows, so the dots use the operands in hand.  64 products per 16 rows
// against 288 of the block-triangular form, and no matrix staged in LDS.
template <int WAVES, typename Take>
__device__ __forceinline__ void bgm_colour5(const double* __restrict__ jt, const uint16_t* __restrict__ orb,
                                            const float* __restrict__ sec, int tid, Take take) {
  constexpr int RS = BgmShape<5>::NROW;
  static_assert(WAVES == RS / 16, "16 rows a wave");
  const int l = tid & 63, j = l & 15, kq = l >> 4;
  const int row = 16 * (tid >> 6) + j;
  const double* x = jt + row;
  double a[2][4][8];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double* y = x + (int)orb[(4 * q + kq) * 8 + b] * 2 * RS;
      a[0][q][b] = y[0];
      a[1][q][b] = y[RS];
    }
  double f = 0.0;
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) bgm_butterfly<8>(a[p][q]);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    bgm_f64x4 acc[2] = {bgm_f64x4{0.0, 0.0, 0.0, 0.0}, bgm_f64x4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double m = (double)sec[(s * 4 + q) * 64 + l];
#pragma unroll
      for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, a[p][q][s], acc[p], 0, 0, 0);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) f += a[p][q][s] * acc[p][q];
  }
  take(row, f);
}

// Four gluons: the 32 rows x two parts of an event are the lanes of its wave; the
// sectors (4 x 4, upper triangle with the elements above the diagonal doubled) are
// uniform.  Returns lane l's part of the form of row l % 32.
__device__ __forceinline__ double bgm_colour4(const double* __restrict__ je, const uint16_t* __restrict__ orb,
                                              const float* __restrict__ sec, int tid) {
  using S = BgmShape<4>;
  constexpr int RS = BgmLaunchShape<4>::EV * S::NROW;
  const int l = tid & 63, row = l & 31;
  const double* x = je + (l >> 5) * RS + row;
  double a[4][8];
#pragma unroll
  for (int o = 0; o < 4; ++o) {
#pragma unroll
    for (int b = 0; b < 8; ++b) a[o][b] = x[(int)orb[o * 8 + b] * 2 * RS];
    bgm_butterfly<8>(a[o]);
  }
  double f = 0.0;
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double t = (double)sec[(s * 4 + i) * 4 + i] * a[i][s];
#pragma unroll
      for (int k = i + 1; k < 4; ++k) t += (double)sec[(s * 4 + i) * 4 + k] * a[k][s];
      f += a[i][s] * t;
    }
  return f;
}

// Records, for each row of an event, the largest |Re| and |Im| of its amplitudes
// (bits of a non-negative double, which order as the unsigned integers) with LDS
// atomics: the power-of-two scale of the FP16 colour form without a pass over the
// row.
struct BgmRowMax {
  unsigned long long* m;
  __device__ __forceinline__ void operator()(int k, double re, double im) const {
    atomicMax(m + k, (unsigned long long)__double_as_longlong(fmax(fabs(re), fabs(im))));
  }
};

// Six gluons: 16 rows' real or imaginary parts at a time.  The workgroup transforms the
// 48 orbits of the 16 columns into LDS ([sector][orbit][column]); each wave then takes
// two sectors, three 16-row blocks each, on the matrix cores as above (blocks below the
// diagonal skipped, those above doubled), its matrix operands held in registers, while
// the next columns' amplitudes are on their way.  192 x 2 products per column group of 16
// against 2 x 4140 of the block-triangular form of 720 flows.
template <int WAVES>
__device__ __forceinline__ double bgm_colour6(double* lds, const double* __restrict__ jt,
                                              const uint16_t* __restrict__ orb, const float* __restrict__ sec,
                                              const int* weight) {
  constexpr int RS = BgmShape<6>::NROW, NO = 48, G = 16, THREADS = 64 * WAVES, NI = (NO * 16 + THREADS - 1) / THREADS,
                SW = G / WAVES, NP = 24;
  const int l = threadIdx.x & 63, j = l & 15, kq = l >> 4, w = threadIdx.x >> 6;
  double a[NI][G];
  auto gather = [&](int grp) {
    const double* x = jt + (grp & 1) * RS + 16 * (grp >> 1);
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int i = threadIdx.x + THREADS * k;
      if (i < NO * 16)
#pragma unroll
        for (int b = 0; b < G; ++b) a[k][b] = x[(int)orb[(i >> 4) * G + b] * 2 * RS + (i & 15)];
    }
  };
  float m[SW][NP];
#pragma unroll
  for (int q = 0; q < SW; ++q)
#pragma unroll
    for (int p = 0; p < NP; ++p) m[q][p] = sec[((w + WAVES * q) * NP + p) * 64 + l];
  gather(0);
  double sum = 0.0;
#pragma unroll 1
  for (int grp = 0; grp < RS / 8; ++grp) {
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int i = threadIdx.x + THREADS * k;
      if (i < NO * 16) {
        bgm_butterfly<G>(a[k]);
#pragma unroll
        for (int s = 0; s < G; ++s) lds[(s * NO + (i >> 4)) * 16 + (i & 15)] = a[k][s];
      }
    }
    __syncthreads();
    if (grp + 1 < RS / 8) gather(grp + 1);
    double f = 0.0;
#pragma unroll
    for (int q = 0; q < SW; ++q) {
      double b[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) b[k] = lds[((w + WAVES * q) * NO + 4 * k + kq) * 16 + j];
      bgm_f64x4 acc[3];
      int p = 0;
#pragma unroll
      for (int mb = 0; mb < 3; ++mb) {
        acc[mb] = bgm_f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 4 * mb; k < 12; ++k) {
          asm volatile("" : "+v"(m[q][p]));   // converted here, not held as doubles
          acc[mb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)m[q][p++], b[k], acc[mb], 0, 0, 0);
        }
      }
#pragma unroll
      for (int mb = 0; mb < 3; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) f += b[4 * mb + v] * acc[mb][v];
    }
    const int row = 16 * (grp >> 1) + j;
    sum += weight[row] ? (double)weight[row] * f : 0.0;
    __syncthreads();
  }
  return sum;
}

// Split-precision colour matrix staged in LDS for the fused kernel: flows in blocks
// of 32, the block-triangular form (blocks (mb, kb), kb >= mb: CF on the diagonal,
// 2 CF above; the same quadratic form as CF; the doubled entries stay exact), the
// 32 rows of each block permuted so that a lane's accumulator rows are the flows
// of its own B operand (M index i = 8 q + 4 h + s, q < 4, h < 2, s < 4 holds flow
// 16 (q >> 1) + 8 h + 4 (q & 1) + s), rows of BGM_SV 16-byte vectors (4 + 1: the
// pad puts the 16-byte reads of 8 consecutive rows on distinct banks).
constexpr int BGM_SV = 5;
template <int NCOL>
struct BgmSplit {
  static constexpr int MB = (NCOL + 31) / 32;
  static constexpr int NBLK = MB * (MB + 1) / 2;
  static constexpr int VECS = NBLK * 32 * BGM_SV;   // 16-byte vectors per table
  static constexpr int blk(int mb, int kb) { return mb * MB - mb * (mb - 1) / 2 + (kb - mb); }
  static __device__ __forceinline__ int flow(int i) {
    return 16 * (i >> 4) + 8 * ((i >> 2) & 1) + 4 * ((i >> 3) & 1) + (i & 3);
  }
};

// Split-precision colour form (FMT = CS_FMT_FP16 or CS_FMT_BF16) of the rows
// 0 .. nr - 1 of jt [2 NCOL][rows], by the whole workgroup: one wave per tile of 16
// rows (32 B columns: real and imaginary parts), each row split into hi + lo in the
// format (FP16 rows first scaled by the power of two that puts their largest
// element, rmax[row], in [1, 2): exact), v_mfma_f32_32x32x16 against the staged
// block-triangular matrix, FP64 row dots.  The column blocks kb are taken from the
// last to the first, so that the rows of block kb are complete once kb is done and
// their dots use the amplitudes just loaded for it: every amplitude is read once.
// The matrix cores' FP32 sums do not round symmetrically under a change of sign, so a
// row's mirror image, whose amplitudes are s times the complex conjugates, s =
// (-1)^(u + v + gluons), has another rounding error (of the order of the form's own):
// each of the two is formed by its own products.
// cf_hi / cf_lo: the format's [32 MB][16 KS] tables (cf_lo may be null); cfs holds
// 2 BgmSplit<NCOL>::VECS vectors.  out[row] = the sum of the two forms whose helicities
// are good, in units of the integer matrix.
template <int N, int FMT, int THREADS>
__device__ __forceinline__ void bgm_colour_split(const double* __restrict__ jt, int64_t rows, int nr,
                                                      const void* __restrict__ cf_hi_raw,
                                                      const void* __restrict__ cf_lo_raw, void* cfs_raw,
                                                      const unsigned long long* rmax, const int* weight,
                                                      const int* mirror, double* __restrict__ out) {
  constexpr int NCOL = BgmShape<N>::NCOL, NROW = BgmShape<N>::NROW, NGH = BgmShape<N>::NGH;
  typedef cs_types<FMT> T;
  typedef typename T::vec vec;
  typedef typename T::elem elem;
  using B = BgmSplit<NCOL>;
  constexpr int MB = B::MB;
  constexpr int KP = 16 * ((NCOL + 15) / 16);   // row length of the global tables
  vec* cfs = reinterpret_cast<vec*>(cfs_raw);
  const bool two = cf_lo_raw != nullptr;
  for (int i = threadIdx.x; i < (two ? 2 : 1) * B::NBLK * 128; i += THREADS) {
    const int tb = i / (B::NBLK * 128), rem = i % (B::NBLK * 128);
    const int b = rem >> 7, row = (rem >> 2) & 31, w = rem & 3;
    int mb = 0;
    while (mb + 1 < MB && B::blk(mb + 1, mb + 1) <= b) ++mb;
    const int kb = mb + (b - B::blk(mb, mb));
    const int fa = 32 * mb + B::flow(row), col = 32 * kb + 8 * w;
    vec v;
    if (fa < NCOL && col < KP) {
      v = reinterpret_cast<const vec*>(tb ? cf_lo_raw : cf_hi_raw)[(fa * KP + col) / 8];
      if (kb > mb)
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = (elem)(2.0f * (float)v[t]);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = (elem)0.0f;
    }
    cfs[tb * B::VECS + (b * 32 + row) * BGM_SV + w] = v;
  }
  __syncthreads();
  const int l = threadIdx.x & 63;
  const int j = l & 31, r = j & 15, part = j >> 4;
  const int ntile = (nr + 15) >> 4;
  for (int tile = threadIdx.x >> 6; tile < ntile; tile += THREADS / 64) {
    const int row = 16 * tile + r;
    const bool valid = row < nr;
    double scale = 1.0, unscale = 1.0;
    if (FMT == CS_FMT_FP16) {
      const double m = valid ? __longlong_as_double((long long)rmax[row]) : 0.0;
      if (m > 0.0) {
        const int e = ilogb(m);
        scale = ldexp(1.0, -e);
        unscale = ldexp(1.0, e);
      }
    }
    // does the mirror image change this part's sign?
    const int rr = row & (NROW - 1), uv = rr / NGH;
    const bool minus = ((uv ^ (uv >> 1) ^ N) & 1) != 0;   // s = -1
    const bool flip = part ? !minus : minus;
    // the row's amplitudes of this lane, read once for both passes
    int half = l >> 5;
    asm volatile("" : "+v"(half));   // offsets formed in each tile, not held across tiles
    const double* x = jt + (int64_t)part * rows + (valid ? row : 0);
    double xa[MB][2][8];
#pragma unroll
    for (int kb = 0; kb < MB; ++kb)
#pragma unroll
      for (int ss = 0; ss < 2; ++ss)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int c = 32 * kb + 16 * ss + 8 * half + t;
          xa[kb][ss][t] = (c < NCOL && valid) ? x[(int64_t)(2 * c) * rows] : 0.0;
        }
    double total = 0.0;
#pragma unroll 1
    for (int image = 0; image < 2; ++image) {
      // the matrix operands are read as they are needed in each pass, not hoisted
      int ho = half;
      asm volatile("" : "+v"(ho) : : "memory");
      const vec* ap = cfs + j * BGM_SV + ho;
      const double turn = image && flip ? -1.0 : 1.0;   // exact
      f32x16 acc[MB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[mb][v] = 0.0f;
      double sum = 0.0;
#pragma unroll
      for (int kb = MB - 1; kb >= 0; --kb) {
#pragma unroll
        for (int ss = 0; ss < 2; ++ss) {
          vec bh, bl;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const double v = xa[kb][ss][t] * (turn * scale);
            const elem hi = cs_round<elem>(v);
            bh[t] = hi;
            bl[t] = cs_round<elem>(v - (double)hi);
          }
#pragma unroll
          for (int mb = 0; mb <= kb; ++mb) {
            const vec a = ap[B::blk(mb, kb) * 32 * BGM_SV + 2 * ss];
            acc[mb] = T::mfma(a, bh, acc[mb]);
            acc[mb] = T::mfma(a, bl, acc[mb]);
            if (two) {
              const vec a2 = ap[B::VECS + B::blk(mb, kb) * 32 * BGM_SV + 2 * ss];
              acc[mb] = T::mfma(a2, bh, acc[mb]);
              acc[mb] = T::mfma(a2, bl, acc[mb]);
            }
          }
        }
        // rows of block kb: D element v is M row i = 8 (v >> 2) + 4 half + (v & 3),
        // flow 32 kb + 16 (v >> 3) + 8 half + 4 ((v >> 2) & 1) + (v & 3)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum += xa[kb][v >> 3][4 * ((v >> 2) & 1) + (v & 3)] * (double)acc[kb][v];
      }
      sum *= turn;
      sum += __shfl_xor(sum, 32);   // the two K halves
      sum += __shfl_xor(sum, 16);   // real + imaginary parts
      if (image ? mirror[rr] : weight[rr]) total += sum * unscale;
    }
    if (l < 16 && valid) out[row] = total;
  }
}

__device__ __forceinline__ double bgm_wave_sum(double v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

// Launch variants 4 and 5: workgroup b takes the blocks of EV events b, b + gridDim.x,
// ... (one block each when the grid covers the launch's events, a persistent grid
// otherwise).  For each it writes the dual amplitudes of its rows to its own scratch
// slot, reads them back for the colour form on the matrix cores (FMT < 0: FP64 in
// symmetry sectors; else split FP16 / BF16 with the format's tables cf_hi, cf_lo, the
// block-triangular matrix staged in the LDS of the frames), and writes out[e] = scale *
// the sum of the rows, each taken once per good helicity of its mirror pair.
template <int N, int FMT, bool PERSIST>
__global__ void __launch_bounds__(64 * BgmLaunchShape<N>::EV * BgmLaunchShape<N>::WPE)
    __attribute__((amdgpu_waves_per_eu(BgmLaunchShape<N>::W)))
bgm_fused_kernel(const double* __restrict__ mom, int64_t n, double g0, double mt, const int* __restrict__ hels,
                 int nhel, const uint32_t* __restrict__ tabs, const uint16_t* __restrict__ orb,
                 const float* __restrict__ sec, const double* __restrict__ alphas, double* __restrict__ jt,
                 const void* __restrict__ cf_hi, const void* __restrict__ cf_lo, double* __restrict__ out,
                 double scale) {
  using S = BgmShape<N>;
  using B = BgmLaunchShape<N>;
  constexpr int EV = B::EV, WAVES = EV * B::WPE, THREADS = 64 * WAVES, RS = EV * S::NROW;
  // row values after the split forms' two staged tables (float index)
  constexpr int RV = FMT < 0 ? 0 : 2 * BgmSplit<S::NCOL>::VECS * 4;
  static_assert(RV * sizeof(float) + RS * sizeof(double) <= (size_t)EV * S::FRAME * sizeof(double),
                "the staged colour matrix and the row values must fit in the frames");
  extern __shared__ __attribute__((aligned(16))) double bgm_lds[];
  // whether each row's helicity, and its mirror image's, is good
  __shared__ int weight[S::NROW], mirror[S::NROW];
  __shared__ double part[WAVES];
  // the rows' largest amplitude components (FP16 scaling), written by the prefix items
  __shared__ unsigned long long rmax[FMT == CS_FMT_FP16 ? RS : 1];
  for (int i = threadIdx.x; i < S::NROW; i += THREADS) weight[i] = mirror[i] = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < nhel; k += THREADS) {
    const int h = hels[k];
    (((h >> (N + 1)) & 1) ? mirror : weight)[bgm_row<N>(h)] = 1;
  }
  __syncthreads();
  if constexpr (FMT < 0)   // equal forms: counted together
    for (int i = threadIdx.x; i < S::NROW; i += THREADS) weight[i] += mirror[i];
  double* slot = jt + (int64_t)blockIdx.x * EV * S::SLOT;
  const uint32_t* items = bgm_tables<N>(bgm_lds, tabs);
  for (int64_t e0 = (int64_t)blockIdx.x * EV; e0 < n; e0 += PERSIST ? (int64_t)gridDim.x * EV : n) {
    const int nev = (int)(n - e0 < EV ? n - e0 : EV);
    const double* al = alphas ? alphas + e0 : nullptr;
    if constexpr (FMT == CS_FMT_FP16) {
      for (int i = threadIdx.x; i < RS; i += THREADS) rmax[i] = 0ull;
      bgm_events<N>(bgm_lds, items, mom + e0 * (N + 2) * 4, al, nev, g0, mt, slot, threadIdx.x, BgmRowMax{rmax});
    } else {
      bgm_events<N>(bgm_lds, items, mom + e0 * (N + 2) * 4, al, nev, g0, mt, slot, threadIdx.x, BghNoNote());
    }
    // every amplitude of the block is stored (workgroup-scope fence and barrier) and
    // the frames are no longer read
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    // the colour phase (matrix cores, LDS) at a raised wave priority, so that its
    // issue is not held behind the other workgroup's recursion (vector ALU)
    __builtin_amdgcn_s_setprio(1);
    if constexpr (FMT >= 0) {
      float* cfs = reinterpret_cast<float*>(bgm_lds);
      double* rv = reinterpret_cast<double*>(cfs + RV);
      bgm_colour_split<N, FMT, THREADS>(slot, RS, RS, cf_hi, cf_lo, cfs, rmax, weight, mirror, rv);
      __syncthreads();
      if (w < nev) {
        double v = 0.0;
        for (int r = l; r < S::NROW; r += 64) v += rv[w * S::NROW + r];
        v = bgm_wave_sum(v);
        if (l == 0) out[e0 + w] = scale * v;
      }
    } else if constexpr (N == 4) {
      if (w < nev) {
        const double f = bgm_colour4(slot + w * S::NROW, orb, sec, threadIdx.x);
        const int k = weight[l & 31];
        const double v = bgm_wave_sum(k ? (double)k * f : 0.0);
        if (l == 0) out[e0 + w] = scale * v;
      }
    } else {
      double v = 0.0;
      if constexpr (N == 5)
        bgm_colour5<WAVES>(slot, orb, sec, threadIdx.x,
                           [&](int row, double f) { v += weight[row] ? (double)weight[row] * f : 0.0; });
      else
        v = bgm_colour6<WAVES>(bgm_lds, slot, orb, sec, weight);
      v = bgm_wave_sum(v);
      if (l == 0) part[w] = v;
      __syncthreads();
      if (threadIdx.x == 0) {
        double acc = 0.0;
        for (int k = 0; k < WAVES; ++k) acc += part[k];
        out[e0] = scale * acc;
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // the frames, the staged matrix and the slot are reused by the next block
    if constexpr (PERSIST) __syncthreads();
  }
}

// Inverse-CDF draw by one wave over the non-negative weights weight(k), k = 0 .. n - 1 <=
// 64 K, lane l holding K consecutive ones: the first k whose running sum exceeds r times
// the total, or the last with a positive weight.
template <int K, typename Weight>
__device__ __forceinline__ int bgm_draw(int l, int n, double r, Weight weight, double* total) {
  double v[K], s = 0.0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    v[i] = l * K + i < n ? weight(l * K + i) : 0.0;
    s += v[i];
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double y = __shfl_up(s, d);
    if (l >= d) s += y;
  }
  *total = __shfl(s, 63);
  double cum = __shfl_up(s, 1);
  if (l == 0) cum = 0.0;
  int last;
  const int pick = bgm_pick<K>(v, l * K, n, cum, r * *total, &last);
  const unsigned long long hit = __ballot(pick >= 0), pos = __ballot(last >= 0);
  if (hit) return __shfl(pick, __ffsll((long long)hit) - 1);
  return pos ? __shfl(last, 63 - __clzll((long long)pos)) : 0;
}

// Selection: as the FP64 fused kernel, but each row's form is kept, and the event's wave
// (five gluons: wave 0) draws a helicity with the forms of the good ones (a row's form is
// that of both helicities of its mirror pair) and a flow with the |J_c|^2 of its row,
// read back from the slot.  The row's amplitudes are there already: the one-lane route
// formed every flow of every helicity from its diagrams and then those of the drawn one
// once more.  16384 g g -> t t~ g g g on an MI355X: 1.77 ms, 106.7 by that route.
// PERSIST: a workgroup has one slot for all the blocks that it takes (a slot a block would
// be 2 GB of scratch for these events).  The first is its own, the others come from the
// counter, as compute units do not keep the same pace: block b + gridDim.x after b took 6 %
// more for 16384 events, 13 % for 100003.  Every block asks once, and the last to ask
// leaves the counter cleared for the next launch.
// Up to four rounds of the resident workgroups every block has a slot and a workgroup of
// its own: 600 and 1024 events 97 and 130 us (119 and 136 with PERSIST; four gluons, 2600
// events, 43 and 55); from there on PERSIST is as fast (2600 events 311 us, 321 without)
// and then faster (262144 four-gluon events 2.66 ms, 2.89).
template <int N, bool PERSIST>
__global__ void __launch_bounds__(64 * BgmLaunchShape<N>::EV * BgmLaunchShape<N>::WPE)
    __attribute__((amdgpu_waves_per_eu(BgmLaunchShape<N>::W)))
bgm_select_kernel(const double* __restrict__ mom, int64_t n, double g0, double mt, const int* __restrict__ hels,
                  int nhel, const uint32_t* __restrict__ tabs, const uint16_t* __restrict__ orb,
                  const float* __restrict__ sec, double* __restrict__ jt, const double* __restrict__ r_hel,
                  const double* __restrict__ r_col, double* __restrict__ out, int* __restrict__ sel_hel,
                  int* __restrict__ sel_col, double scale, unsigned* __restrict__ counter) {
  using S = BgmShape<N>;
  using B = BgmLaunchShape<N>;
  constexpr int EV = B::EV, WAVES = EV * B::WPE, RS = EV * S::NROW;
  extern __shared__ __attribute__((aligned(16))) double bgm_lds[];
  __shared__ double form[RS];
  __shared__ unsigned ticket;
  double* slot = jt + (int64_t)blockIdx.x * EV * S::SLOT;
  const uint32_t* items = bgm_tables<N>(bgm_lds, tabs);
  int64_t e0 = (int64_t)blockIdx.x * EV;
  while (e0 < n) {
    unsigned next = 0;
    int o = 0, tid = threadIdx.x;
    if constexpr (PERSIST) {
      // the block after this one, asked for now
      if (threadIdx.x == 0) {
        const unsigned k = atomicAdd(counter, 1u);
        if (k == (unsigned)((n + EV - 1) / EV) - 1u) atomicExch(counter, 0u);
        next = gridDim.x + k;
      }
      // an opaque zero: records and operands are read in each round, not held across rounds
      asm volatile("" : "+s"(o), "+v"(tid));
      __builtin_assume(tid >= 0 && tid < 64 * WAVES);
    }
    const int nev = (int)(n - e0 < EV ? n - e0 : EV);
    bgm_events<N>(bgm_lds, items + o, mom + e0 * (N + 2) * 4, nullptr, nev, g0, mt, slot + o, tid, BghNoNote());
    __syncthreads();   // every amplitude of the block is stored
    const int w = tid >> 6, l = tid & 63;
    if constexpr (N == 4) {
      if (w < nev) {
        double f = bgm_colour4(slot + w * S::NROW, orb + o, sec + o, tid);
        f += __shfl_xor(f, 32);   // real and imaginary parts
        if (l < 32) form[w * S::NROW + l] = f;
      }
    } else {
      bgm_colour5<WAVES>(slot, orb + o, sec + o, tid, [&](int row, double f) {
        f += __shfl_xor(f, 32);
        f += __shfl_xor(f, 16);
        if (l < 16) form[row] = f;
      });
    }
    __syncthreads();
    if (w < nev) {
      const double* fe = form + w * S::NROW;
      double total;
      const int k =
          bgm_draw<(4 << N) / 64>(l, nhel, r_hel[e0 + w], [&](int i) { return fe[bgm_row<N>(hels[o + i])]; }, &total);
      const int h = hels[o + k];
      const double* x = slot + w * S::NROW + bgm_row<N>(h);
      double flows;
      const int c = bgm_draw<(S::NCOL + 63) / 64>(l, S::NCOL, r_col[e0 + w], [&](int i) {
        const double re = x[(int64_t)(2 * i) * RS], im = x[(int64_t)(2 * i + 1) * RS];
        return re * re + im * im;
      }, &flows);
      if (l == 0) {
        out[e0 + w] = scale * total;
        sel_hel[e0 + w] = h;
        sel_col[e0 + w] = c;
      }
    }
    if constexpr (!PERSIST) return;
    if (threadIdx.x == 0) ticket = next;
    __syncthreads();   // the frames, the forms and the slot are the next block's
    e0 = (int64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)ticket) * EV;
  }
}

template <int N, int FMT, bool PERSIST>
const void* bgm_fused_fn() {
  return (const void*)bgm_fused_kernel<N, FMT, PERSIST>;
}

template <int N>
constexpr int bgm_threads() {
  return 64 * BgmLaunchShape<N>::EV * BgmLaunchShape<N>::WPE;
}
template <int N>
constexpr size_t bgm_lds_bytes() {
  return (size_t)BgmLaunchShape<N>::EV * BgmShape<N>::FRAME * sizeof(double) +
         (BgmLaunchShape<N>::LTAB ? BgmShape<N>::TWORDS * sizeof(uint32_t) : 0);
}

// Resident workgroups per compute unit of the fused kernels (0 if not built), the
// least over the colour-sum formats.
template <int N>
int bgm_fused_per_cu() {
  if constexpr (N >= 4) {
    int best = 1 << 20;
    std::initializer_list<const void*> fns;
    if constexpr (N == 6)
      fns = {bgm_fused_fn<N, -1, false>()};
    else
      fns = {bgm_fused_fn<N, -1, true>(),  bgm_fused_fn<N, CS_FMT_FP16, true>(),  bgm_fused_fn<N, CS_FMT_BF16, true>(),
             bgm_fused_fn<N, -1, false>(), bgm_fused_fn<N, CS_FMT_FP16, false>(), bgm_fused_fn<N, CS_FMT_BF16, false>()};
    for (const void* fn : fns) {
      if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bgm_lds_bytes<N>()) != hipSuccess)
        return 0;
      int nb = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, bgm_threads<N>(), bgm_lds_bytes<N>()) !=
          hipSuccess)
        return 0;
      best = nb < best ? nb : best;
    }
    return best;
  } else {
    return 0;
  }
}

// Doubles of scratch and events per workgroup of the fused kernels (0 if not built).
template <int N>
int64_t bgm_fused_slot_doubles() {
  if constexpr (N >= 4) {
    return (int64_t)BgmLaunchShape<N>::EV * BgmShape<N>::SLOT;
  } else {
    return 0;
  }
}
template <int N>
int bgm_block_events() {
  if constexpr (N >= 4) {
    return BgmLaunchShape<N>::EV;
  } else {
    return 0;
  }
}

// Variant 4: one workgroup per event block (the launch's blocks must not exceed a.grid
// slots); variant 5: a persistent grid of a.grid workgroups.
template <int N, int FMT, bool PERSIST>
hipError_t launch_bgm_fused_fmt(const BgArgs& a) {
  constexpr int EV = BgmLaunchShape<N>::EV;
  constexpr size_t lds = bgm_lds_bytes<N>();
  static const hipError_t attr = hipFuncSetAttribute(bgm_fused_fn<N, FMT, PERSIST>(),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  if (!a.bgm || !a.orb || !a.sec || !a.out || a.grid < 1 || (FMT >= 0 && !a.cf_hi)) return hipErrorInvalidValue;
  if (a.n == 0 || a.nhel == 0) return hipSuccess;
  const int64_t blocks = (a.n + EV - 1) / EV;
  if (!PERSIST && blocks > a.grid) return hipErrorInvalidValue;   // one slot per block
  const unsigned grid = (unsigned)(blocks < a.grid ? blocks : a.grid);
  hipLaunchKernelGGL((bgm_fused_kernel<N, FMT, PERSIST>), dim3(grid), dim3(bgm_threads<N>()), lds, a.stream, a.mom,
                     a.n, a.g, a.mt, a.hels, a.nhel, a.bgm, a.orb, a.sec, a.alphas, a.jt, a.cf_hi, a.cf_lo, a.out,
                     a.out_scale);
  return hipGetLastError();
}

// One block a workgroup where the launch's blocks are no more than a.grid slots, else
// a.grid persistent workgroups.
template <int N, bool PERSIST>
hipError_t launch_bgm_select(const BgArgs& a) {
  constexpr int EV = BgmLaunchShape<N>::EV;
  constexpr size_t lds = bgm_lds_bytes<N>();
  static const hipError_t attr = hipFuncSetAttribute((const void*)bgm_select_kernel<N, PERSIST>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  const int64_t blocks = (a.n + EV - 1) / EV;
  if (!a.bgm || !a.orb || !a.sec || !a.out || !a.r_hel || !a.r_col || !a.sel_col || a.nhel < 1 ||
      a.nhel > (4 << N) || a.grid < 1 || blocks > 0x7fffffff || (PERSIST ? !a.counter : blocks > a.grid))
    return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(PERSIST ? a.grid : blocks);
  hipLaunchKernelGGL((bgm_select_kernel<N, PERSIST>), dim3(grid), dim3(bgm_threads<N>()), lds, a.stream, a.mom, a.n,
                     a.g, a.mt, a.hels, a.nhel, a.bgm, a.orb, a.sec, a.jt, a.r_hel, a.r_col, a.out, a.sel_hel,
                     a.sel_col, a.out_scale, a.counter);
  return hipGetLastError();
}

template <int N, bool PERSIST>
hipError_t launch_bgm_fused_p(const BgArgs& a) {
  if (a.fmt == CS_FMT_FP16) return launch_bgm_fused_fmt<N, CS_FMT_FP16, PERSIST>(a);
  if (a.fmt == CS_FMT_BF16) return launch_bgm_fused_fmt<N, CS_FMT_BF16, PERSIST>(a);
  return launch_bgm_fused_fmt<N, -1, PERSIST>(a);
}

// Launch of the executor's kernel in the chosen variant (3: one-sided helicity
// recycling, me_bgh.h; 4 and 5: the two-sided recursion with the colour form and the
// helicity sum fused when a per-event output is given; built for four and five gluons).
template <int N>
hipError_t launch_bg(const BgArgs& a) {
  if constexpr (N == 4 || N == 5) {
    if (a.sel_hel)
      return (a.n + BgmLaunchShape<N>::EV - 1) / BgmLaunchShape<N>::EV > a.grid ? launch_bgm_select<N, true>(a)
                                                                               : launch_bgm_select<N, false>(a);
    if ((a.variant == 4 || a.variant == 5) && a.out)
      return a.variant == 5 ? launch_bgm_fused_p<N, true>(a) : launch_bgm_fused_p<N, false>(a);
    if (a.variant >= 3) return launch_bgh<N>(a);
  } else {
    if constexpr (N == 6)
      if (a.out) return launch_bgm_fused_fmt<N, -1, false>(a);
    if (a.variant >= 3) return hipErrorInvalidValue;
  }
  if (a.variant == 1) return launch_bg_v<N, 1>(a);
  if (a.variant == 2) return launch_bg_v<N, 2>(a);
  return launch_bg_v<N, 0>(a);
}
#endif

}  // namespace me
