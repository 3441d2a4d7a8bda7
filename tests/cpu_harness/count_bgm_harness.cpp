// Operation count of the two-sided recursion's device functions (test-only): the FP64
// type becomes a counting scalar (see count_harness.cpp), one event is evaluated phase
// by phase as the kernel does, and the counted operations are returned.
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "me_bgm_tables.h"

namespace cnt {
long long flops = 0;
struct CD {
  double v;
  CD() = default;
  CD(double x) : v(x) {}
};
inline CD operator+(CD a, CD b) { ++flops; return CD(a.v + b.v); }
inline CD operator-(CD a, CD b) { ++flops; return CD(a.v - b.v); }
inline CD operator*(CD a, CD b) { ++flops; return CD(a.v * b.v); }
inline CD operator/(CD a, CD b) { ++flops; return CD(a.v / b.v); }
inline CD operator-(CD a) { return CD(-a.v); }
inline CD& operator+=(CD& a, CD b) { ++flops; a.v += b.v; return a; }
inline CD& operator-=(CD& a, CD b) { ++flops; a.v -= b.v; return a; }
inline CD& operator*=(CD& a, CD b) { ++flops; a.v *= b.v; return a; }
inline bool operator<(CD a, CD b) { return a.v < b.v; }
inline bool operator>(CD a, CD b) { return a.v > b.v; }
inline bool operator<=(CD a, CD b) { return a.v <= b.v; }
inline bool operator>=(CD a, CD b) { return a.v >= b.v; }
inline bool operator==(CD a, CD b) { return a.v == b.v; }
inline bool operator!=(CD a, CD b) { return a.v != b.v; }
inline CD sqrt(CD a) { ++flops; return CD(std::sqrt(a.v)); }
}  // namespace cnt

using cnt::CD;
using cnt::sqrt;
#define double CD
#define volatile
#define asm(...) (void)0
#include "me_bgm.h"
#undef asm
#undef volatile
#undef double

// set-up, stored currents, spinors, Q.J, prefix items
template <int N>
void count_event(const double* mom, long long* out) {
  using namespace me;
  using S = BgmShape<N>;
  const std::vector<uint32_t>& t = bgm_items<N>();
  std::vector<cx16> frame((S::FRAME + 1) / 2), slot(S::SLOT / 2);
  CD* F = &frame[0].r;
  CD* jt = &slot[0].r;
  for (int i = 0; i < (N + 2) * 4; ++i) F[S::MOFF + i] = CD(mom[i]);
  F[S::GOFF] = CD(1.2);
  const CD mt(173.0);
  auto lap = [&](int k) {
    out[k] += cnt::flops;
    cnt::flops = 0;
  };
  for (int k = 0; k < 5; ++k) out[k] = 0;
  cnt::flops = 0;
  for (int i = 0; i < (1 << N); ++i) bgm_setup_subset<N>(F, mt, i);
  for (int i = 0; i < 2 * N - 1; ++i) bgm_setup_gluon<N>(F, i);
  for (int i = 0; i < 4; ++i) bgm_setup_spinor<N>(F, mt, i);
  for (int i = 0; i < 4; ++i) bgm_setup_q<N>(F, i);
  lap(0);
  cx j[4];
  for (int i = 0; i < S::V(2); ++i) {
    bgm_current<N, 2>(F, BgmRec<S::F2>(t.data() + S::T2, S::V(2), i), j);
    bgm_store<N>(F, S::cslot(2) + i, j);
  }
  for (int i = 0; i < S::SV(3); ++i) {
    bgm_current<N, 3>(F, BgmRec<S::F3>(t.data() + S::T3, S::SV(3), i), j);
    bgm_store<N>(F, S::cslot(3) + i, j);
  }
  if (N >= 5)
    for (int i = 0; i < S::CV(4); ++i) {
      bgm_current<N, 4>(F, BgmRec<S::F4>(t.data() + S::T4, S::CV(4), i), j);
      bgm_store<N>(F, S::cslot(4) + i, j);
    }
  cx16* j5 = &slot[S::XJOFF / 2];
  cx16* qj = S::BIG ? &slot[S::XQOFF / 2] : &frame[S::QJOFF / 2];
  if constexpr (S::BIG)
    for (int i = 0; i < S::CV(5); ++i) {
      bgm_current5<N>(F, BgmRec<S::F5>(t.data() + S::T5, S::CV(5), i), j);
      for (int c = 0; c < 4; ++c) j5[c * S::CV(5) + i] = cx16{j[c].r, j[c].i};
    }
  lap(1);
  for (int i = 0; i < 2 * S::V(1); ++i) {
    bgm_row1_item<N>(F, t.data(), mt, i >> 1, i & 1);
    bgm_col1_item<N>(F, t.data(), mt, i >> 1, i & 1);
  }
  for (int i = 0; i < 2 * S::V(2); ++i) {
    bgm_row2_item<N>(F, t.data(), mt, i >> 1, i & 1);
    if (S::TWO) bgm_col2_item<N>(F, t.data(), mt, i >> 1, i & 1);
  }
  lap(2);
  for (int i = 0; i < S::NCAN * S::NGH; ++i) bgm_qj_item<N>(F, BgmRec<S::FQ>(t.data() + S::TQ, S::CV(N), i), j5, qj, i);
  lap(3);
  BgmEnds ends;
  bgm_ends<N>(F, ends);
  if constexpr (S::BIG) {
    for (int i = 0; i < S::VP; ++i) 
        bgm_prefix6_item<S::NROW>(F, t.data(), BgmRec<S::FP>(t.data() + S::TP, S::VP, i), ends, mt, j5, qj, jt, i);
  } else {
    for (int i = 0; i < S::VP2; ++i) {
      BgmPrefix<N, 2> p;
      p.read(t.data(), i);
      bgm_prefix_item<N, S::NROW, 2>(F, p, ends, jt, BghNoNote());
    }
    for (int i = S::VP2; i < S::VP; ++i) {
      BgmPrefix<N, 1> p;
      p.read(t.data(), i);
      bgm_prefix_item<N, S::NROW, 1>(F, p, ends, jt, BghNoNote());
    }
  }
  lap(4);
}

extern "C" int count_bgm_event(int n, const double* mom, long long* out) {
  switch (n) {
    case 4: count_event<4>(mom, out); return 0;
    case 5: count_event<5>(mom, out); return 0;
    case 6: count_event<6>(mom, out); return 0;
    default: return -1;
  }
}
