// Host build of the two-sided recursion (test-only): one event at a time, every phase's
// items in turn, exactly the device functions the kernel runs per thread.
#include <cstring>
#include <vector>

#include "me_bgm.h"
#include "me_bgm_tables.h"
#include "me_pair_desc.h"

template <int N>
void bgm_eval(const double* mom, int nevt, double g, double mt, double* jamps) {
  using namespace me;
  using S = BgmShape<N>;
  const std::vector<uint32_t>& t = bgm_items<N>();
  std::vector<cx16> frame((S::FRAME + 1) / 2), slot(S::SLOT / 2);
  double* F = &frame[0].r;
  double* jt = &slot[0].r;
  for (int e = 0; e < nevt; ++e) {
    for (int i = 0; i < (N + 2) * 4; ++i) F[S::MOFF + i] = mom[e * (N + 2) * 4 + i];
    F[S::GOFF] = g;
    for (int i = 0; i < (1 << N); ++i) bgm_setup_subset<N>(F, mt, i);
    for (int i = 0; i < 2 * N - 1; ++i) bgm_setup_gluon<N>(F, i);
    for (int i = 0; i < 4; ++i) bgm_setup_spinor<N>(F, mt, i);
    for (int i = 0; i < 4; ++i) bgm_setup_q<N>(F, i);
    cx j[4];
    for (int i = 0; i < S::V(2); ++i) {
      bgm_current<N, 2>(F, BgmRec<S::F2>(t.data() + S::T2, S::V(2), i), j);
      bgm_store<N>(F, S::cslot(2) + i, j);
    }
    for (int i = 0; i < 2 * S::V(1); ++i) {
      bgm_row1_item<N>(F, t.data(), mt, i >> 1, i & 1);
      bgm_col1_item<N>(F, t.data(), mt, i >> 1, i & 1);
    }
    for (int i = 0; i < S::SV(3); ++i) {
      bgm_current<N, 3>(F, BgmRec<S::F3>(t.data() + S::T3, S::SV(3), i), j);
      bgm_store<N>(F, S::cslot(3) + i, j);
    }
    for (int i = 0; i < 2 * S::V(2); ++i) {
      bgm_row2_item<N>(F, t.data(), mt, i >> 1, i & 1);
      if (S::TWO) bgm_col2_item<N>(F, t.data(), mt, i >> 1, i & 1);
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
    for (int i = 0; i < S::NCAN * S::NGH; ++i) bgm_qj_item<N>(F, BgmRec<S::FQ>(t.data() + S::TQ, S::CV(N), i), j5, qj, i);
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
    for (int r = 0; r < S::NROW; ++r)
      for (int c = 0; c < 2 * S::NCOL; ++c)
        jamps[(((size_t)e * S::NROW + r) * S::NCOL + c / 2) * 2 + c % 2] = jt[(size_t)c * S::NROW + r];
  }
}

extern "C" int harness_bgm_words(int n) {
  return n == 4   ? (int)me::bgm_items<4>().size() - me::BgmShape<4>::TWORDS
         : n == 5 ? (int)me::bgm_items<5>().size() - me::BgmShape<5>::TWORDS
                  : (int)me::bgm_items<6>().size() - me::BgmShape<6>::TWORDS;
}

// row of helicity h of n gluons
extern "C" int harness_bgm_row(int n, int h) {
  return n == 4 ? me::bgm_row<4>(h) : n == 5 ? me::bgm_row<5>(h) : me::bgm_row<6>(h);
}

// mirror pairs of nh good helicities of all; returns their number
extern "C" int harness_mirror_pairs(const int* good, int nh, int all, int* pairs) {
  const std::vector<int> p = me::mirror_pairs(std::vector<int>(good, good + nh), all);
  std::copy(p.begin(), p.end(), pairs);
  return (int)p.size();
}

// orbits (norb x 2^nsym columns) and sectors of the colour form; returns norb
extern "C" int harness_bgm_sectors(int n, const int* cf, int* orb, double* sec) {
  const me::BgmSectors s = me::bgm_sectors(n, cf);
  std::copy(s.orb.begin(), s.orb.end(), orb);
  std::copy(s.sec.begin(), s.sec.end(), sec);
  return s.norb;
}

// The draw of bgm_draw<2> with the wave's steps in turn: running sums of the lanes' weights
// by doubling distances, then every lane's pick; cum[64] = the running sum before each lane.
extern "C" int harness_bgm_draw(int n, const double* w, double t, double* cum) {
  constexpr int K = 2;
  double v[64][K], s[64], up[64];
  for (int l = 0; l < 64; ++l) {
    s[l] = 0.0;
    for (int i = 0; i < K; ++i) s[l] += v[l][i] = l * K + i < n ? w[l * K + i] : 0.0;
  }
  for (int d = 1; d < 64; d <<= 1) {
    std::copy(s, s + 64, up);
    for (int l = d; l < 64; ++l) s[l] += up[l - d];
  }
  int last = -1;
  for (int l = 0; l < 64; ++l) cum[l] = l ? s[l - 1] : 0.0;
  for (int l = 0; l < 64; ++l) {
    int pos;
    const int pick = me::bgm_pick<K>(v[l], l * K, n, cum[l], t, &pos);
    if (pick >= 0) return pick;
    if (pos >= 0) last = pos;
  }
  return last < 0 ? 0 : last;
}

// jamps [nevt][NROW][n!][2]; hel[NROW] = helicity index of each row
extern "C" int harness_bgm_eval(int n, const double* mom, int nevt, double g, double mt, double* jamps, int* hel) {
  for (int r = 0; r < (2 << n); ++r)
    hel[r] = n == 4 ? me::bgm_helicity<4>(r) : n == 5 ? me::bgm_helicity<5>(r) : me::bgm_helicity<6>(r);
  switch (n) {
    case 4: bgm_eval<4>(mom, nevt, g, mt, jamps); return 0;
    case 5: bgm_eval<5>(mom, nevt, g, mt, jamps); return 0;
    case 6: bgm_eval<6>(mom, nevt, g, mt, jamps); return 0;
    default: return -1;
  }
}
