// Sizes shared by the two-sided recursion's kernels and its host tables (me_bgm.h,
// me_bgm_tables.h).  Plain C++.
#pragma once

namespace me {

// Gluon 0 keeps one helicity (see me_bgm.h): a sequence has 2^(gluons other than
// gluon 0) helicity variants.
template <int N>
struct BgmShape {
  static constexpr int perm(int n, int k) { return k == 0 ? 1 : n * perm(n - 1, k - 1); }
  static constexpr int fact(int n) { return perm(n, n); }
  static constexpr int comb(int n, int k) { return perm(n, k) / fact(k); }
  // variants of the sequences of length L: those with gluon 0, then those without
  static constexpr int V(int L) {
    return L * perm(N - 1, L - 1) * (1 << (L - 1)) + (L < N ? perm(N - 1, L) * (1 << L) : 0);
  }
  // stored variants: J(c b a) = J(a b c), so of two mirrored sequences of length 3 one
  static constexpr int SV(int L) { return L == 3 ? V(3) / 2 : V(L); }
  // variants of the canonical sequences (lowest gluon first) of length L
  static constexpr int CV(int L) {
    return fact(L - 1) * (comb(N - 1, L - 1) * (1 << (L - 1)) + (L < N ? comb(N - 1, L) * (1 << L) : 0));
  }
  static constexpr int NCOL = fact(N);
  static constexpr int NGH = 1 << (N - 1);        // gluon helicities with gluon 0 fixed
  static constexpr int NROW = 4 * NGH;            // rows of an event: (u, v) x gluon helicities
  static constexpr int NCAN = fact(N - 1);        // orderings that start with gluon 0
  static constexpr int QKK = comb(N - 1, (N - 1) / 2);   // most terms of an expansion over them
  static constexpr bool TWO = N >= 5;             // column spinors of two gluons are stored
  static constexpr bool BIG = N == 6;             // currents of length 5 and Q.J in memory, not in LDS
  // slots of stored four-vectors: currents of length 1, 2, 3 and, from five gluons on,
  // 4 (canonical); row spinors of length 1, 2 per top helicity; column
  // spinors of length 1 (2) per antitop helicity; ubar[2], v[2], Q[2][2]
  static constexpr int cslot(int L) { return L == 1 ? 0 : L == 2 ? V(1) : L == 3 ? V(1) + V(2) : V(1) + V(2) + SV(3); }
  static constexpr int R1S = cslot(4) + (N >= 5 ? CV(4) : 0);
  static constexpr int R2S = R1S + 2 * V(1);
  static constexpr int C1S = R2S + 2 * V(2);
  static constexpr int C2S = C1S + 2 * V(1);
  static constexpr int UBS = C2S + (TWO ? 2 * V(2) : 0);
  static constexpr int VS = UBS + 2;
  static constexpr int QS = VS + 2;
  static constexpr int NS = QS + 4;
  // words of a record and items of each phase, in the order of the tables
  static constexpr int F1 = 1, F2 = 3, FR2 = 6, F3 = 7, F4 = 11, F5 = 20, F6 = 35;
  static constexpr int VP = V(N - 1);             // prefix items
  static constexpr int VP2 = (N - 1) * perm(N - 1, N - 2) * (1 << (N - 2));   // those with gluon 0: two leaves
  static constexpr int FP = (N == 4 ? 5 : N == 5 ? 11 : 26) + 1 + QKK + 1;
  static constexpr int FL = N == 4 ? 4 : N == 5 ? 8 : 15;
  static constexpr int words(int f) { return (f + 1) / 2; }
  static constexpr int T1 = 0;
  static constexpr int T2 = T1 + words(F1) * V(1);
  static constexpr int TR2 = T2 + words(F2) * V(2);
  static constexpr int T3 = TR2 + words(FR2) * V(2);
  static constexpr int T4 = T3 + words(F3) * SV(3);
  static constexpr int T5 = T4 + words(F4) * CV(4);
  static constexpr int T6 = T5 + (N >= 5 ? words(F5) * CV(5) : 0);
  static constexpr int TP = T6 + (BIG ? words(F6) * CV(6) : 0);
  // those of the currents of all gluons
  static constexpr int FQ = N == 4 ? F4 : N == 5 ? F5 : F6;
  static constexpr int TQ = N == 4 ? T4 : N == 5 ? T5 : T6;
  static constexpr int TL0 = TP + words(FP) * VP;
  static constexpr int TL1 = TL0 + words(FL) * VP;
  static constexpr int TWORDS = TL1 + words(FL) * VP2;
  // frame in doubles: the slots (component-major: component c of slot s is the complex
  // number at c NS + s), Q.J of the canonical orderings (complex [NCAN][4][NGH]; up to
  // five gluons), momentum sums and propagators of every subset, momenta, coupling
  static constexpr int QJOFF = 8 * NS;
  static constexpr int PSOFF = QJOFF + (BIG ? 0 : 2 * NCAN * NROW);   // momentum sums [2^N][4]
  static constexpr int GIOFF = PSOFF + (4 << N);          // 1 / P(mask)^2
  static constexpr int TFOFF = GIOFF + (1 << N);          // 1 / (q^2 - mt^2), q = p3 - P(mask)
  static constexpr int MOFF = TFOFF + (1 << N);           // momenta [N + 2][4]
  static constexpr int GOFF = MOFF + 4 * (N + 2);         // coupling
  static constexpr int FRAME = GOFF + 2;
  // doubles of an event's scratch: dual amplitudes [2 NCOL][NROW]; for six gluons also
  // Q.J and the canonical currents of length 5, complex [4][CV(5)]
  static constexpr int XQOFF = 2 * NCOL * NROW;
  static constexpr int XJOFF = XQOFF + (BIG ? 2 * NCAN * NROW : 0);
  static constexpr int SLOT = XJOFF + (BIG ? 8 * CV(5) : 0);
};

}  // namespace me
