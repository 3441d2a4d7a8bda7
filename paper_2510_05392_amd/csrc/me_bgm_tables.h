// Host-side tables of the two-sided recursion (me_bgm.h): for every work item of a
// level, the addresses of the currents and spinors it reads.  Plain C++.
#pragma once
#include <algorithm>
#include <cstdint>
#include <map>
#include <vector>

#include "me_bgm_shape.h"

namespace me {

// One phase's records: `fields` 16-bit values per item, two to a word, word w of
// item i at words[w items + i] (consecutive items are consecutive words).
struct BgmPhase {
  int items, fields;
  std::vector<std::vector<uint16_t>> rec;
  BgmPhase(int items_, int fields_) : items(items_), fields(fields_) {}
  void append(std::vector<uint32_t>& out) const {
    const int words = (fields + 1) / 2;
    const size_t base = out.size();
    out.resize(base + (size_t)words * items, 0);
    for (int i = 0; i < items; ++i)
      for (int f = 0; f < fields; ++f)
        out[base + (size_t)(f / 2) * items + i] |= (uint32_t)rec.at(i).at(f) << (16 * (f & 1));
  }
};

template <int N>
class BgmBuilder {
  using S = BgmShape<N>;
  typedef std::vector<int> Seq;
  // by code(s): first variant of every sequence among those of its length, the same among
  // the stored sequences of length 3 (first gluon < last) and the canonical sequences
  // (lowest gluon first), and the sequence's rank among its length's
  std::vector<int> var_, var3_, canon_, rank_;
  std::vector<std::vector<Seq>> full_, can_;   // by length, in variant order

  static int mask(const Seq& s, int a, int b) {
    int m = 0;
    for (int i = a; i < b; ++i) m |= 1 << s[i];
    return m;
  }
  static int code(const Seq& s) {
    int c = 0;
    for (int g : s) c = 8 * c + g + 1;
    return c;
  }
  static int nvar(int m) { return 1 << __builtin_popcount(m >> 1); }
  // bits of hv deposited at the gluons of m other than gluon 0 (bit b - 1 = gluon b)
  static int deposit(int hv, int m) {
    int r = 0, k = 0;
    for (int b = 1; b < N; ++b)
      if (m >> b & 1) r |= (hv >> k++ & 1) << (b - 1);
    return r;
  }
  static int extract(int gh, int m) {
    int r = 0, k = 0;
    for (int b = 1; b < N; ++b)
      if (m >> b & 1) r |= (gh >> (b - 1) & 1) << k++;
    return r;
  }
  static Seq part(const Seq& s, int a, int b) { return Seq(s.begin() + a, s.begin() + b); }
  static uint16_t slot(int s) { return (uint16_t)(16 * s); }   // byte offset of the slot's first component

  int variant(const Seq& s, int gh) const { return var_.at(code(s)) + extract(gh, mask(s, 0, (int)s.size())); }
  int cvariant(const Seq& s, int gh) const { return canon_.at(code(s)) + extract(gh, mask(s, 0, (int)s.size())); }

  // stored current of s[a:b] at gluon helicities gh
  uint16_t cur(const Seq& s, int a, int b, int gh) const {
    const Seq p = part(s, a, b);
    const int L = b - a;
    if (L == 3 && p[0] > p[2]) return cur(Seq(p.rbegin(), p.rend()), 0, 3, gh);
    if (L <= 3) return slot(S::cslot(L) + (L == 3 ? var3_.at(code(p)) + extract(gh, mask(p, 0, 3)) : variant(p, gh)));
    return slot(S::cslot(L) + cvariant(p, gh));   // canonical sequences of length 4
  }

  // J(alpha, x, beta) = (-1)^|alpha| sum J(x, rho) over the shuffles rho of reversed
  // alpha with beta, x the lowest gluon: the canonical sequences, sign in *neg
  static std::vector<Seq> expand(const Seq& s, bool* neg) {
    const int p = (int)(std::min_element(s.begin(), s.end()) - s.begin());
    *neg = p & 1;
    Seq al(s.begin(), s.begin() + p), be(s.begin() + p + 1, s.end());
    std::reverse(al.begin(), al.end());
    const int na = (int)al.size(), n = na + (int)be.size();
    std::vector<Seq> out;
    for (int m = 0; m < (1 << n); ++m) {
      if (__builtin_popcount(m) != na) continue;
      Seq r{s[p]};
      int ia = 0, ib = 0;
      for (int k = 0; k < n; ++k) r.push_back(m >> k & 1 ? al[ia++] : be[ib++]);
      out.push_back(r);
    }
    return out;
  }
  static uint16_t info(size_t count, bool neg) { return (uint16_t)(count | (neg ? 0x8000 : 0)); }

  // count addresses of the expansion of s[a:b] (length 4) and its info word
  void kk4(std::vector<uint16_t>& r, const Seq& s, int a, int b, int gh) const {
    bool neg;
    const std::vector<Seq> e = expand(part(s, a, b), &neg);
    for (int t = 0; t < 3; ++t) r.push_back(cur(e[t < (int)e.size() ? t : 0], 0, 4, gh));
    r.push_back(info(e.size(), neg));
  }

  // the same for s[a:b] of length 5 (variant numbers)
  void kk5(std::vector<uint16_t>& r, const Seq& s, int a, int b, int gh) const {
    bool neg;
    const std::vector<Seq> e = expand(part(s, a, b), &neg);
    for (int t = 0; t < 6; ++t) r.push_back((uint16_t)cvariant(e[t < (int)e.size() ? t : 0], gh));
    r.push_back(info(e.size(), neg));
  }

  static void perms(const Seq& from, int len, Seq& cur, std::vector<Seq>& out) {
    if ((int)cur.size() == len) {
      out.push_back(cur);
      return;
    }
    for (int g : from)
      if (std::find(cur.begin(), cur.end(), g) == cur.end()) {
        cur.push_back(g);
        perms(from, len, cur, out);
        cur.pop_back();
      }
  }

 public:
  BgmBuilder()
      : var_(1 << 3 * N, -1), var3_(var_), canon_(var_), rank_(var_), full_(N + 1), can_(N + 1) {
    Seq all;
    for (int g = 0; g < N; ++g) all.push_back(g);
    for (int L = 1; L <= N; ++L) {
      Seq c;
      perms(all, L, c, full_[L]);
      int nf = 0, nc = 0, n3 = 0;
      for (const Seq& s : full_[L]) {
        if (L == 3 && s[0] < s[2]) {
          var3_[code(s)] = n3;
          n3 += nvar(mask(s, 0, 3));
        }
        rank_[code(s)] = &s - &full_[L][0];
        var_[code(s)] = nf;
        nf += nvar(mask(s, 0, L));
        if (*std::min_element(s.begin(), s.end()) == s[0]) {
          canon_[code(s)] = nc;
          can_[L].push_back(s);
          nc += nvar(mask(s, 0, L));
        }
      }
    }
  }

  std::vector<uint32_t> build() const {
    std::vector<uint32_t> out;
    std::vector<Seq> stored3;
    BgmPhase one(S::V(1), S::F1), two(S::V(2), S::F2), three(S::SV(3), S::F3), rtwo(S::V(2), S::FR2);
    for (const Seq& s : full_[1])
      for (int hv = 0; hv < nvar(mask(s, 0, 1)); ++hv) one.rec.push_back({(uint16_t)mask(s, 0, 1)});
    for (const Seq& s : full_[2])
      for (int hv = 0; hv < nvar(mask(s, 0, 2)); ++hv) {
        const int gh = deposit(hv, mask(s, 0, 2));
        two.rec.push_back({cur(s, 0, 1, gh), cur(s, 1, 2, gh),
                           (uint16_t)(mask(s, 0, 1) | mask(s, 0, 2) << 8)});
        rtwo.rec.push_back({cur(s, 0, 1, gh), cur(s, 1, 2, gh), cur(s, 0, 2, gh),
                            slot(S::R1S + variant(part(s, 0, 1), gh)), slot(S::C1S + variant(part(s, 1, 2), gh)),
                            (uint16_t)mask(s, 0, 2)});
      }
    for (const Seq& s : full_[3])
      if (s[0] < s[2]) stored3.push_back(s);
    for (const Seq& s : stored3)
      for (int hv = 0; hv < nvar(mask(s, 0, 3)); ++hv) {
        const int gh = deposit(hv, mask(s, 0, 3));
        three.rec.push_back({cur(s, 0, 1, gh), cur(s, 1, 2, gh), cur(s, 2, 3, gh), cur(s, 0, 2, gh),
                             cur(s, 1, 3, gh), (uint16_t)(mask(s, 0, 1) | mask(s, 0, 2) << 8),
                             (uint16_t)mask(s, 0, 3)});
      }
    // canonical currents of length 4
    BgmPhase four(S::CV(4), S::F4);
    for (const Seq& s : can_[4])
      for (int hv = 0; hv < nvar(mask(s, 0, 4)); ++hv) {
        const int gh = deposit(hv, mask(s, 0, 4));
        std::vector<uint16_t> r;
        for (int L = 1; L <= 3; ++L)
          for (int a = 0; a + L <= 4; ++a) r.push_back(cur(s, a, a + L, gh));
        r.push_back((uint16_t)(mask(s, 0, 1) | mask(s, 0, 2) << 8));
        r.push_back((uint16_t)(mask(s, 0, 3) | mask(s, 0, 4) << 8));
        four.rec.push_back(r);
      }
    one.append(out);
    two.append(out);
    rtwo.append(out);
    three.append(out);
    four.append(out);
    if (N >= 5) {
      // canonical currents of length 5
      BgmPhase five(S::CV(5), S::F5);
      for (const Seq& s : can_[5])
        for (int hv = 0; hv < nvar(mask(s, 0, 5)); ++hv) {
          const int gh = deposit(hv, mask(s, 0, 5));
          std::vector<uint16_t> r;
          for (int L = 1; L <= 3; ++L)
            for (int a = 0; a + L <= 5; ++a) r.push_back(cur(s, a, a + L, gh));
          r.push_back(cur(s, 0, 4, gh));
          kk4(r, s, 1, 5, gh);
          r.push_back((uint16_t)(mask(s, 0, 1) | mask(s, 0, 2) << 8));
          r.push_back((uint16_t)(mask(s, 0, 3) | mask(s, 0, 4) << 8));
          r.push_back((uint16_t)mask(s, 0, 5));
          five.rec.push_back(r);
        }
      five.append(out);
    }
    if (N == 6) {
      // orderings of all six gluons that start with gluon 0
      BgmPhase six(S::CV(6), S::F6);
      for (const Seq& s : can_[N])
        for (int gh = 0; gh < S::NGH; ++gh) {
          std::vector<uint16_t> r;
          for (int L = 1; L <= 3; ++L)
            for (int a = 0; a + L <= 6; ++a) r.push_back(cur(s, a, a + L, gh));
          r.push_back(cur(s, 0, 4, gh));
          kk4(r, s, 1, 5, gh);
          kk4(r, s, 2, 6, gh);
          r.push_back((uint16_t)cvariant(part(s, 0, 5), gh));
          kk5(r, s, 1, 6, gh);
          r.push_back((uint16_t)(mask(s, 0, 1) | mask(s, 0, 2) << 8));
          r.push_back((uint16_t)(mask(s, 0, 3) | mask(s, 0, 4) << 8));
          r.push_back((uint16_t)mask(s, 0, 5));
          six.rec.push_back(r);
        }
      six.append(out);
    }
    // prefix items: sequences of length N - 1 (the last gluon follows from them), those
    // with gluon 0 inside first (two leaves each), by the position of gluon 0 and then
    // of gluon 1, so that the lanes of a wave expand into the same numbers of terms; six
    // gluons first by the gluons inside, so that items at work at the same time read the
    // same currents of length 5 from memory
    std::vector<Seq> order = full_[N - 1];
    auto pos = [](const Seq& s, int g) { return (int)(std::find(s.begin(), s.end(), g) - s.begin()); };
    std::stable_sort(order.begin(), order.end(), [&](const Seq& a, const Seq& b) {
      const int a0 = pos(a, 0), b0 = pos(b, 0);
      if (N == 6 && mask(a, 0, N - 1) != mask(b, 0, N - 1))
        return (a0 == N - 1) != (b0 == N - 1) ? a0 < b0 : mask(a, 0, N - 1) < mask(b, 0, N - 1);
      return a0 != b0 ? a0 < b0 : pos(a, 1) < pos(b, 1);
    });
    BgmPhase pre(S::VP, S::FP), leaf0(S::VP, S::FL), leaf1(S::VP2, S::FL);
    for (const Seq& s : order) {
      const int m = mask(s, 0, N - 1);
      int last = 0;
      while (m >> last & 1) ++last;
      Seq f = s;
      f.push_back(last);
      bool neg;
      const std::vector<Seq> qe = expand(f, &neg);
      for (int hv = 0; hv < nvar(m); ++hv) {
        const int gh = deposit(hv, m);
        std::vector<uint16_t> r{slot(S::R1S + variant(part(s, 0, 1), gh)), slot(S::R2S + variant(part(s, 0, 2), gh)),
                                cur(f, 2, 3, gh), cur(f, 1, 3, gh), cur(f, 0, 3, gh)};
        if (N == 5) {
          r.push_back(cur(f, 2, 4, gh));
          r.push_back(cur(f, 1, 4, gh));
          kk4(r, f, 0, 4, gh);
        }
        if (N == 6) {
          kk4(r, f, 0, 4, gh);
          for (int a : {1, 2, 3}) r.push_back(cur(f, a, 4, gh));
          kk5(r, f, 0, 5, gh);
          kk4(r, f, 1, 5, gh);
          for (int a : {2, 3}) r.push_back(cur(f, a, 5, gh));
          r.push_back((uint16_t)mask(f, 0, 3));
        }
        r.push_back((uint16_t)rank_.at(code(f)));
        for (int t = 0; t < S::QKK; ++t) r.push_back((uint16_t)rank_.at(code(qe[t < (int)qe.size() ? t : 0])));
        r.push_back(info(qe.size(), neg));
        pre.rec.push_back(r);
        for (int h = 0; h < (last ? 2 : 1); ++h) {
          const int gl = gh | (last ? h << (last - 1) : 0);
          std::vector<uint16_t> q;
          if (N == 5) {
            kk4(q, f, 1, 5, gl);
            q.push_back(cur(f, 2, 5, gl));
            q.push_back(slot(S::C2S + variant(part(f, 3, 5), gl)));
          } else if (N == 6) {
            kk5(q, f, 1, 6, gl);
            kk4(q, f, 2, 6, gl);
            q.push_back(cur(f, 3, 6, gl));
            q.push_back(slot(S::C2S + variant(part(f, 4, 6), gl)));
          } else {
            q.push_back(cur(f, 1, 4, gl));
            q.push_back(cur(f, 2, 4, gl));
          }
          q.push_back(slot(S::C1S + variant(part(f, N - 1, N), gl)));
          q.push_back((uint16_t)gl);
          (h ? leaf1 : leaf0).rec.push_back(q);
        }
      }
    }
    pre.append(out);
    leaf0.append(out);
    leaf1.append(out);
    return out;
  }
};

// The work-item tables of N gluons, built on first use (they depend on nothing else).
template <int N>
const std::vector<uint32_t>& bgm_items() {
  static const std::vector<uint32_t> items = BgmBuilder<N>().build();
  return items;
}

// Orbits of the orderings of n gluons under the exchanges of gluons 0 and 1, 2 and 3,
// (4 and 5) and the reversal, all of which leave the colour matrix unchanged, and the
// matrix in the sums and differences over them.  orb[o][b] = column of member b of
// orbit o (bit k of b applies the k-th symmetry to the first member); with
//   a_s[o] = sum_b (-1)^popcount(s & b) A(orb[o][b])
// the form sum_xy A_x C_xy A_y is sum_s sum_oo' a_s[o] sec[s][o][o'] a_s[o'].  (An
// orbit on which two members coincide counts each twice in a_s.)  All elements are
// integers over a power of two.
struct BgmSectors {
  int nsym = 0, norb = 0;
  std::vector<uint16_t> orb;   // [norb][2^nsym]
  std::vector<double> sec;     // [2^nsym][norb][norb]
};

inline BgmSectors bgm_sectors(int n, const int* cf) {
  std::vector<std::vector<int>> seqs;
  std::vector<int> s(n);
  for (int i = 0; i < n; ++i) s[i] = i;
  std::map<std::vector<int>, int> col;
  do {
    col[s] = (int)seqs.size();
    seqs.push_back(s);
  } while (std::next_permutation(s.begin(), s.end()));
  const int nex = n / 2, ncol = (int)seqs.size();
  BgmSectors r;
  r.nsym = nex + 1;
  const int G = 1 << r.nsym;
  auto act = [&](int b, std::vector<int> x) {
    for (int k = 0; k < nex; ++k)
      if (b >> k & 1)
        for (int& g : x)
          if (g / 2 == k) g ^= 1;
    if (b >> nex & 1) std::reverse(x.begin(), x.end());
    return x;
  };
  std::vector<bool> seen(ncol, false);
  for (int c = 0; c < ncol; ++c) {
    if (seen[c]) continue;
    for (int b = 0; b < G; ++b) {
      const int d = col.at(act(b, seqs[c]));
      seen[d] = true;
      r.orb.push_back((uint16_t)d);
    }
    ++r.norb;
  }
  r.sec.assign((size_t)G * r.norb * r.norb, 0.0);
  // members that coincide with an earlier one, and the sectors in which one coincides
  // with its own negative (a_s[o] is zero there)
  std::vector<bool> first((size_t)r.norb * G, true), null((size_t)r.norb * G, false);
  for (int o = 0; o < r.norb; ++o)
    for (int b = 0; b < G; ++b)
      for (int d = 0; d < b; ++d)
        if (r.orb[(size_t)o * G + b] == r.orb[(size_t)o * G + d]) {
          first[(size_t)o * G + b] = false;
          for (int s2 = 0; s2 < G; ++s2)
            if (__builtin_popcount(s2 & (b ^ d)) & 1) null[(size_t)o * G + s2] = true;
        }
  for (int o = 0; o < r.norb; ++o)
    for (int p = 0; p < r.norb; ++p) {
      // the projection of A on a sector is (-1)^popcount(s & b) a_s[o] / G at member b;
      // each distinct member once
      std::vector<double> by(G, 0.0);
      for (int b = 0; b < G; ++b)
        for (int c = 0; c < G; ++c)
          if (first[(size_t)o * G + b] && first[(size_t)p * G + c])
            by[b ^ c] += cf[(size_t)r.orb[(size_t)o * G + b] * ncol + r.orb[(size_t)p * G + c]];
      for (int s2 = 0; s2 < G; ++s2) {
        if (null[(size_t)o * G + s2] || null[(size_t)p * G + s2]) continue;
        double m = 0.0;
        for (int d = 0; d < G; ++d) m += __builtin_popcount(s2 & d) & 1 ? -by[d] : by[d];
        r.sec[((size_t)s2 * r.norb + o) * r.norb + p] = m / ((double)G * G);
      }
    }
  return r;
}

// The sectors as the kernels read them (FP32, exact): four orbits as they are, upper
// triangle with the elements above the diagonal doubled [8][4][4]; more orbits in the
// lane order of the matrix operand, 16 x 16 blocks (mb, kb >= mb) of each sector in turn,
// those above the diagonal doubled: element ((block) 4 + q) 64 + l =
// sec[s][16 mb + l % 16][16 kb + 4 q + l / 16].
inline std::vector<float> bgm_sector_operands(const BgmSectors& s) {
  std::vector<float> r;
  const int G = 1 << s.nsym, n = s.norb;
  auto at = [&](int k, int i, int j) { return (float)s.sec[((size_t)k * n + i) * n + j]; };
  for (int k = 0; k < G; ++k) {
    if (n == 4) {
      for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) r.push_back(j < i ? 0.0f : j == i ? at(k, i, j) : 2.0f * at(k, i, j));
    } else {
      for (int mb = 0; mb < n / 16; ++mb)
        for (int kb = mb; kb < n / 16; ++kb)
          for (int q = 0; q < 4; ++q)
            for (int l = 0; l < 64; ++l)
              r.push_back((kb > mb ? 2.0f : 1.0f) * at(k, 16 * mb + l % 16, 16 * kb + 4 * q + l / 16));
    }
  }
  return r;
}

}  // namespace me
