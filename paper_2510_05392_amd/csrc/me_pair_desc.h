// Arguments of the one-launch kernels of the processes with few flows (me_pair.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace me {

// The mirror pairs (h, all - 1 - h) of helicities that hold a good one: the lower index of
// the pair, its number of good helicities in the upper half.
inline std::vector<int> mirror_pairs(const std::vector<int>& good, int all) {
  std::vector<int> count(all, 0), pairs;
  for (int h : good) ++count[std::min(h, all - 1 - h)];
  for (int h = 0; h < all; ++h)
    if (count[h]) pairs.push_back(h | count[h] << 16);
  return pairs;
}

struct PairArgs {
  const double* mom;      // device, [n][npar][4]
  int64_t n;
  double g, mt;
  const int* pairs;       // device: helicity | weight << 16, one per mirror pair with a good helicity
  int npair;
  const double* alphas;   // device [n] (replaces g), or nullptr
  double* out;            // |M|^2 [n]
  double scale;
  hipStream_t stream;
};
using PairLauncher = hipError_t (*)(const PairArgs&);

}  // namespace me
