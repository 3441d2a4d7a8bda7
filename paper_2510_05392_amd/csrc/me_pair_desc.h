// Arguments of the one-launch kernels of the processes with few flows (me_pair.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace me {

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
