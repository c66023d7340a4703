// What the step kernels' translation units share: the kernel arguments and
// small device helpers.
#pragma once

#include "adg_internal.h"

namespace adg {

// most cells per wavefront for n nodes per direction (at most four)
constexpr int max_cpw_c(int n) { return (4 * n * n <= kWave) ? 4 : ((2 * n * n <= kWave) ? 2 : 1); }

// A wave-uniform double moved to scalar registers.
__device__ inline double uniform(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

struct StepArgs {
  const double* Qin;    // [C][4][n][n]
  double* Qout;         // corrector output (may alias Qin)
  double* Qs;           // [C][4][n][n]  Q* = Q^n + dt (volume + source)
  double* FD;           // [C][4 faces][2][4][n]
  double* dtc;          // [C] per-cell CFL candidates
  double* clock;        // [S][4]: t, dt, (unused), steps
  const int* scen;      // [C] scenario of each cell (NULL: scenario 0)
  const double* geom;   // [C][4]
  const int* nbr;       // [C][4][4]
  const double* gtab;
  double* iter_store;   // optional [C][iters][n][4][n][n]: Picard iterates q^1..q^I (adjoint)
  double* advance;      // optional clock [4] the corrector advances (t += dt, steps += 1)
  int C, iters;
};

// kernel arguments of a group's bound buffers
StepArgs make_args(const Group& g);

}  // namespace adg
