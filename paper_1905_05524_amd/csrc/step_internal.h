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

// A value with the rounding of the operation that gave it: the compiler may not
// contract that operation into a sum that takes the value.  Where kernels share
// their arithmetic but not their data paths (one sums in registers what another
// passes through LDS) the products either meet their sums in explicit fused
// operations or pass through here, so that results agree bit for bit.
__device__ inline double rounded(double v) {
  asm("" : "+v"(v));
  return v;
}

// A wavefront-uniform table read through scalar loads (opaque, so that the
// entries are loaded where they are used instead of being held).
typedef const __attribute__((address_space(4))) double* ctab;
__device__ inline ctab scalar_table(const double* g) {
  asm volatile("" : "+s"(g));
  return (ctab)g;
}

// out = T in for a centro-antisymmetric T in even-odd form (layout with
// GTab): 36 operations instead of 49 at n = 7.
template <int n>
struct EO {
  static constexpr int h = n / 2, mid = (n - 1) / 2;
  double A[h][h], B[h][h], C[h], M[h];
  __device__ explicit EO(ctab g) {
#pragma unroll
    for (int i = 0; i < h; ++i) {
#pragma unroll
      for (int m = 0; m < h; ++m) { A[i][m] = g[i * h + m]; B[i][m] = g[h * h + i * h + m]; }
      C[i] = n % 2 ? g[2 * h * h + i] : 0.0;
      M[i] = n % 2 ? g[2 * h * h + h + i] : 0.0;
    }
  }
  __device__ inline void apply(const double in[n], double out[n]) const {
    double e[h], o[h];
#pragma unroll
    for (int m = 0; m < h; ++m) { e[m] = in[m] + in[n - 1 - m]; o[m] = in[m] - in[n - 1 - m]; }
    double mv = in[mid];
    if constexpr (n % 2) {
      double S = M[0] * o[0];
#pragma unroll
      for (int m = 1; m < h; ++m) S = fma(M[m], o[m], S);
      out[mid] = h == 1 ? rounded(S) : S;   // a bare product at n = 3
    }
    if constexpr (h == 1) {
      double U = B[0][0] * e[0];
      if constexpr (n % 2) U = fma(C[0], mv, U);
      else U = rounded(U);
      out[0] = fma(A[0][0], o[0], U);
      out[n - 1] = fma(A[0][0], o[0], -U);
      return;
    }
#pragma unroll
    for (int i = 0; i < h; ++i) {
      double S = A[i][0] * o[0], U = B[i][0] * e[0];
#pragma unroll
      for (int m = 1; m < h; ++m) { S = fma(A[i][m], o[m], S); U = fma(B[i][m], e[m], U); }
      if constexpr (n % 2) U = fma(C[i], mv, U);
      out[i] = S + U;
      out[n - 1 - i] = S - U;
    }
  }
};

// Per-launch and per-cell constants of the flux.
struct FluxC {
  double gm1, hgm1, mu, mu23, kap, gh;   // gm1, gm1/2, mu/h, (2/3) mu/h, kappa/(h R), g h
  double gz, pb;                         // g z and background pressure of the lane's row
};

struct StepArgs {
  const double* Qin;    // [C][4][n][n]
  double* Qout;         // corrector output (may alias Qin)
  double* Qs;           // [C][4][n][n]  Q* = Q^n + dt (volume + source)
  double* FD;           // [C][4 faces][2][4][n]
  double* dtc;          // [C] per-cell CFL candidates
  double* clock;        // [S][4]: t, dt, (unused), steps
  const int* scen;      // [C] scenario of each cell (NULL: scenario 0)
  const double* geom;   // [C][4]
  const double* bg;     // [C][n + 2][2]
  const int* nbr;       // [C][4][4]
  const double* gtab;
  double* iter_store;   // optional [C][iters][n][4][n][n]: Picard iterates q^1..q^I (adjoint)
  double* advance;      // optional clock [4] the corrector advances (t += dt, steps += 1)
  int C, iters;
};

// kernel arguments of a group's bound buffers
StepArgs make_args(const Group& g);

}  // namespace adg
