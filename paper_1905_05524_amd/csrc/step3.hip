// Three-dimensional ADER-DG step kernels for gfx950 on a uniform grid of
// cubes: space-time predictor, corrector with the viscous Rusanov face flux
// (periodic and wall faces) and the CFL candidate of every cell, initial
// states and the health check.
//
// Work decomposition of the corrector, the time step and the predictor of
// N = 1 and 2.  A workgroup of kThreads3 threads holds CB cells; the
// thread t owns spatial node t % nd (nd = n^3) of cell slot t / nd, so a
// cell's nodes are consecutive lanes.  For n = 2 and n = 4 every cell lies in
// one wavefront and the LDS hand-offs between its nodes need only a
// wavefront barrier; otherwise cells straddle wavefronts and the workgroup
// synchronises.  Threads past CB * nd (when nd does not divide the
// workgroup) mirror the threads of slot 0: same cell, same node, hence the
// same values written to the same LDS addresses, and no global stores.
// Tensor-product contractions along x, y and z read n values of an LDS slice
// per output; the space-time iterate of a node (n time levels x 5 variables)
// stays in registers.  The predictor of N = 3 (k_pred3_w64) keeps that layout
// with one wavefront per cell and contracts with matrix instructions; those of
// N = 4 and 5 (k_pred3_rows) work on all time levels at once.
#include "adg3_internal.h"
#include "step_internal.h"

namespace adg {

constexpr int kThreads3 = 256;

template <int n>
struct Cfg3 {
  static constexpr int nn = n * n, nd = n * n * n;
  static constexpr int CB = kThreads3 / nd;               // cells per workgroup
  static constexpr bool spare = CB * nd != kThreads3;      // threads without a cell
  static constexpr bool WL = (kWave % nd == 0);           // cells never straddle a wavefront
  static constexpr int pred_slot = 20 * nd;               // state slice [5][nd] + fluxes [3][5][nd]
  static constexpr int corr_slot = 30 * nn + 12 * nn + 2; // G [6][5][nn], speeds [2][6 nn], maxima [2]
};

template <bool WL>
__device__ inline void sync3() {
  if constexpr (WL) wave_sync();
  else __syncthreads();
}

// ---------------------------------------------------------------- physics
__device__ inline double pressure3(const Phys& ph, const double q[5], double z) {
  const double geo = q[0] * (ph.geff * z);
  return ph.gm1 * (q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0] - geo);
}

// Per-launch and per-lane constants of the flux: the 1/h of the viscous and
// heat fluxes (gradients are in reference coordinates, h times the physical
// ones) sits in mu, mu2, mu23, kap and gh.
struct FluxC3 {
  double gm1, hgm1, mu, mu2, mu23, kap, gh;   // gm1, gm1/2, mu/h, 2 mu/h, (2/3) mu/h, kappa/(h R), g h
  double gz, pb;                              // g z and background pressure at the node
};
__device__ inline FluxC3 flux_consts3(const Phys& ph, double h) {
  FluxC3 c;
  c.gm1 = ph.gm1;
  c.hgm1 = 0.5 * ph.gm1;
  c.mu = ph.mu / h;
  c.mu2 = 2.0 * c.mu;
  c.mu23 = (2.0 / 3.0) * c.mu;
  c.kap = ph.kappa / h * ph.iR;
  c.gh = ph.geff * h;
  c.gz = 0.0;
  c.pb = 0.0;
  return c;
}

// Momentum and energy fluxes F[d][0..3] along x, y, z at one node: the
// equation set of Section 2 in three dimensions (eqs. equation-set, eos,
// temperature, stress-tensor, heat-conduction-coeff,
// momentum-equation-split).  q: state, g[d]: its gradient along d in
// reference coordinates.  The mass fluxes are the momenta and are left out;
// a[c][d] = rho du_c/dx_d, so that the divisions by rho collect in ir, and the
// off-diagonal fluxes m_a u_b + sigma_ab are symmetric and formed once.
__device__ inline void flux_xyz(const FluxC3& k, const double q[5], const double g[3][5], double F[3][4]) {
  const double rho = q[0], E = q[4];
  const double ir = recip(rho);
  const double u[3] = {q[1] * ir, q[2] * ir, q[3] * ir};
  const double ke = fma(q[1], u[0], fma(q[2], u[1], q[3] * u[2]));   // rho |v|^2
  const double p = fma(-k.hgm1, ke, k.gm1 * fma(-k.gz, rho, E));
  const double pm = p - k.pb, pir = p * ir;                          // pir = R T
  double a[3][3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) a[c][d] = fma(-u[c], g[d][0], g[d][1 + c]);
  const double hv = fma(0.5 * ir, ke, k.gz);
  double Qd[3];                                                      // gm1 dp' - R T drho: heat flux along d
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double dp = fma(-u[2], a[2][d], fma(-u[1], a[1][d], fma(-u[0], a[0][d], fma(-hv, g[d][0], g[d][4]))));
    if (d == 2) dp = fma(-k.gh, rho, dp);
    Qd[d] = fma(-pir, g[d][0], k.gm1 * dp);
  }
  const double m = k.mu * ir, m2 = k.mu2 * ir;
  const double t = (k.mu23 * ir) * ((a[0][0] + a[1][1]) + a[2][2]);
  const double s01 = -m * (a[0][1] + a[1][0]), s02 = -m * (a[0][2] + a[2][0]), s12 = -m * (a[1][2] + a[2][1]);
  const double kk = k.kap * ir, H = E + p;
  const double s0 = fma(-m2, a[0][0], t), s1 = fma(-m2, a[1][1], t), s2 = fma(-m2, a[2][2], t);
  F[0][0] = fma(q[1], u[0], pm + s0);
  F[1][1] = fma(q[2], u[1], pm + s1);
  F[2][2] = fma(q[3], u[2], pm + s2);
  F[0][1] = F[1][0] = fma(q[1], u[1], s01);
  F[0][2] = F[2][0] = fma(q[1], u[2], s02);
  F[1][2] = F[2][1] = fma(q[2], u[2], s12);
  F[0][3] = fma(-kk, Qd[0], fma(u[2], s02, fma(u[1], s01, u[0] * (H + s0))));
  F[1][3] = fma(-kk, Qd[1], fma(u[2], s12, fma(u[0], s01, u[1] * (H + s1))));
  F[2][3] = fma(-kk, Qd[2], fma(u[1], s12, fma(u[0], s02, u[2] * (H + s2))));
}

// speed of sound, ir = 1/rho (one reciprocal and one square root per state)
__device__ inline double sound3(const Phys& ph, const double q[5], double ir, double z) {
  const double ke = fma(q[1], q[1], fma(q[2], q[2], q[3] * q[3])) * ir;   // rho |v|^2
  const double p = ph.gm1 * (fma(-0.5, ke, q[4]) - q[0] * (ph.geff * z));
  return root(ph.gamma * p * ir);
}

// largest wave speed along d and the viscous speed at a face node
__device__ inline void eig3(const Phys& ph, int d, const double q[5], double zf, double& lam, double& lv) {
  const double ir = recip(q[0]);
  const double mx = q[1], my = q[2], mz = q[3];
  const double un = d == 0 ? mx : (d == 1 ? my : mz);
  lam = fabs(un * ir) + sound3(ph, q, ir, zf);
  lv = ph.lv_coef * ir;
}

// No-slip wall with normal direction d (Section 4.2): the ghost carries the
// background density and pressure at the face height with the mirrored
// velocity; its normal flux mirrors the interior one for mass and energy
// (the energy flux around twice the background heat flux kappa g / cp through
// horizontal walls) and repeats it for the momenta.  Without gravity the
// interior density and pressure stand in for the background.
// bg: the background at the face node.
__device__ inline void wall_ghost3(const Phys& ph, int d, double zf, const double bg[2], const double Qi[5],
                                   const double Fi[5], double Qg[5], double Fg[5]) {
  const double ir = 1.0 / Qi[0];
  const double u[3] = {Qi[1] * ir, Qi[2] * ir, Qi[3] * ir};
  double rb, pb;
  if (ph.gravity) { rb = bg[0]; pb = bg[1]; }
  else { rb = Qi[0]; pb = pressure3(ph, Qi, zf); }
  const double geo = ph.gravity ? rb * (ph.g * zf) : 0.0;
  Qg[0] = rb;
#pragma unroll
  for (int a = 0; a < 3; ++a) Qg[1 + a] = -(rb * u[a]);
  Qg[4] = pb / ph.gm1 + 0.5 * rb * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) + geo;
  const double qbg = (ph.gravity && d == 2) ? ph.kappa * ph.g / ph.cp : 0.0;
  Fg[0] = -Fi[0];
#pragma unroll
  for (int a = 0; a < 3; ++a) Fg[1 + a] = Fi[1 + a];
  Fg[4] = 2.0 * qbg - Fi[4];
}

// Background density and pressure at the node rows, the bottom and the top of
// every layer of cells, once per handle: the predictor would spend a tenth of its instructions on
// the power function (250 of 2,500 to 4,500 per node at n = 2 to 4).
__global__ void k_background3(Phys ph, Args3 a, int n, double* bg) {
  const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long long)a.nz * (n + 2)) return;
  const int ck = (int)(g / (n + 2)), k = (int)(g % (n + 2));
  const double zc = a.z0 + ck * a.h;
  double rb, pb;
  background(ph, k < n ? zc + a.h * a.gtab[GTab::XI * n + k] : (k > n ? zc + a.h : zc), rb, pb);
  bg[2 * g] = rb;
  bg[2 * g + 1] = pb;
}

// ---------------------------------------------------------------- predictor
// Gradient of the slice src ([5][nd] in LDS) at node (k, j, i) along x, y, z
// with the derivative-matrix rows of the node, then the flux and source.
template <int n>
__device__ inline void grad_flux3(const FluxC3& fc, const double* src, int i, int j, int k, const double Di[n],
                                  const double Dj[n], const double Dk[n], const double q[5], double F[3][5]) {
  constexpr int nn = n * n, nd = nn * n;
  double g[3][5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double* s = src + v * nd;
    double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
    for (int m = 0; m < n; ++m) {
      gx = fma(Di[m], s[(k * n + j) * n + m], gx);
      gy = fma(Dj[m], s[(k * n + m) * n + i], gy);
      gz = fma(Dk[m], s[(m * n + j) * n + i], gz);
    }
    g[0][v] = gx; g[1][v] = gy; g[2][v] = gz;
  }
  double F4[3][4];
  flux_xyz(fc, q, g, F4);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    F[d][0] = q[1 + d];
#pragma unroll
    for (int v = 0; v < 4; ++v) F[d][1 + v] = F4[d][v];
  }
}

// sum over the three directions of the contraction of the flux components
// ([3][5][nd] in LDS) with the rows Ti, Tj, Tk: the divergence for the
// derivative matrix, the volume term for the weighted transposed one
template <int n>
__device__ inline double div3(const double* sF, int v, int i, int j, int k, const double Ti[n], const double Tj[n],
                              const double Tk[n]) {
  constexpr int nn = n * n, nd = nn * n;
  const double* fx = sF + v * nd;
  const double* fy = sF + (5 + v) * nd;
  const double* fz = sF + (10 + v) * nd;
  double s = 0.0;
#pragma unroll
  for (int m = 0; m < n; ++m) {
    s = fma(Ti[m], fx[(k * n + j) * n + m], s);
    s = fma(Tj[m], fy[(k * n + m) * n + i], s);
    s = fma(Tk[m], fz[(m * n + j) * n + i], s);
  }
  return s;
}

// Face data FD[f][kind][v][s][t] of one cell from its averaged state sq
// ([5][nd]) and fluxes sF ([3][5][nd]) in LDS: kind 0 the state, 1 the normal
// flux, extrapolated along the face normal with the boundary values of the
// basis.  The cell's nd threads (r = node index) share the 60 n^2 outputs.
template <int n>
__device__ inline void face_data3(const Tab<n>& tb, const double* sq, const double* sF, double* FDc, int r) {
  constexpr int nn = n * n, nd = nn * n;
  for (int o = r; o < 60 * nn; o += nd) {
    const int f = o / (10 * nn), rem = o - f * 10 * nn;
    const int kind = rem / (5 * nn), v = (rem / nn) % 5, st = rem % nn, s = st / n, t = st % n;
    const int d = f >> 1;
    const double* src = kind ? sF + (d * 5 + v) * nd : sq + v * nd;
    const int base = d == 0 ? (s * n + t) * n : (d == 1 ? s * nn + t : s * n + t);
    const int stride = d == 0 ? 1 : (d == 1 ? n : nn);
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < n; ++m) acc = fma((f & 1) ? tb.e1[m] : tb.e0[m], src[base + m * stride], acc);
    FDc[o] = acc;
  }
}

// Space-time predictor (Section 3): Picard sweeps
//   X_a = Q + dt sum_b P_ab R(X_b),  R = S - div F,  P = K1^{-1} W,
// from X_a = Q, then the time averages of state, flux and source, the update
// Q* = Q + dt (volume term of the averaged flux / h + averaged source) and
// the face data (averaged state and normal flux extrapolated to each face).
template <int n>
__global__ __launch_bounds__(kThreads3) void k_pred3(Phys ph, Tab<n> tb, Args3 a) {
  using G = Cfg3<n>;
  constexpr int nn = G::nn, nd = G::nd;
  constexpr bool WL = G::WL;
  extern __shared__ double lds[];
  const int tid = threadIdx.x, r = tid % nd;
  const bool mirror = G::spare && tid >= G::CB * nd;
  const int slot = mirror ? 0 : tid / nd;
  const int cell = blockIdx.x * G::CB + slot;
  const bool valid = !mirror && cell < a.C;
  const int c = cell < a.C ? cell : a.C - 1;   // loads stay in bounds; only valid threads store
  double* sq = lds + slot * G::pred_slot;
  double* sF = sq + 5 * nd;
  const int i = r % n, j = (r / n) % n, k = r / nn;
  const double h = a.h;
  const int ck = c / (a.nx * a.ny);
  const double z = (a.z0 + ck * h) + h * a.gtab[GTab::XI * n + k];
  const double rb = a.bg[2 * (ck * (n + 2) + k)];
  FluxC3 fc = flux_consts3(ph, h);
  fc.gz = ph.geff * z;
  fc.pb = a.bg[2 * (ck * (n + 2) + k) + 1];
  const double dt = a.clock[1], sdt = -dt / h;
  double Di[n], Dj[n], Dk[n];
#pragma unroll
  for (int m = 0; m < n; ++m) {
    Di[m] = a.gtab[GTab::d(n) + i * n + m];
    Dj[m] = a.gtab[GTab::d(n) + j * n + m];
    Dk[m] = a.gtab[GTab::d(n) + k * n + m];
  }
  const double* Qc = a.Q + (size_t)c * 5 * nd;
  double Q0[5], X[n][5], R[n][5];
#pragma unroll
  for (int v = 0; v < 5; ++v) Q0[v] = Qc[v * nd + r];
#pragma unroll
  for (int b = 0; b < n; ++b)
#pragma unroll
    for (int v = 0; v < 5; ++v) X[b][v] = Q0[v];

  for (int it = 0; it < a.iters; ++it) {
#pragma unroll
    for (int b = 0; b < n; ++b) {
      if (b > 0 && it == 0) {
        // the first sweep starts from Q^n at every time level: all levels
        // share level 0's residual (bit for bit)
#pragma unroll
        for (int v = 0; v < 5; ++v) R[b][v] = R[0][v];
        continue;
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) sq[v * nd + r] = X[b][v];
      sync3<WL>();
      double F[3][5];
      const double Sw = -ph.geff * (X[b][0] - rb);
      grad_flux3<n>(fc, sq, i, j, k, Di, Dj, Dk, X[b], F);
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int v = 0; v < 5; ++v) sF[(d * 5 + v) * nd + r] = F[d][v];
      sync3<WL>();
#pragma unroll
      for (int v = 0; v < 5; ++v) R[b][v] = sdt * div3<n>(sF, v, i, j, k, Di, Dj, Dk);
      R[b][3] = fma(dt, Sw, R[b][3]);
    }
#pragma unroll
    for (int a2 = 0; a2 < n; ++a2)
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < n; ++b) s = fma(tb.P[a2][b], R[b][v], s);
        X[a2][v] = Q0[v] + s;
      }
  }

  // time averages; the slice alternates between two LDS buffers so that one
  // barrier per time level suffices
  double Qb[5], Fb[3][5], Sb = 0.0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    Qb[v] = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) Fb[d][v] = 0.0;
  }
#pragma unroll
  for (int b = 0; b < n; ++b) {
    double* buf = (b & 1) ? sF : sq;
#pragma unroll
    for (int v = 0; v < 5; ++v) buf[v * nd + r] = X[b][v];
    sync3<WL>();
    double F[3][5];
    const double Sw = -ph.geff * (X[b][0] - rb);
    grad_flux3<n>(fc, buf, i, j, k, Di, Dj, Dk, X[b], F);
    const double w = tb.w[b];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Qb[v] = fma(w, X[b][v], Qb[v]);
#pragma unroll
      for (int d = 0; d < 3; ++d) Fb[d][v] = fma(w, F[d][v], Fb[d][v]);
    }
    Sb = fma(w, Sw, Sb);
  }
  sync3<WL>();
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    sq[v * nd + r] = Qb[v];
#pragma unroll
    for (int d = 0; d < 3; ++d) sF[(d * 5 + v) * nd + r] = Fb[d][v];
  }
  sync3<WL>();

  // volume term (Dw[i][m] = w_m D[m][i] / w_i along each direction) and Q*
  double Wi[n], Wj[n], Wk[n];
#pragma unroll
  for (int m = 0; m < n; ++m) {
    Wi[m] = a.gtab[GTab::dw(n) + i * n + m];
    Wj[m] = a.gtab[GTab::dw(n) + j * n + m];
    Wk[m] = a.gtab[GTab::dw(n) + k * n + m];
  }
  const double ih = 1.0 / h;
  if (valid) {
    double* Qsc = a.Qs + (size_t)c * 5 * nd;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double vol = div3<n>(sF, v, i, j, k, Wi, Wj, Wk);
      Qsc[v * nd + r] = Q0[v] + dt * (vol * ih + (v == 3 ? Sb : 0.0));
    }
    face_data3<n>(tb, sq, sF, a.FD + (size_t)c * 60 * nn, r);
  }
}

// X <- K1^{-1} W X over the time levels: in-place solve with the unpivoted LU
// factors, the weights folded into them
template <int n>
__device__ inline void solve_time(const double* lu, double X[n][5]) {
  int o = 0;
#pragma unroll
  for (int ii = 1; ii < n; ++ii) {
#pragma unroll
    for (int jj = 0; jj < ii; ++jj) {
      const double l = lu[o++];
#pragma unroll
      for (int v = 0; v < 5; ++v) X[ii][v] = fma(-l, X[jj][v], X[ii][v]);
    }
  }
#pragma unroll
  for (int ii = n - 1; ii >= 0; --ii) {
    const double iu = lu[o++];
#pragma unroll
    for (int v = 0; v < 5; ++v) X[ii][v] *= iu;
#pragma unroll
    for (int jj = ii + 1; jj < n; ++jj) {
      const double u = lu[o++];
#pragma unroll
      for (int v = 0; v < 5; ++v) X[ii][v] = fma(-u, X[jj][v], X[ii][v]);
    }
  }
}

// ------------------------------------------------ predictor, n = 4 (N = 3)
// One cell per wavefront, lane l = 16 k + 4 j + i, the four time levels of a
// node in registers.  Lines of four nodes are what one 4 x 4 x 4 matrix
// instruction (four blocks, here the four rows j) contracts: along z
// directly (the lane bits of k are the contracted ones), along x after a
// transposition of every x-z plane, itself a product with the identity
// (exact).  A matrix instruction takes the time of four vector FMAs, so a z
// contraction costs what its FMAs would and an x contraction twice that, with
// no lane exchange; the y contractions go through LDS (one slice of the
// variables, three values read per output beside the lane's own).
// Bound by the FP64 issue rate: per cell 3,390 vector and 451 matrix
// instructions (8,820 vector ones when the x and z operands moved through the
// DPP network, six moves per contraction, and the background's power function
// ran per lane).  25^3 cells, 4 iterations: 172 us, 238 us before.  Three
// waves per SIMD: at four (128 registers) the sweep spills, 187 us.

// D[i][j] = sum_k A[i][k] B[k][j] + C[i][j] in every block b, with A in lane
// 16 k + 4 b + i, B in lane 16 k + 4 b + j, C and D in lane 16 i + 4 b + j
__device__ inline double mm4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
// tables of the lane for a matrix T: its entry at (lane bits 0-1, bits 4-5),
// and its row for the y contraction, own node first, then the nodes one, two
// and three steps further
struct Tab4 {
  double T, y[4];
};
__device__ inline Tab4 tab4(const double* g, int lane) {
  const int lo = lane & 3, j = (lane >> 2) & 3, k = lane >> 4;
  Tab4 t;
  t.T = g[lo * 4 + k];
#pragma unroll
  for (int m = 0; m < 4; ++m) t.y[m] = g[j * 4 + ((j + m) & 3)];
  return t;
}
// the lane's node m steps further along y
__device__ inline int step_y(int lane, int m) { return (lane & 51) | ((lane + 4 * m) & 12); }

// Workgroups of one wavefront: LDS and barriers are per cell anyway, and the
// last round of workgroups ends sooner (four cells: 173.7 us at 25^3).
constexpr int kW64Cells = 1;
__global__ __launch_bounds__(kWave * kW64Cells, 3) void k_pred3_w64(Phys ph, Tab<4> tb, Args3 a) {
  constexpr int n = 4, nd = 64;
  extern __shared__ double lds[];
  const int tid = threadIdx.x, slot = tid >> 6, r = tid & 63;
  const int cell = blockIdx.x * kW64Cells + slot;
  const bool valid = cell < a.C;
  const int c = valid ? cell : a.C - 1;   // loads stay in bounds; nothing is stored for such lanes
  double* sq = lds + slot * 20 * nd;      // state slice [5][nd]; the averaged state in the epilogue
  double* sF = sq + 5 * nd;               // y fluxes [4][nd]; all averaged fluxes [3][5][nd] in the epilogue
  const int k = r >> 4;
  const double h = a.h;
  const int ck = c / (a.nx * a.ny);
  const double z = (a.z0 + ck * h) + h * a.gtab[GTab::XI * n + k];
  const double rb = a.bg[2 * (ck * (n + 2) + k)];
  FluxC3 fc = flux_consts3(ph, h);
  fc.gz = ph.geff * z;
  fc.pb = a.bg[2 * (ck * (n + 2) + k) + 1];
  const double dt = a.clock[1], ih = 1.0 / h;
  const Tab4 D = tab4(a.gtab + GTab::d(n), r);
  const double one = (r & 3) == (r >> 4) ? 1.0 : 0.0;
  const int y1 = step_y(r, 1), y2 = step_y(r, 2), y3 = step_y(r, 3);
  const double* Qc = a.Q + (size_t)c * 5 * nd + r;
  double X[n][5];
#pragma unroll
  for (int b = 0; b < n; ++b)
#pragma unroll
    for (int v = 0; v < 5; ++v) X[b][v] = Qc[v * nd];

  // gradients of one level: its slice to LDS for y, x and z in registers
  auto gradients = [&](const double q[5], double g[3][5]) {
#pragma unroll
    for (int v = 0; v < 5; ++v) sq[v * nd + r] = q[v];
    wave_sync();
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      g[0][v] = mm4(mm4(q[v], one, 0.0), D.T, 0.0);
      g[2][v] = mm4(D.T, q[v], 0.0);
      const double* s = sq + v * nd;
      g[1][v] = fma(D.y[3], s[y3], fma(D.y[2], s[y2], fma(D.y[1], s[y1], D.y[0] * q[v])));
    }
  };

  for (int it = 0; it < a.iters; ++it) {
#pragma unroll
    for (int b = 0; b < n; ++b) {
      if (b > 0 && it == 0) {
        // the first sweep starts from Q^n at every time level: all levels
        // share level 0's residual (bit for bit)
#pragma unroll
        for (int v = 0; v < 5; ++v) X[b][v] = X[0][v];
        continue;
      }
      double g[3][5], F[3][4];
      gradients(X[b], g);
      flux_xyz(fc, X[b], g, F);
#pragma unroll
      for (int v = 0; v < 4; ++v) sF[v * nd + r] = F[1][v];
      wave_sync();
      // the residual of time level b (times -h) replaces its iterate; the
      // mass flux is the momentum, its divergence a sum of gradients
      const double src = fc.gh * (X[b][0] - rb);
      X[b][0] = (g[0][1] + g[1][2]) + g[2][3];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double* s = sF + v * nd;
        double acc = mm4(D.T, F[2][v], mm4(mm4(F[0][v], one, 0.0), D.T, 0.0));
        acc = fma(D.y[0], F[1][v], acc);
        acc = fma(D.y[1], s[y1], acc);
        acc = fma(D.y[2], s[y2], acc);
        acc = fma(D.y[3], s[y3], acc);
        X[b][1 + v] = v == 2 ? acc + src : acc;
      }
      wave_sync();
    }
    // X <- Q - (dt/h) K1^{-1} W X
    solve_time<n>(a.gtab + GTab::lu(n), X);
    const double sdt = -dt * ih;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double q0 = Qc[v * nd];
#pragma unroll
      for (int a2 = 0; a2 < n; ++a2) X[a2][v] = fma(sdt, X[a2][v], q0);
    }
  }

  // time averages; the averaged fluxes accumulate in the lane's own LDS
  // words [3][5][nd] (registers are short here), the state in registers
  double Qb[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) Qb[v] = 0.0;
#pragma unroll
  for (int b = 0; b < n; ++b) {
    double g[3][5], F[3][4];
    gradients(X[b], g);
    flux_xyz(fc, X[b], g, F);
    const double w = tb.w[b];
#pragma unroll
    for (int v = 0; v < 5; ++v) Qb[v] = fma(w, X[b][v], Qb[v]);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double* acc = sF + (d * 5 + 1 + v) * nd + r;
        *acc = b == 0 ? w * F[d][v] : fma(w, F[d][v], *acc);
      }
    wave_sync();
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) sq[v * nd + r] = Qb[v];
#pragma unroll
  for (int d = 0; d < 3; ++d) sF[d * 5 * nd + r] = Qb[1 + d];
  const double Sb = -ph.geff * (Qb[0] - rb);
  wave_sync();

  // Lane indices and cell again from the thread id: kept live across the
  // sweeps they would occupy registers that the sweeps need (and spill).
  int t2 = threadIdx.x;
  asm volatile("" : "+v"(t2));
  const int r2 = t2 & 63;
  const int cell2 = blockIdx.x * kW64Cells + (t2 >> 6);
  // Volume term with the weighted transposed derivative matrix, and the face
  // data: the values at both ends of a line are a product with the two rows
  // e0, e1 (lanes with k = 0 and 1 hold the lower and the upper face's nodes);
  // along y from LDS.
  const int lo2 = r2 & 3, j2 = (r2 >> 2) & 3, k2 = r2 >> 4;
  const Tab4 W = tab4(a.gtab + GTab::dw(n), r2);
  const double one2 = lo2 == k2 ? 1.0 : 0.0;
  const double E = lo2 < 2 ? a.gtab[(lo2 == 0 ? GTab::E0 : GTab::E1) * n + k2] : 0.0;
  const bool ok = cell2 < a.C;
  double* FDc = a.FD + (size_t)(ok ? cell2 : 0) * 60 * 16;
  double* Qsc = a.Qs + (size_t)(ok ? cell2 : 0) * 5 * nd;
  const double* Q2 = a.Q + (size_t)(ok ? cell2 : 0) * 5 * nd;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double q = sq[v * nd + r2], fx = sF[v * nd + r2], fy = sF[(5 + v) * nd + r2], fz = sF[(10 + v) * nd + r2];
    const double qt = mm4(q, one2, 0.0), fxt = mm4(fx, one2, 0.0);   // x and z exchanged
    double acc = mm4(W.T, fz, mm4(fxt, W.T, 0.0));
    const double* s = sF + (5 + v) * nd;
    acc = fma(W.y[0], fy, acc);
#pragma unroll
    for (int m = 1; m < 4; ++m) acc = fma(W.y[m], s[step_y(r2, m)], acc);
    const double xq = mm4(E, qt, 0.0), xf = mm4(E, fxt, 0.0), zq = mm4(E, q, 0.0), zf = mm4(E, fz, 0.0);
    if (ok) {
      Qsc[v * nd + r2] = fma(dt, fma(acc, ih, v == 3 ? Sb : 0.0), Q2[v * nd + r2]);
      if (k2 < 2) {
        double* fx0 = FDc + (k2 * 10 + v) * 16 + lo2 * 4 + j2;        // faces 0, 1: nodes (z, y)
        fx0[0] = xq;
        fx0[5 * 16] = xf;
        double* fz0 = FDc + ((4 + k2) * 10 + v) * 16 + j2 * 4 + lo2;  // faces 4, 5: nodes (y, x)
        fz0[0] = zq;
        fz0[5 * 16] = zf;
      }
    }
  }
  // faces 2, 3: nodes (z, x), 20 lines of 16 nodes
#pragma unroll
  for (int it = 0; it < 5; ++it) {
    const int q = it * 4 + k2, hi = q >= 10, kv = hi ? q - 10 : q;   // face, (kind, variable)
    const int st = r2 & 15, zz = st >> 2, xx = st & 3;
    const double* s = (kv < 5 ? sq + kv * nd : sF + kv * nd) + zz * 16 + xx;
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) acc = fma(a.gtab[(hi ? GTab::E1 : GTab::E0) * n + m], s[4 * m], acc);
    if (ok) FDc[(size_t)((2 + hi) * 10 + kv) * 16 + st] = acc;
  }
}

// ------------------------------------------- predictor, n = 5 and 6
// One cell per workgroup, all time levels at once, the iterate in LDS, and
// every contraction along lines that one lane holds in registers.  The threads
// change between three roles, with a barrier between them:
//   nodes   (k, j, i): all levels of one node, for the time solve;
//   rows    (level, k, j): a line of nodes along x, for the x contractions
//           and the flux;
//   planes  (level, variable, i): the nodes of one variable at one x, for the
//           y and z contractions.
// Two slices of five variables serve the exchanges: A holds the iterate, then
// the y gradients, the y fluxes, their sum of divergences, the residual; B the
// z gradients, then the z fluxes.  Reads and writes of one node and level: 37
// and 32 doubles per sweep, where k_pred3's 150 and 20 kept the LDS busy.
// Bound by latency: LDS 40 and vector units 34 per cent busy with the six
// wavefronts that 50 kB per cell admit at n = 5 (one slice only, with more
// held in registers, spills: 384 us).  13^3 cells of N = 4: 153 us, 255 us
// with k_pred3; 9^3 of N = 5: 177, 245; one round of cells (5^3 of N = 4,
// 3^3 of N = 5): 35 and 60, 52 and 82.  At n = 3 and 2 k_pred3 is the faster
// (27^3 of N = 2 122, 135; 40^3 of N = 1 64, 112): its lines are short.
template <int n>
struct Rows3 {
  static constexpr int nn = n * n, nd = nn * n;
  static constexpr int NT = (nd + kWave - 1) / kWave * kWave;   // threads
  // strides of level, k, j, i and variable: free of bank conflicts for rows
  // and, at n = 5, nodes; planes at most 1.5 times the time without conflicts
  static constexpr int SB = n == 6 ? 36 : nd, SK = n == 6 ? 6 : nn, SJ = n == 6 ? 1 : n, SI = n == 6 ? 217 : 1;
  static constexpr int VS = n == 6 ? 1302 : 629;
  static constexpr int B = 5 * VS;                              // slice B behind slice A
  static constexpr int size = 10 * VS;
  static_assert((n - 1) * (SB + SK + SJ + SI) < VS && 20 * nd <= size && 5 * nn <= NT, "layout");
};

template <int n>
__global__ __launch_bounds__(Rows3<n>::NT, n == 6 ? 1 : 2) void k_pred3_rows(Phys ph, Tab<n> tb, Args3 a) {
  using L = Rows3<n>;
  constexpr int nn = L::nn, nd = L::nd, VS = L::VS, B = L::B;
  extern __shared__ double lds[];
  const int tid = threadIdx.x, c = blockIdx.x, layer = c / (a.nx * a.ny);
  const double h = a.h, dt = a.clock[1], ih = 1.0 / h;

  // nodes; threads past the last read another node's words and write nothing
  const bool tact = tid < nd;
  const int r = tact ? tid : 0;
  const int i = r % n, j = (r / n) % n, k = r / nn;
  double* tp = lds + k * L::SK + j * L::SJ + i * L::SI;
  // rows
  const int xb = tid / nn, xk = (tid / n) % n, xj = tid % n;
  double* xp = lds + xb * L::SB + xk * L::SK + xj * L::SJ;
  FluxC3 fc = flux_consts3(ph, h);
  fc.gz = ph.geff * ((a.z0 + layer * h) + h * a.gtab[GTab::XI * n + xk]);
  const double rb = a.bg[2 * (layer * (n + 2) + xk)];
  fc.pb = a.bg[2 * (layer * (n + 2) + xk) + 1];
  // planes: of all variables, and of the four with a flux to contract
  const int pb5 = tid / (5 * n), pb4 = tid / (4 * n);
  double* p5 = lds + pb5 * L::SB + (tid / n) % 5 * VS + tid % n * L::SI;
  double* p4 = lds + pb4 * L::SB + ((tid / n) % 4 + 1) * VS + tid % n * L::SI;

  const double* Qc = a.Q + (size_t)c * 5 * nd + r;
  double X[n][5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    X[0][v] = Qc[v * nd];
#pragma unroll
    for (int b = 1; b < n; ++b) X[b][v] = X[0][v];
  }

  // Gradients of lv levels, from the iterate in A: along x in gx, y in A, z in
  // B.  q is the row's state.
  auto gradients = [&](int lv, bool xact, double q[5][n], double gx[5][n]) {
    __syncthreads();
    if (xact) {
#pragma unroll
      for (int v = 0; v < 5; ++v)
#pragma unroll
        for (int m = 0; m < n; ++m) q[v][m] = xp[v * VS + m * L::SI];
    }
    __syncthreads();
    const EO<n> eo(scalar_table(a.gtab + GTab::eo_d(n)));
    if (pb5 < lv) {
      double in[n][n];
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int y = 0; y < n; ++y) in[z][y] = p5[z * L::SK + y * L::SJ];
#pragma unroll
      for (int z = 0; z < n; ++z) {
        double out[n];
        eo.apply(in[z], out);
#pragma unroll
        for (int y = 0; y < n; ++y) p5[z * L::SK + y * L::SJ] = out[y];
      }
#pragma unroll
      for (int y = 0; y < n; ++y) {
        double col[n], out[n];
#pragma unroll
        for (int z = 0; z < n; ++z) col[z] = in[z][y];
        eo.apply(col, out);
#pragma unroll
        for (int z = 0; z < n; ++z) p5[B + z * L::SK + y * L::SJ] = out[z];
      }
    }
    if (xact) {
#pragma unroll
      for (int v = 0; v < 5; ++v) eo.apply(q[v], gx[v]);
    }
    __syncthreads();
  };
  // state and gradients of node m of the row
  auto node_flux = [&](int m, const double q[5][n], const double gx[5][n], double g[3][5], double F[3][4]) {
    double qm[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      qm[v] = q[v][m];
      g[0][v] = gx[v][m];
      g[1][v] = xp[v * VS + m * L::SI];
      g[2][v] = xp[B + v * VS + m * L::SI];
    }
    flux_xyz(fc, qm, g, F);
  };

  for (int it = 0; it < a.iters; ++it) {
    // the first sweep starts from Q^n at every time level: all levels share
    // level 0's residual (bit for bit)
    const int lv = it ? n : 1;
    const bool xact = xb < lv;
    if (tact) {
#pragma unroll
      for (int b = 0; b < n; ++b)
        if (b < lv) {
#pragma unroll
          for (int v = 0; v < 5; ++v) tp[v * VS + b * L::SB] = X[b][v];
        }
    }
    double q[5][n], R[5][n];
    {
      double gx[5][n];
      gradients(lv, xact, q, gx);
      if (xact) {
        double Fx[4][n];
#pragma unroll
        for (int m = 0; m < n; ++m) {
          double g[3][5], F[3][4];
          node_flux(m, q, gx, g, F);
          // the mass flux is the momentum, its divergence a sum of gradients
          R[0][m] = (g[0][1] + g[1][2]) + g[2][3];
          R[3][m] = fc.gh * (q[0][m] - rb);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            Fx[v][m] = F[0][v];
            xp[(1 + v) * VS + m * L::SI] = F[1][v];
            xp[B + (1 + v) * VS + m * L::SI] = F[2][v];
          }
        }
        const EO<n> eo(scalar_table(a.gtab + GTab::eo_d(n)));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double out[n];
          eo.apply(Fx[v], out);
#pragma unroll
          for (int m = 0; m < n; ++m) R[1 + v][m] = v == 2 ? R[3][m] + out[m] : out[m];
        }
      }
    }
    __syncthreads();
    {
      const EO<n> eo(scalar_table(a.gtab + GTab::eo_d(n)));
      if (pb4 < lv) {
        double S[n][n];
#pragma unroll
        for (int y = 0; y < n; ++y) {
          double col[n], out[n];
#pragma unroll
          for (int z = 0; z < n; ++z) col[z] = p4[B + z * L::SK + y * L::SJ];
          eo.apply(col, out);
#pragma unroll
          for (int z = 0; z < n; ++z) S[z][y] = out[z];
        }
#pragma unroll
        for (int z = 0; z < n; ++z) {
          double in[n], out[n];
#pragma unroll
          for (int y = 0; y < n; ++y) in[y] = p4[z * L::SK + y * L::SJ];
          eo.apply(in, out);
#pragma unroll
          for (int y = 0; y < n; ++y) p4[z * L::SK + y * L::SJ] = S[z][y] + out[y];
        }
      }
    }
    __syncthreads();
    if (xact) {
#pragma unroll
      for (int m = 0; m < n; ++m) {
        xp[m * L::SI] = R[0][m];
#pragma unroll
        for (int v = 1; v < 5; ++v) xp[v * VS + m * L::SI] += R[v][m];
      }
    }
    __syncthreads();
    // (no condition on the thread: no iterate has to be kept across the sweep)
#pragma unroll
    for (int b = 0; b < n; ++b)
#pragma unroll
      for (int v = 0; v < 5; ++v) X[b][v] = tp[v * VS + (it ? b * L::SB : 0)];
    solve_time<n>(a.gtab + GTab::lu(n), X);
    const double sdt = -dt * ih;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double q0 = Qc[v * nd];
#pragma unroll
      for (int b = 0; b < n; ++b) X[b][v] = fma(sdt, X[b][v], q0);
    }
  }

  // time averages: x and y fluxes of the levels through A and B, then the z ones
  double Qb[5], Fb[3][4];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    Qb[v] = 0.0;
#pragma unroll
    for (int b = 0; b < n; ++b) Qb[v] = fma(tb.w[b], X[b][v], Qb[v]);
  }
  if (tact) {
#pragma unroll
    for (int b = 0; b < n; ++b)
#pragma unroll
      for (int v = 0; v < 5; ++v) tp[v * VS + b * L::SB] = X[b][v];
  }
  {
    const bool xact = xb < n;
    double q[5][n], gx[5][n], Fz[4][n];
    gradients(n, xact, q, gx);
    if (xact) {
#pragma unroll
      for (int m = 0; m < n; ++m) {
        double g[3][5], F[3][4];
        node_flux(m, q, gx, g, F);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          xp[(1 + v) * VS + m * L::SI] = F[0][v];
          xp[B + (1 + v) * VS + m * L::SI] = F[1][v];
          Fz[v][m] = F[2][v];
        }
      }
    }
    auto average = [&](int d, const double* p) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s = tb.w[0] * p[(1 + v) * VS];
#pragma unroll
        for (int b = 1; b < n; ++b) s = fma(tb.w[b], p[(1 + v) * VS + b * L::SB], s);
        Fb[d][v] = s;
      }
    };
    __syncthreads();
    average(0, tp);
    average(1, tp + B);
    __syncthreads();
    if (xact) {
#pragma unroll
      for (int m = 0; m < n; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) xp[(1 + v) * VS + m * L::SI] = Fz[v][m];
    }
    __syncthreads();
    average(2, tp);
  }
  __syncthreads();
  double* sF = lds + 5 * nd;   // averaged state [5][nd] and fluxes [3][5][nd]
  if (tact) {
#pragma unroll
    for (int v = 0; v < 5; ++v) lds[v * nd + r] = Qb[v];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      sF[d * 5 * nd + r] = Qb[1 + d];
#pragma unroll
      for (int v = 0; v < 4; ++v) sF[(d * 5 + 1 + v) * nd + r] = Fb[d][v];
    }
  }
  __syncthreads();
  if (tact) {
    // volume term (Dw[i][m] = w_m D[m][i] / w_i along each direction) and Q*
    double Wi[n], Wj[n], Wk[n];
#pragma unroll
    for (int m = 0; m < n; ++m) {
      Wi[m] = a.gtab[GTab::dw(n) + i * n + m];
      Wj[m] = a.gtab[GTab::dw(n) + j * n + m];
      Wk[m] = a.gtab[GTab::dw(n) + k * n + m];
    }
    const double Sb = -ph.geff * (Qb[0] - a.bg[2 * (layer * (n + 2) + k)]);
    double* Qsc = a.Qs + (size_t)c * 5 * nd + r;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double vol = div3<n>(sF, v, i, j, k, Wi, Wj, Wk);
      Qsc[v * nd] = fma(dt, fma(vol, ih, v == 3 ? Sb : 0.0), Qc[v * nd]);
    }
    face_data3<n>(tb, lds, sF, a.FD + (size_t)c * 60 * nn, r);
  }
}

// ---------------------------------------------------------------- corrector
// Per face node: the neighbour's face data (or the wall ghost), the largest
// wave and viscous speeds over both sides of the face, then the Rusanov flux
//   G = (F_L + F_R)/2 - (lambda + 2 eta lambda_v)/2 (Q_R - Q_L)
// with L the -axis side; per node: Q = Q* - dt/h (lifting of the six face
// fluxes), and the cell's CFL candidate from the new state.
// Memory and the LDS stages between barriers bound it.  A node keeps the jump
// and the sum of the fluxes, not the two sides, and the momentum along the
// face's axis is picked from values: picked from an array by its index, the
// sides lay in scratch (N >= 3).  25^3 cells of N = 3 53.4 and 46.5 us, 13^3 of
// N = 4 22.7 and 19.1, 9^3 of N = 5 18.7 and 17.7; N = 1 and 2 as before.
template <int n>
__global__ __launch_bounds__(kThreads3) void k_corr3(Phys ph, Args3 a) {
  using G = Cfg3<n>;
  constexpr int nn = G::nn, nd = G::nd, NJ = 6 * nn, IT = (NJ + nd - 1) / nd;
  constexpr bool WL = G::WL;
  extern __shared__ double lds[];
  const int tid = threadIdx.x, r = tid % nd;
  const bool mirror = G::spare && tid >= G::CB * nd;
  const int slot = mirror ? 0 : tid / nd;
  const int cell = blockIdx.x * G::CB + slot;
  const bool valid = !mirror && cell < a.C;
  const int c = cell < a.C ? cell : a.C - 1;
  double* sG = lds + slot * G::corr_slot;
  double* sl = sG + 30 * nn;
  double* sv = sl + 6 * nn;
  unsigned long long* smax = reinterpret_cast<unsigned long long*>(sv + 6 * nn);
  const int ci = c % a.nx, cj = (c / a.nx) % a.ny, ck = c / (a.nx * a.ny);
  const double h = a.h, dt = a.clock[1];
  const double zc = a.z0 + ck * h;
  if (r == 0) { smax[0] = 0ull; smax[1] = 0ull; }

  double jump[IT][5], fsum[IT][5];   // Q_R - Q_L, F_L + F_R
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int q = r + it * nd;
    const bool act = q < NJ;
    const int qq = act ? q : 0;
    const int f = qq / nn, st = qq - f * nn, s = st / n;
    const int d = f >> 1, hi = f & 1;
    const double* own = a.FD + ((size_t)c * 6 + f) * 10 * nn + st;
    double Qo[5], Fo[5], Qn[5], Fn[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) { Qo[v] = own[v * nn]; Fo[v] = own[(5 + v) * nn]; }
    const int dim = d == 0 ? a.nx : (d == 1 ? a.ny : a.nz);
    const int pos = d == 0 ? ci : (d == 1 ? cj : ck);
    int np = pos + (hi ? 1 : -1);
    const bool outside = np < 0 || np >= dim;
    const bool wall = outside && ((a.wall >> f) & 1);
    if (outside && !wall) np = np < 0 ? np + dim : np - dim;
    const double zf = f == 4 ? zc : (f == 5 ? zc + h : zc + h * a.gtab[GTab::XI * n + s]);
    if (wall) {
      wall_ghost3(ph, d, zf, a.bg + 2 * (ck * (n + 2) + (d == 2 ? n + hi : s)), Qo, Fo, Qn, Fn);
    } else {
      const int o = d == 0 ? (ck * a.ny + cj) * a.nx + np
                           : (d == 1 ? (ck * a.ny + np) * a.nx + ci : (np * a.ny + cj) * a.nx + ci);
      const double* oth = a.FD + ((size_t)o * 6 + (f ^ 1)) * 10 * nn + st;
#pragma unroll
      for (int v = 0; v < 5; ++v) { Qn[v] = oth[v * nn]; Fn[v] = oth[(5 + v) * nn]; }
    }
    double l1, v1, l2, v2;
    eig3(ph, d, Qo, zf, l1, v1);
    eig3(ph, d, Qn, zf, l2, v2);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      jump[it][v] = hi ? Qn[v] - Qo[v] : Qo[v] - Qn[v];
      fsum[it][v] = Fo[v] + Fn[v];
    }
    if (act) { sl[q] = fmax(l1, l2); sv[q] = fmax(v1, v2); }
  }
  sync3<WL>();
  // The faces' maxima in two steps, rows of a face first: 4 n reads a node
  // instead of 2 n^2 (13^3 cells of N = 4 20.9 and 19.1 us, 9^3 of N = 5 18.7
  // and 17.7, 9^3 of N = 3 10.0 and 8.8).  A face of four nodes is read at once.
  constexpr bool by_rows = n > 2;
  constexpr int step = by_rows ? n : 1;
  if constexpr (by_rows) {
    for (int q = r; q < 12 * n; q += nd) {
      double* p = sl + q * n;   // rows of sl, then of sv
      double m = p[0];
#pragma unroll
      for (int t = 1; t < n; ++t) m = fmax(m, p[t]);
      p[0] = m;
    }
    sync3<WL>();
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int q = r + it * nd;
    if (q < NJ) {
      const int f = q / nn, st = q - f * nn;
      double lm = sl[f * nn], vm = sv[f * nn];
      for (int m = step; m < nn; m += step) { lm = fmax(lm, sl[f * nn + m]); vm = fmax(vm, sv[f * nn + m]); }
      const double sp = lm + 2.0 * a.eta * vm;
#pragma unroll
      for (int v = 0; v < 5; ++v)
        sG[(f * 5 + v) * nn + st] = 0.5 * fsum[it][v] - 0.5 * sp * jump[it][v];
    }
  }
  sync3<WL>();

  const int i = r % n, j = (r / n) % n, k = r / nn;
  const double L0i = a.gtab[GTab::L0 * n + i], L1i = a.gtab[GTab::L1 * n + i];
  const double L0j = a.gtab[GTab::L0 * n + j], L1j = a.gtab[GTab::L1 * n + j];
  const double L0k = a.gtab[GTab::L0 * n + k], L1k = a.gtab[GTab::L1 * n + k];
  const double* Qsc = a.Qs + (size_t)c * 5 * nd;
  const double sc = dt / h;
  double qn[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double* Gv = sG + v * nn;
    const double lx = L1i * Gv[5 * nn + k * n + j] - L0i * Gv[k * n + j];
    const double ly = L1j * Gv[15 * nn + k * n + i] - L0j * Gv[10 * nn + k * n + i];
    const double lz = L1k * Gv[25 * nn + j * n + i] - L0k * Gv[20 * nn + j * n + i];
    qn[v] = Qsc[v * nd + r] - sc * (lx + ly + lz);
  }
  if (valid) {
    double* Qo = a.Qout + (size_t)c * 5 * nd;
#pragma unroll
    for (int v = 0; v < 5; ++v) Qo[v * nd + r] = qn[v];
    // CFL candidate: max over the nodes of max(|u|,|v|,|w|) + c and of
    // lambda_v (non-negative doubles order like their bit patterns)
    const double z = zc + h * a.gtab[GTab::XI * n + k];
    const double ir = recip(qn[0]);
    const double lam = fmax(fabs(qn[1]), fmax(fabs(qn[2]), fabs(qn[3]))) * ir + sound3(ph, qn, ir, z);
    const double lv = ph.lv_coef * ir;
    atomicMax(&smax[0], (unsigned long long)__double_as_longlong(lam));
    atomicMax(&smax[1], (unsigned long long)__double_as_longlong(lv));
  }
  sync3<WL>();
  if (valid && r == 0) {
    const double lam = __longlong_as_double((long long)smax[0]), lv = __longlong_as_double((long long)smax[1]);
    const double o = 2.0 * ph.N + 1.0;
    a.dtc[c] = ph.cfl * h / (3.0 * o * (lam + 2.0 * lv * o / h));
  }
}

// CFL candidate of every cell from the current state
template <int n>
__global__ __launch_bounds__(kThreads3) void k_dt3(Phys ph, Args3 a) {
  using G = Cfg3<n>;
  constexpr int nn = G::nn, nd = G::nd;
  __shared__ unsigned long long smax[G::CB][2];
  const int tid = threadIdx.x, slot = tid / nd, r = tid - slot * nd;
  const bool inslot = !G::spare || slot < G::CB;
  const int cell = blockIdx.x * G::CB + slot;
  const bool valid = inslot && cell < a.C;
  if (inslot && r == 0) { smax[slot][0] = 0ull; smax[slot][1] = 0ull; }
  sync3<G::WL>();
  if (valid) {
    const int ck = cell / (a.nx * a.ny), k = r / nn;
    const double* Qc = a.Q + (size_t)cell * 5 * nd;
    double q[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) q[v] = Qc[v * nd + r];
    const double z = (a.z0 + ck * a.h) + a.h * a.gtab[GTab::XI * n + k];
    const double ir = recip(q[0]);
    const double lam = fmax(fabs(q[1]), fmax(fabs(q[2]), fabs(q[3]))) * ir + sound3(ph, q, ir, z);
    atomicMax(&smax[slot][0], (unsigned long long)__double_as_longlong(lam));
    atomicMax(&smax[slot][1], (unsigned long long)__double_as_longlong(ph.lv_coef * ir));
  }
  sync3<G::WL>();
  if (valid && r == 0) {
    const double lam = __longlong_as_double((long long)smax[slot][0]);
    const double lv = __longlong_as_double((long long)smax[slot][1]);
    const double o = 2.0 * ph.N + 1.0;
    a.dtc[cell] = ph.cfl * a.h / (3.0 * o * (lam + 2.0 * lv * o / a.h));
  }
}

// ----------------------------------------------------------- initial states
// kind 0: hydrostatic background of constant potential temperature perturbed
// in theta at fixed pressure by the bubbles (eqs. cos-pertubation,
// bubbles-pertubation, with the distance in three dimensions), at rest;
// kind 1: the ABC flow (eq. abc-flow) at time t0
__global__ void k_init3(Phys ph, Args3 a, int n, int kind, Bubbles3 B, double t0, double* Q) {
  const int nd = n * n * n;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)a.C * nd) return;
  const int c = (int)(gid / nd), r = (int)(gid % nd);
  const int i = r % n, j = (r / n) % n, k = r / (n * n);
  const int ci = c % a.nx, cj = (c / a.nx) % a.ny, ck = c / (a.nx * a.ny);
  const double* xi = a.gtab + GTab::XI * n;
  const double x = a.x0 + a.h * (ci + xi[i]), y = a.y0 + a.h * (cj + xi[j]), z = a.z0 + a.h * (ck + xi[k]);
  double q[5];
  if (kind == 0) {
    double th = 0.0;
    for (int b = 0; b < B.nb; ++b) {
      const double* bb = B.b + 7 * b;
      const double dx = x - bb[4], dy = y - bb[5], dz = z - bb[6];
      const double rr = sqrt(dx * dx + dy * dy + dz * dz);
      if (bb[0] == 0.0) th += rr <= bb[2] ? 0.5 * bb[1] * (1.0 + cos(M_PI * rr / bb[2])) : 0.0;
      else th += rr <= bb[2] ? bb[1] : bb[1] * exp(-(rr - bb[2]) * (rr - bb[2]) / (bb[3] * bb[3]));
    }
    const double pi = 1.0 - ph.g * z / (ph.cp * ph.theta);
    const double pbg = ph.p0 * pow(pi, ph.cp_over_R);
    const double rho = pbg / (ph.R * (ph.theta + th) * pi);
    q[0] = rho; q[1] = 0.0; q[2] = 0.0; q[3] = 0.0;
    q[4] = pbg / ph.gm1 + rho * ph.g * z;
  } else {
    const double e1 = exp(-ph.mu * t0), e2 = exp(-2.0 * ph.mu * t0);
    const double u = e1 * (sin(z) + cos(y)), v = e1 * (sin(x) + cos(z)), w = e1 * (sin(y) + cos(x));
    const double p = 100.0 / ph.gamma - e2 * (cos(x) * sin(y) + sin(x) * cos(z) + sin(z) * cos(y));
    q[0] = 1.0; q[1] = u; q[2] = v; q[3] = w;
    q[4] = p / ph.gm1 + 0.5 * (u * u + v * v + w * w);
  }
  double* Qc = Q + (size_t)c * 5 * nd;
  for (int v = 0; v < 5; ++v) Qc[v * nd + r] = q[v];
}

// flag non-finite values and non-positive density or pressure
__global__ void k_health3(Phys ph, Args3 a, int n, int* flag) {
  const int nd = n * n * n;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)a.C * nd) return;
  const int c = (int)(gid / nd), r = (int)(gid % nd);
  const int ck = c / (a.nx * a.ny);
  const double* Qc = a.Q + (size_t)c * 5 * nd;
  double q[5];
  bool bad = false;
  for (int v = 0; v < 5; ++v) { q[v] = Qc[v * nd + r]; bad = bad || !isfinite(q[v]); }
  bad = bad || !(q[0] > 0.0);
  if (!bad) bad = !(pressure3(ph, q, (a.z0 + ck * a.h) + a.h * a.gtab[GTab::XI * n + r / (n * n)]) > 0.0);
  if (bad) atomicOr(flag, 1);
}

// --------------------------------------------------------------- launchers
template <int n>
static int pred3_n(const Phys& ph, const HostBasis& B, const Args3& a, hipStream_t s) {
  using G = Cfg3<n>;
  const int blocks = (a.C + G::CB - 1) / G::CB;
  const size_t lds = sizeof(double) * (size_t)G::CB * G::pred_slot;
  if constexpr (n == 4)
    hipLaunchKernelGGL(k_pred3_w64, dim3((a.C + kW64Cells - 1) / kW64Cells), dim3(kWave * kW64Cells),
                       sizeof(double) * kW64Cells * 20 * 64, s, ph, tab_of<n>(B), a);
  else if constexpr (n > 4)
    hipLaunchKernelGGL(k_pred3_rows<n>, dim3(a.C), dim3(Rows3<n>::NT), sizeof(double) * Rows3<n>::size, s, ph,
                       tab_of<n>(B), a);
  else
    hipLaunchKernelGGL(k_pred3<n>, dim3(blocks), dim3(kThreads3), lds, s, ph, tab_of<n>(B), a);
  return check_launch("predictor3");
}
template <int n>
static int corr3_n(const Phys& ph, const Args3& a, hipStream_t s) {
  using G = Cfg3<n>;
  const int blocks = (a.C + G::CB - 1) / G::CB;
  const size_t lds = sizeof(double) * (size_t)G::CB * G::corr_slot;
  hipLaunchKernelGGL(k_corr3<n>, dim3(blocks), dim3(kThreads3), lds, s, ph, a);
  return check_launch("corrector3");
}
template <int n>
static int dt3_n(const Phys& ph, const Args3& a, hipStream_t s) {
  using G = Cfg3<n>;
  const int blocks = (a.C + G::CB - 1) / G::CB;
  hipLaunchKernelGGL(k_dt3<n>, dim3(blocks), dim3(kThreads3), 0, s, ph, a);
  return check_launch("cell_dt3");
}

#define ADG3_DISPATCH(fn, n, ...)                                        \
  switch (n) {                                                           \
    case 2: return fn<2>(__VA_ARGS__);                                   \
    case 3: return fn<3>(__VA_ARGS__);                                   \
    case 4: return fn<4>(__VA_ARGS__);                                   \
    case 5: return fn<5>(__VA_ARGS__);                                   \
    case 6: return fn<6>(__VA_ARGS__);                                   \
    default: return fail(ADG_EUNSUPPORTED, "order not supported in 3D"); \
  }

int launch_pred3(const Phys& ph, const HostBasis& B, const Args3& a, hipStream_t s) {
  if (a.C == 0) return ADG_OK;
  ADG3_DISPATCH(pred3_n, B.n, ph, B, a, s);
}
int launch_corr3(const Phys& ph, int n, const Args3& a, hipStream_t s) {
  if (a.C == 0) return ADG_OK;
  ADG3_DISPATCH(corr3_n, n, ph, a, s);
}
int launch_dt3(const Phys& ph, int n, const Args3& a, hipStream_t s) {
  if (a.C == 0) return ADG_OK;
  ADG3_DISPATCH(dt3_n, n, ph, a, s);
}
int launch_background3(const Phys& ph, int n, const Args3& a, double* bg, hipStream_t s) {
  const long long tot = (long long)a.nz * (n + 2);
  hipLaunchKernelGGL(k_background3, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, ph, a, n, bg);
  return check_launch("background3");
}
int launch_init3(const Phys& ph, int n, const Args3& a, int kind, const Bubbles3& B, double t0, double* Q,
                 hipStream_t s) {
  const long long tot = (long long)a.C * n * n * n;
  if (tot == 0) return ADG_OK;
  hipLaunchKernelGGL(k_init3, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, ph, a, n, kind, B, t0, Q);
  return check_launch("init_state3");
}
int launch_health3(const Phys& ph, int n, const Args3& a, int* flag, hipStream_t s) {
  const long long tot = (long long)a.C * n * n * n;
  if (tot == 0) return ADG_OK;
  hipLaunchKernelGGL(k_health3, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, ph, a, n, flag);
  return check_launch("health3");
}

}  // namespace adg
