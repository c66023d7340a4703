// Hand-written adjoint (reverse mode) of one ADER-DG step, of the initial
// state map from the potential-temperature perturbation, and of the
// potential-temperature loss, for gfx950.
//
// The step is Q^{n+1} = Q*(Q^n) - (dt/h) lift(G(FD(Q^n))) with a frozen dt.
// Its adjoint maps lambda^{n+1} = dL/dQ^{n+1} to lambda^n = dL/dQ^n:
//   1. the forward predictor is recomputed from the checkpoint Q^n, storing
//      the Picard iterates (iterate store);
//   2. lifting adjoint: per cell and face, the face-flux adjoint of both
//      cells' halves of the surface integral;
//   3. face adjoint: per face, the reverse of the Rusanov flux (and of a wall
//      ghost) onto this cell's face data;
//      non-smooth points take the subgradient of the first maximum in the
//      scan order (side L nodes 0..n-1, then side R), and d|x|/dx = 0 at 0;
//   4. reverse predictor: face extrapolations, volume term and time
//      averages, then the Picard sweeps in reverse order (R = S - div F:
//      transposed derivative contractions and the reverse of the pointwise
//      flux), accumulating dL/dQ^n.
#include "step_internal.h"

namespace adg {

// --------------------------------------------------------- pointwise VJP
// Reverse of the predictor's fluxes at one node.  q: state; gx, gz: gradients
// in reference coordinates; aFx, aFz: adjoints of the fluxes.  Returns the
// adjoints of the state and of the gradients.  Notation and constants are
// those of the forward flux: a = rho du/dx and so on, so that the stresses
// and the conductivity are proportional to 1/rho and their share of the
// density's adjoint is one sum.
__device__ inline void flux_vjp(const FluxC& c, const double q[4], const double gx[4], const double gz[4],
                                const double aFx[4], const double aFz[4], double aq[4], double agx[4], double agz[4]) {
  // forward
  const double rho = q[0], mx = q[1], mz = q[2], E = q[3];
  const double ir = recip(rho);
  const double u = mx * ir, w = mz * ir;
  const double ke = fma(mx, u, mz * w);
  const double p = fma(-c.hgm1, ke, c.gm1 * fma(-c.gz, rho, E));
  const double pir = p * ir;
  const double ax = fma(-u, gx[0], gx[1]), az = fma(-u, gz[0], gz[1]);
  const double cx = fma(-w, gx[0], gx[2]), cz = fma(-w, gz[0], gz[2]);
  const double kin = 0.5 * ir * ke, hv = kin + c.gz;
  const double dx = fma(-w, cx, fma(-u, ax, fma(-hv, gx[0], gx[3])));
  const double dz = fma(-c.gh, rho, fma(-w, cz, fma(-u, az, fma(-hv, gz[0], gz[3]))));
  const double m23 = c.mu23 * ir, mi = c.mu * ir, k = c.kap * ir;
  const double sxx = m23 * fma(-2.0, ax, cz), szz = m23 * fma(-2.0, cz, ax), sxz = -mi * (az + cx);
  const double qx = fma(-pir, gx[0], c.gm1 * dx), qz = fma(-pir, gz[0], c.gm1 * dz);
  const double H = E + p;
  // reverse: Fx1 = mx u + p + sxx, Fx2 = Fz1 = mx w + sxz, Fz2 = mz w + p + szz,
  // Fx3 = u (H + sxx) + w sxz - k qx, Fz3 = w (H + szz) + u sxz - k qz
  const double A1 = aFx[1], A2 = aFx[2] + aFz[1], A3 = aFx[3], B2 = aFz[2], B3 = aFz[3];
  const double bxx = fma(A3, u, A1), bzz = fma(B3, w, B2), bxz = fma(B3, u, fma(A3, w, A2));
  double bu = fma(A3, H + sxx, fma(B3, sxz, A1 * mx));
  double bw = fma(B3, H + szz, fma(A3, sxz, fma(A2, mx, B2 * mz)));
  const double bH = fma(A3, u, B3 * w);
  const double bk = -fma(A3, qx, B3 * qz);
  const double bqx = -k * A3, bqz = -k * B3;
  const double bdx = c.gm1 * bqx, bdz = c.gm1 * bqz;
  const double bpir = -fma(bqx, gx[0], bqz * gz[0]);
  const double bhv = -fma(bdx, gx[0], bdz * gz[0]);
  const double t = -mi * bxz;
  const double bax = fma(m23, fma(-2.0, bxx, bzz), -u * bdx), bcz = fma(m23, fma(-2.0, bzz, bxx), -w * bdz);
  const double bcx = fma(-w, bdx, t), baz = fma(-u, bdz, t);
  bu -= fma(bdx, ax, bdz * az);
  bw -= fma(bdx, cx, bdz * cz);
  bu = fma(bhv, u, fma(-gx[0], bax, fma(-gz[0], baz, bu)));
  bw = fma(bhv, w, fma(-gx[0], bcx, fma(-gz[0], bcz, bw)));
  const double T = c.gm1 * (fma(ir, bpir, bH) + (A1 + B2));
  double br = fma(sxx, bxx, fma(szz, bzz, fma(sxz, bxz, fma(k, bk, fma(pir, bpir, fma(u, bu, w * bw))))));
  br = fma(-ir, br, fma(T, kin - c.gz, -c.gh * bdz));
  agx[0] = -fma(pir, bqx, fma(hv, bdx, fma(u, bax, w * bcx)));
  agz[0] = -fma(pir, bqz, fma(hv, bdz, fma(u, baz, w * bcz)));
  agx[1] = bax; agx[2] = bcx; agx[3] = bdx;
  agz[1] = baz; agz[2] = bcz; agz[3] = bdz;
  aq[0] = br;
  aq[1] = fma(-T, u, fma(ir, bu, fma(A1, u, fma(A2, w, aFx[0]))));
  aq[2] = fma(-T, w, fma(ir, bw, fma(B2, w, aFz[0])));
  aq[3] = T + bH;
}

struct AdjArgs {
  const double* Qn;      // checkpoint [C][4][n][n]
  const double* lam_in;  // dL/dQ^{n+1}
  double* lam_out;       // dL/dQ^n
  const double* FD;      // forward face data (recomputed)
  const double* store;   // iterates [C][I][n][4][n][n]
  const double* clock;
  const double* geom;
  const double* bg;      // [C][n + 2][2]
  const int* nbr;
  const double* gtab;
  int C, iters;
};

// ---------------------------------------------------------- lifting adjoint
// The corrector's surface term of cell c, -(dt/h) (L1 G_{+} - L0 G_{-}) per
// row or column, transposed: cell c's half of the adjoint of face f's flux
// at face node k, variable v (L0 = e0/w, L1 = e1/w).
template <int n>
__device__ inline double lift_adj_half(const AdjArgs& a, int c, int f, int k, int v) {
  constexpr int nn = n * n;
  const double sc = a.clock[1] / a.geom[4 * c + 2];
  const double* lam = a.lam_in + (size_t)c * 4 * nn + v * nn;
  const double* Lt = a.gtab + (((f & 1) ? GTab::L1 : GTab::L0) * n);
  const double sgn = (f & 1) ? -sc : sc;   // +face: -(dt/h) L1, -face: +(dt/h) L0
  double s = 0.0;
#pragma unroll
  for (int m = 0; m < n; ++m) {
    const int idx = (f < 2) ? (k * n + m) : (m * n + k);   // x-faces: row k; z-faces: column k
    s = fma(Lt[m], lam[idx], s);
  }
  return sgn * s;
}

// ------------------------------------------------------------ face adjoint
__device__ inline void eig_a(const Phys& ph, int d, const double q[4], double zf, double& lam, double& lv) {
  const double ir = 1.0 / q[0];
  const double p = pressure(ph, q[0], q[1], q[2], q[3], zf);
  lam = fabs((d == 0 ? q[1] : q[2]) * ir) + sqrt(ph.gamma * p * ir);
  lv = ph.lv_coef * ir;
}

// gradient of lambda = |v_d| + c and of lambda_v with respect to the state
__device__ inline void eig_grad(const Phys& ph, int d, const double q[4], double zf, double gl[4], double gv[4]) {
  const double rho = q[0], ir = 1.0 / rho;
  const double u = q[1] * ir, w = q[2] * ir;
  const double p = pressure(ph, q[0], q[1], q[2], q[3], zf);
  const double c = sqrt(ph.gamma * p * ir);
  const double vn = (d == 0 ? q[1] : q[2]) * ir;
  const double sg = vn > 0.0 ? 1.0 : (vn < 0.0 ? -1.0 : 0.0);
  const double geo = ph.gravity ? ph.g * zf : 0.0;
  // dp/dQ
  const double dp[4] = {ph.gm1 * (0.5 * (u * u + w * w) - geo), -ph.gm1 * u, -ph.gm1 * w, ph.gm1};
  // dc = gamma/(2c) (dp/rho - p drho/rho^2)
  const double k = ph.gamma / (2.0 * c);
  for (int v = 0; v < 4; ++v) gl[v] = k * dp[v] * ir;
  gl[0] += -k * p * ir * ir;
  gl[0] += sg * (-vn * ir);
  if (d == 0) gl[1] += sg * ir;
  else gl[2] += sg * ir;
  gv[0] = -ph.lv_coef * ir * ir; gv[1] = 0.0; gv[2] = 0.0; gv[3] = 0.0;
}

// wall ghost (as in the forward corrector) and its reverse; bg: the background
// at the face node
__device__ inline void ghost_fwd(const Phys& ph, int d, double zf, const double bg[2], const double Qi[4],
                                 const double Fi[4], double Qg[4], double Fg[4]) {
  const double u = Qi[1] / Qi[0], w = Qi[2] / Qi[0];
  double rb, pb;
  if (ph.gravity) { rb = bg[0]; pb = bg[1]; }
  else { rb = Qi[0]; pb = pressure(ph, Qi[0], Qi[1], Qi[2], Qi[3], zf); }
  const double geo = ph.gravity ? rb * (ph.g * zf) : 0.0;
  Qg[0] = rb; Qg[1] = -(rb * u); Qg[2] = -(rb * w);
  Qg[3] = pb / ph.gm1 + 0.5 * rb * (u * u + w * w) + geo;
  const double qbg = (ph.gravity && d == 1) ? ph.kappa * ph.g / ph.cp : 0.0;
  Fg[0] = -Fi[0]; Fg[1] = Fi[1]; Fg[2] = Fi[2]; Fg[3] = 2.0 * qbg - Fi[3];
}

// adjoints of the ghost (aQg, aFg) -> adjoints of the interior data
__device__ inline void ghost_vjp(const Phys& ph, double zf, const double bg[2], const double Qi[4], const double aQg[4],
                                 const double aFg[4], double aQi[4], double aFi[4]) {
  aFi[0] = -aFg[0]; aFi[1] = aFg[1]; aFi[2] = aFg[2]; aFi[3] = -aFg[3];
  const double rho = Qi[0], ir = 1.0 / rho;
  const double u = Qi[1] * ir, w = Qi[2] * ir;
  double rb, pb, brb = 0.0, bpb = 0.0, bu = 0.0, bw = 0.0;
  if (ph.gravity) { rb = bg[0]; pb = bg[1]; }
  else { rb = rho; pb = pressure(ph, Qi[0], Qi[1], Qi[2], Qi[3], zf); }
  // Qg0 = rb ; Qg1 = -rb u ; Qg2 = -rb w ; Qg3 = pb/gm1 + 1/2 rb (u^2+w^2) + rb g z
  brb += aQg[0] - aQg[1] * u - aQg[2] * w + aQg[3] * (0.5 * (u * u + w * w) + (ph.gravity ? ph.g * zf : 0.0));
  bu += -aQg[1] * rb + aQg[3] * rb * u;
  bw += -aQg[2] * rb + aQg[3] * rb * w;
  bpb += aQg[3] / ph.gm1;
  aQi[0] = 0.0; aQi[1] = 0.0; aQi[2] = 0.0; aQi[3] = 0.0;
  if (!ph.gravity) {
    aQi[0] += brb;
    // pb = gm1 (E - 1/2 (mx^2 + mz^2)/rho)
    aQi[3] += bpb * ph.gm1;
    aQi[1] += -bpb * ph.gm1 * u;
    aQi[2] += -bpb * ph.gm1 * w;
    aQi[0] += bpb * ph.gm1 * 0.5 * (u * u + w * w);
  }
  // u = mx/rho, w = mz/rho
  aQi[1] += bu * ir; aQi[2] += bw * ir;
  aQi[0] += -(bu * u + bw * w) * ir;
}

// Reverse of the Rusanov flux on one face of a cell, a lane per face node k:
// total flux adjoint of face f (this cell's half plus the neighbour's, both
// from the lifting adjoint of the incoming adjoint state), then the adjoints of
// this cell's own face data (at walls also through the ghost).  `load` fetches
// the node's data and publishes its speeds and its share of dL/ds, which
// `reverse` needs from every node of the face.
template <int n>
struct FaceAdj {
  double Qm[4], Fm[4], Qo[4], Fo[4], aG[4], bg[2], zf, h;
  int d, wall;
  bool lower;     // this cell is side R

  // sx [5][n] of the face: speeds [2][n], viscous speeds [2][n], shares [n]
  __device__ inline void load(const Phys& ph, const AdjArgs& a, int c, int f, int k, double* sx) {
    const double* gt = a.gtab;
    const int* nb = a.nbr + (size_t)c * 16 + f * 4;
    const double z0 = a.geom[4 * c + 1];
    h = a.geom[4 * c + 2];
    d = f >> 1;
    lower = (f & 1) == 0;
    wall = nb[0] != kConforming;
    zf = (d == 0) ? z0 + h * gt[GTab::XI * n + k] : z0 + ((f & 1) ? h : 0.0);
    const double* fd = a.FD + (size_t)c * 32 * n + f * 8 * n;
    for (int v = 0; v < 4; ++v) {
      Qm[v] = fd[v * n + k]; Fm[v] = fd[4 * n + v * n + k];
      aG[v] = lift_adj_half<n>(a, c, f, k, v);
    }
    if (!wall) {
      const int o = nb[1];
      const double* fo = a.FD + (size_t)o * 32 * n + (f ^ 1) * 8 * n;
      for (int v = 0; v < 4; ++v) {
        Qo[v] = fo[v * n + k]; Fo[v] = fo[4 * n + v * n + k];
        aG[v] += lift_adj_half<n>(a, o, f ^ 1, k, v);
      }
    } else {
      const double* b = a.bg + 2 * ((size_t)c * (n + 2) + (d == 0 ? k : n + (f & 1)));
      bg[0] = b[0]; bg[1] = b[1];
      ghost_fwd(ph, d, zf, bg, Qm, Fm, Qo, Fo);
    }
    double l, lv, ds = 0.0;
    eig_a(ph, d, lower ? Qo : Qm, zf, l, lv); sx[k] = l; sx[2 * n + k] = lv;
    eig_a(ph, d, lower ? Qm : Qo, zf, l, lv); sx[n + k] = l; sx[3 * n + k] = lv;
    // this node's share of dL/ds = sum_v aG . (-1/2 (QR - QL))
    for (int v = 0; v < 4; ++v) ds += aG[v] * (lower ? -0.5 * (Qm[v] - Qo[v]) : -0.5 * (Qo[v] - Qm[v]));
    sx[4 * n + k] = ds;
  }

  // out [2][4][n]: adjoints of the face's state and flux
  __device__ inline void reverse(const Phys& ph, int k, const double* sx, double* out) const {
    // speed and its argmax: first maximum in the order L nodes 0..n-1, R nodes 0..n-1
    double lam = sx[0], lvm = sx[2 * n], bs = 0.0;
    int al = 0, av = 0;
    for (int m = 1; m < 2 * n; ++m) {
      if (sx[m] > lam) { lam = sx[m]; al = m; }
      if (sx[2 * n + m] > lvm) { lvm = sx[2 * n + m]; av = m; }
    }
    for (int m = 0; m < n; ++m) bs += sx[4 * n + m];
    const double eta = (2.0 * ph.N + 1.0) / (h * 1.2533141373155002512);
    const double s = lam + 2.0 * eta * lvm;
    // G = 1/2 (FL + FR) - 1/2 s (QR - QL): adjoints of both sides' data at node
    // k, m this cell's and g the other's
    double aQm[4], aQg[4], aF[4];
    for (int v = 0; v < 4; ++v) {
      aF[v] = 0.5 * aG[v];
      aQg[v] = (lower ? 0.5 : -0.5) * s * aG[v];
      aQm[v] = -aQg[v];
    }
    // speed terms at the argmax nodes (if they are this node)
    const int km = lower ? n + k : k, kg = lower ? k : n + k;
    double gl[4], gv[4];
    if (al == km || av == km) {
      eig_grad(ph, d, Qm, zf, gl, gv);
      for (int v = 0; v < 4; ++v) {
        if (al == km) aQm[v] += bs * gl[v];
        if (av == km) aQm[v] += bs * 2.0 * eta * gv[v];
      }
    }
    if (wall) {
      if (al == kg || av == kg) {
        eig_grad(ph, d, Qo, zf, gl, gv);
        for (int v = 0; v < 4; ++v) {
          if (al == kg) aQg[v] += bs * gl[v];
          if (av == kg) aQg[v] += bs * 2.0 * eta * gv[v];
        }
      }
      double aQi[4], aFi[4];
      ghost_vjp(ph, zf, bg, Qm, aQg, aF, aQi, aFi);
      for (int v = 0; v < 4; ++v) { aQm[v] += aQi[v]; aF[v] += aFi[v]; }
    }
    for (int v = 0; v < 4; ++v) { out[v * n + k] = aQm[v]; out[4 * n + v * n + k] = aF[v]; }
  }
};

// ------------------------------------------------------- reverse predictor
// One workgroup of four wavefronts per CB cells.  All time levels of a sweep
// run side by side, and the threads change between three roles, with a barrier
// between them:
//   time columns (variable, cell, j, i): all levels of one value, for the
//           transposed time matrix; the iterate's adjoint lives here;
//   lines   (variable, cell, level, j or i): a row or a column in registers,
//           for the derivatives and their transposes;
//   nodes   (cell, level, j, i): the reverse of the fluxes.
// Wavefront w works on variable w in the first two roles.  Adjoints are
// divided by the quadrature weights w_i w_j of their node: along a line
// D^T = W Dw W^{-1} and Dw^T = W D W^{-1}, so the transposed contractions are
// those of the forward sweep and have its even-odd form.  The face adjoints of
// the cell come first, in the same kernel (in one of their own they cost a
// launch and a trip through memory, 4 us).  Buffers, each
// [4 variables][level][j][i]: A and B along x and z (adjoints of the fluxes,
// gradients, adjoints of the gradients), C (residual adjoints, then the direct
// adjoints of the state), Q (the iterate).
//
// Bound by the chain of a cell: six barriers and some 550 FP64 and 150 LDS
// instructions of a wavefront per sweep at n = 7, 3.5 us.  Step adjoint
// without the predictor, before (time levels one per wavefront, lines as dot
// products, face adjoints apart) and now: 27 x 27 cells of n = 7 74 and 60 us,
// 41 x 23 of n = 5 54 and 26, 45 x 45 of n = 6 128 and 95, of n = 3 37 and 18,
// 9 x 9 of n = 7 40 and 33.  Loading the next iterate a sweep ahead: no gain,
// and at n = 7 spills.
template <int n, int CB>
struct AdjLay {
  static constexpr int nn = n * n;
  static constexpr bool grid8 = CB == 1 && (n == 6 || n == 7);   // lane 8 hi + lo, else hi n + lo
  static_assert(grid8 || CB * nn <= kWave, "a lane per line of each cell");
  // strides of level, row and node within a variable: free of bank conflicts
  // for rows, columns and time columns
  static constexpr int BS = grid8 ? 8 : n, JS = 1;
  static constexpr int IS = grid8 ? 55 : n == 8 ? 65 : n == 7 ? 49 : n == 6 ? 41 : n == 5 ? 25 : n == 4 ? 19 : n == 3 ? 10 : 4;
  static constexpr int VS = (n - 1) * (BS + JS + IS) + 1;
  static constexpr int buf = 4 * VS, cell = 4 * buf;
  static constexpr int NT = 4 * kWave;
  static constexpr int NP = (CB * n * nn + NT - 1) / NT;           // nodes per thread
  static_assert(NP == 1 || CB == 1, "a thread's nodes lie in one cell");
  static_assert(CB * 8 * n <= NT, "one slice line per thread");
};

template <int n, int CB>
__global__ __launch_bounds__(4 * kWave, 3) void k_pred_adj(Phys ph, AdjArgs a) {
  using L = AdjLay<n, CB>;
  constexpr int nn = L::nn, sl = 4 * nn, BS = L::BS, JS = L::JS, IS = L::IS, VS = L::VS, buf = L::buf, NP = L::NP;
  __shared__ double lds[CB * L::cell], sface[CB * 52 * n];   // face adjoints [4][2][4][n], exchange [4][5][n] per cell
  const int t = threadIdx.x, lane = t % kWave;
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const double* gt = a.gtab;
  const double dt = a.clock[1];
  const int I = a.iters;

  // lines and time columns; idle lanes read along with lane 0 and write nothing
  const int s0 = L::grid8 ? 0 : lane / nn;
  const int h0 = L::grid8 ? lane / 8 : lane % nn / n, l0 = L::grid8 ? lane % 8 : lane % n;
  const bool act = L::grid8 ? h0 < n && l0 < n : s0 < CB;
  const int slot = act ? s0 : 0, hi = act ? h0 : 0, lo = act ? l0 : 0, r = hi * n + lo;
  const int c = min((int)blockIdx.x * CB + slot, a.C - 1);   // loads stay in bounds
  const bool valid = act && (int)blockIdx.x * CB + slot < a.C;
  double* A = lds + slot * L::cell + w * VS;
  double* B = A + buf;
  double* Cb = A + 2 * buf;
  double* Qb = A + 3 * buf;
  const int rowo = hi * BS + lo * JS, colo = hi * BS + lo * IS, timo = hi * JS + lo * IS;
  const double dth = dt / a.geom[4 * c + 2];
  const double* Qc = a.Qn + (size_t)c * sl + w * nn;
  const double* store = a.store + (size_t)c * I * n * sl + hi * sl + w * nn;

  // nodes
  const int cn = min((int)blockIdx.x * CB + t % (CB * nn) / nn, a.C - 1);
  FluxC fc;
  {
    const double h = a.geom[4 * cn + 2], ih = 1.0 / h;
    fc.gm1 = ph.gm1;
    fc.hgm1 = 0.5 * ph.gm1;
    fc.mu = ph.mu * ih;
    fc.mu23 = fc.mu * (2.0 / 3.0);
    fc.kap = ph.kappa * ih * ph.iR;
    fc.gh = ph.geff * h;
    fc.pb = 0.0;
  }
  int no[NP], nij[NP];   // offset and slice index of the thread's nodes
  double nw[NP], ngz[NP];   // their time weight and g z
  bool nact[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int id = t + p * L::NT, k = id % (CB * nn), i = id / (CB * nn);
    const int s = k / nn, b = k % nn / n, j = k % n;
    nact[p] = i < n;
    no[p] = nact[p] ? s * L::cell + b * BS + j * JS + i * IS : 0;
    nw[p] = gt[GTab::W * n + b];
    ngz[p] = ph.geff * (a.geom[4 * cn + 1] + a.geom[4 * cn + 2] * gt[GTab::XI * n + j]);
    nij[p] = nact[p] ? s * L::cell + j * n + i : 0;
  }

  // adjoints of the averaged state, fluxes and source, as slices [v][j][i]
  double X[n], aQn;
  {
    const double* lin = a.lam_in + (size_t)c * sl;
    const double ij = 1.0 / gt[GTab::W * n + hi], ii = 1.0 / gt[GTab::W * n + lo];
    aQn = lin[w * nn + r] * (ij * ii);
    double* A0 = A - w * VS;
    if (act) A0[2 * buf + w * nn + r] = aQn;
    FaceAdj<n> face;
    const int fs = t / (4 * n), ff = t % (4 * n) / n, fk = t % n;
    double* sf = sface + fs * 52 * n + ff * 8 * n;
    double* sx = sface + fs * 52 * n + 32 * n + ff * 5 * n;
    if (t < CB * 4 * n) face.load(ph, a, min((int)blockIdx.x * CB + fs, a.C - 1), ff, fk, sx);
    __syncthreads();
    if (t < CB * 4 * n) face.reverse(ph, fk, sx, sf);
    if (t < CB * 8 * n) {
      const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
      const int k = t % (8 * n), dir = k >= 4 * n, v = k % (4 * n) / n, line = k % n;
      const int base = t / (8 * n) * L::cell + v * nn + (dir ? line : line * n), st = dir ? n : 1;
      double in[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) in[m] = lds[2 * buf + base + m * st];
      D.apply(in, out);
#pragma unroll
      for (int m = 0; m < n; ++m) lds[dir * buf + base + m * st] = out[m];
    }
    __syncthreads();
    const double L0i = gt[GTab::L0 * n + lo] * ij, L1i = gt[GTab::L1 * n + lo] * ij;
    const double L0j = gt[GTab::L0 * n + hi] * ii, L1j = gt[GTab::L1 * n + hi] * ii;
    const double* f = sface + slot * 52 * n + w * n;
    double qa = fma(L0i, f[hi], L1i * f[8 * n + hi]);
    qa = fma(L0j, f[16 * n + lo], fma(L1j, f[24 * n + lo], qa));
    if (w == 0) qa = fma(-ph.geff * dt * (ij * ii), lin[2 * nn + r], qa);   // gravity source
    f += 4 * n;
    const double fx = fma(L0i, f[hi], L1i * f[8 * n + hi]), fz = fma(L0j, f[16 * n + lo], L1j * f[24 * n + lo]);
    if (act) {
      double* o = A0 + w * nn + r;
      o[0] = fma(dth, o[0], fx);
      o[buf] = fma(dth, o[buf], fz);
      o[2 * buf] = qa;
    }
  }

  // it = I: the time averages, at the last iterate; then the Picard sweeps in
  // reverse, q^{it+1}[a] = Q^n + dt sum_b P[a][b] R(q^it[b])
#pragma unroll 1
  for (int it = I; it >= 0; it = __builtin_amdgcn_readfirstlane(it - 1)) {
    double qr[n], qc[n];   // row and column of the iterate
    {
      const double* q = it > 0 ? store + (size_t)(it - 1) * n * sl : Qc;
#pragma unroll
      for (int m = 0; m < n; ++m) { qr[m] = q[lo * n + m]; qc[m] = q[m * n + lo]; }
    }
    if (it < I) {
      // R = S - (1/h)(Dx Fx + Dz Fz): residual adjoints times -1/h
      const ctab pt = scalar_table(gt + GTab::pt(n));
#pragma unroll
      for (int b = 0; b < n; ++b) aQn += X[b];
#pragma unroll
      for (int b = 0; b < n; ++b) {
        double s = pt[b * n] * X[0];
#pragma unroll
        for (int m = 1; m < n; ++m) s = fma(pt[b * n + m], X[m], s);
        if (act) Cb[timo + b * BS] = -dth * s;
      }
      __syncthreads();
      const EO<n> W(scalar_table(gt + GTab::eo_dw(n)));
      double in[n], im[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) { in[m] = Cb[rowo + m * IS]; im[m] = Cb[colo + m * JS]; }
      W.apply(in, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) A[rowo + m * IS] = out[m];
      }
      W.apply(im, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) B[colo + m * JS] = out[m];
      }
    }
    if (act) {
#pragma unroll
      for (int m = 0; m < n; ++m) Qb[rowo + m * IS] = qr[m];
    }
    __syncthreads();
    double aFx[NP][4], aFz[NP][4], add[NP][4];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const bool last = it == I;
      const double wb = last ? nw[p] : 1.0;
      const double* s = lds + (last ? nij[p] : no[p]);
      const int vs = last ? nn : VS;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        aFx[p][v] = wb * s[v * vs];
        aFz[p][v] = wb * s[buf + v * vs];
        add[p][v] = last ? wb * s[2 * buf + v * vs] : 0.0;
      }
      if (!last) add[p][0] = fc.gh * s[2 * buf + 2 * VS];   // gravity source of the sweep
    }
    __syncthreads();
    {
      const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
      double out[n];
      D.apply(qr, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) A[rowo + m * IS] = out[m];
      }
      D.apply(qc, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) B[colo + m * JS] = out[m];
      }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (nact[p]) {
        double* s = lds + no[p];
        double q[4], gx[4], gz[4], aq[4], agx[4], agz[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          gx[v] = s[v * VS];
          gz[v] = s[buf + v * VS];
          q[v] = s[3 * buf + v * VS];
        }
        fc.gz = ngz[p];
        flux_vjp(fc, q, gx, gz, aFx[p], aFz[p], aq, agx, agz);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          s[v * VS] = agx[v];
          s[buf + v * VS] = agz[v];
          s[2 * buf + v * VS] = aq[v] + add[p][v];
        }
      }
    __syncthreads();
    {
      // gradient adjoints back to the state
      const EO<n> W(scalar_table(gt + GTab::eo_dw(n)));
      double in[n], im[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) { in[m] = A[rowo + m * IS]; im[m] = B[colo + m * JS]; }
      W.apply(in, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) A[rowo + m * IS] = out[m];
      }
      W.apply(im, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) B[colo + m * JS] = out[m];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < n; ++b) {
      const int o = timo + b * BS;
      X[b] = Cb[o] + (A[o] + B[o]);
    }
  }
  // q^0[b] = Q^n for every b
#pragma unroll
  for (int b = 0; b < n; ++b) aQn += X[b];
  if (valid) a.lam_out[(size_t)c * sl + w * nn + r] = aQn * (gt[GTab::W * n + hi] * gt[GTab::W * n + lo]);
}

// ----------------------------------------------- initial state from theta'
// rho = p_bar / (R pi (theta_bg + theta')), E = p_bar/(gamma-1) + rho g z, at rest.
__global__ void k_ic_theta(Phys ph, int n, int C, const double* geom, const double* gtab, const double* thp,
                           double* Q) {
  const int nn = n * n;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)C * nn) return;
  const int c = (int)(gid / nn), node = (int)(gid % nn);
  const double z = geom[4 * c + 1] + geom[4 * c + 2] * gtab[GTab::XI * n + node / n];
  const double pi = 1.0 - ph.ex_coef * z;
  const double pb = ph.p0 * pow(pi, ph.cp_over_R);
  const double rho = pb / (ph.R * pi * (ph.theta + thp[(size_t)c * nn + node]));
  double* Qc = Q + (size_t)c * 4 * nn;
  Qc[node] = rho; Qc[nn + node] = 0.0; Qc[2 * nn + node] = 0.0;
  Qc[3 * nn + node] = pb / ph.gm1 + rho * ph.g * z;
}

__global__ void k_ic_theta_adj(Phys ph, int n, int C, const double* geom, const double* gtab, const double* thp,
                               const double* lam, double* grad) {
  const int nn = n * n;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)C * nn) return;
  const int c = (int)(gid / nn), node = (int)(gid % nn);
  const double z = geom[4 * c + 1] + geom[4 * c + 2] * gtab[GTab::XI * n + node / n];
  const double pi = 1.0 - ph.ex_coef * z;
  const double pb = ph.p0 * pow(pi, ph.cp_over_R);
  const double th = ph.theta + thp[(size_t)c * nn + node];
  const double rho = pb / (ph.R * pi * th);
  const double drho = -rho / th;
  const double* lc = lam + (size_t)c * 4 * nn;
  grad[(size_t)c * nn + node] = drho * (lc[node] + ph.g * z * lc[3 * nn + node]);
}

// ------------------------------------------------- potential-temperature loss
// L = sqrt(sum_cells h^2 sum_ji w_i w_j (theta - theta_bg)^2), theta =
// T (p0/p)^(R/cp).  Per-cell partial sums, then one workgroup sums them in a
// fixed order and takes the root.
template <int n>
__global__ __launch_bounds__(kWave) void k_loss_part(Phys ph, const double* Q, const double* geom, const double* gtab,
                                                       double* part) {
  constexpr int nn = n * n;
  const int c = blockIdx.x, lane = threadIdx.x;
  double v = 0.0;
  if (lane < nn) {
    const int jz = lane / n, ix = lane % n;
    const double h = geom[4 * c + 2];
    const double z = geom[4 * c + 1] + h * gtab[GTab::XI * n + jz];
    const double* Qc = Q + (size_t)c * 4 * nn;
    const double rho = Qc[lane];
    const double p = pressure(ph, rho, Qc[nn + lane], Qc[2 * nn + lane], Qc[3 * nn + lane], z);
    const double th = p / (rho * ph.R) * pow(ph.p0 / p, ph.R_over_cp) - ph.theta;
    v = h * h * gtab[GTab::W * n + ix] * gtab[GTab::W * n + jz] * th * th;
  }
  v = wave_sum(v);
  if (lane == 0) part[c] = v;
}

__global__ __launch_bounds__(256) void k_loss_sum(const double* part, int C, double* out) {
  __shared__ double s[256];
  const int t = threadIdx.x;
  double v = 0.0;
  for (int c = t; c < C; c += 256) v += part[c];
  s[t] = v;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (t < w) s[t] += s[t + w];
    __syncthreads();
  }
  if (t == 0) out[0] = sqrt(s[0]);
}

// lambda_Q = gL * dL/dQ = gL / L * h^2 w_i w_j (theta - theta_bg) dtheta/dQ
template <int n>
__global__ __launch_bounds__(kWave) void k_loss_adj(Phys ph, const double* Q, const double* geom, const double* gtab,
                                                      const double* L, const double* gL, double* lam) {
  constexpr int nn = n * n;
  const int c = blockIdx.x, lane = threadIdx.x;
  if (lane >= nn) return;
  const int jz = lane / n, ix = lane % n;
  const double h = geom[4 * c + 2];
  const double z = geom[4 * c + 1] + h * gtab[GTab::XI * n + jz];
  const double* Qc = Q + (size_t)c * 4 * nn;
  const double rho = Qc[lane], mx = Qc[nn + lane], mz = Qc[2 * nn + lane];
  const double p = pressure(ph, rho, mx, mz, Qc[3 * nn + lane], z);
  const double kap = ph.R_over_cp;
  const double th = p / (rho * ph.R) * pow(ph.p0 / p, kap);
  const double coef = gL[0] / L[0] * h * h * gtab[GTab::W * n + ix] * gtab[GTab::W * n + jz] * (th - ph.theta);
  // theta = (p0^kap / R) p^(1-kap) / rho
  const double dth_dp = (1.0 - kap) * th / p, dth_drho = -th / rho;
  const double u = mx / rho, w = mz / rho, geo = ph.gravity ? ph.g * z : 0.0;
  double* lc = lam + (size_t)c * 4 * nn;
  lc[lane] = coef * (dth_drho + dth_dp * ph.gm1 * (0.5 * (u * u + w * w) - geo));
  lc[nn + lane] = coef * dth_dp * (-ph.gm1 * u);
  lc[2 * nn + lane] = coef * dth_dp * (-ph.gm1 * w);
  lc[3 * nn + lane] = coef * dth_dp * ph.gm1;
}

// --------------------------------------------------------------- launchers
int launch_predictor(const Group& g, double* store, hipStream_t s);
int launch_corrector(const Group& g, hipStream_t s);

template <int n, int CB>
static void pred_adj_t(const Group& g, const AdjArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_pred_adj<n, CB>), dim3((g.C + CB - 1) / CB), dim3(4 * kWave), 0, s, g.ph, a);
}
template <int n>
static int adj_n(const Group& g, AdjArgs a, hipStream_t s) {
  // Up to one cell per CU, a workgroup for each cell; beyond, as many cells as
  // the lanes of a wavefront hold (one from n = 6 on).  One cell, several: 9 x 9
  // cells of n = 3 14.7, 16.2 us and of n = 5 18.9, 20.1; 16 x 16 of n = 4
  // 15.5, 15.3; 20 x 20 of n = 4 17.9, 15.0 and of n = 5 23.4, 19.9; 45 x 45 of
  // n = 3 35.5, 17.7.
  constexpr int CB = kWave / (n * n), kCus = 256;
  if (g.C <= kCus) pred_adj_t<n, 1>(g, a, s);
  else pred_adj_t<n, CB>(g, a, s);
  return check_launch("step adjoint");
}

int launch_step_adjoint(const Group& g, const double* Qn, const double* lam_in, double* lam_out, double* store,
                        const double* fd, bool recompute, hipStream_t s) {
  if (recompute) {
    // forward predictor from the checkpoint, keeping the iterates and the face data
    Group gf = g;
    gf.Q = const_cast<double*>(Qn);
    gf.FD = const_cast<double*>(fd);
    int rc = launch_predictor(gf, store, s);
    if (rc) return rc;
  }
  AdjArgs a;
  a.Qn = Qn; a.lam_in = lam_in; a.lam_out = lam_out; a.FD = fd; a.store = store;
  a.clock = g.clock; a.geom = g.d_geom; a.bg = g.d_bg; a.nbr = g.d_nbr; a.gtab = g.d_gtab;
  a.C = g.C; a.iters = g.iters;
  switch (g.n) {
    case 2: return adj_n<2>(g, a, s);
    case 3: return adj_n<3>(g, a, s);
    case 4: return adj_n<4>(g, a, s);
    case 5: return adj_n<5>(g, a, s);
    case 6: return adj_n<6>(g, a, s);
    case 7: return adj_n<7>(g, a, s);
    case 8: return adj_n<8>(g, a, s);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}

int launch_ic_theta(const Group& g, const double* thp, hipStream_t s) {
  const long long tot = (long long)g.C * g.n * g.n;
  if (!tot) return ADG_OK;
  hipLaunchKernelGGL(k_ic_theta, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, g.ph, g.n, g.C, g.d_geom,
                     g.d_gtab, thp, g.Q);
  return check_launch("ic_theta");
}

int launch_ic_theta_adj(const Group& g, const double* thp, const double* lam, double* grad, hipStream_t s) {
  const long long tot = (long long)g.C * g.n * g.n;
  if (!tot) return ADG_OK;
  hipLaunchKernelGGL(k_ic_theta_adj, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, g.ph, g.n, g.C,
                     g.d_geom, g.d_gtab, thp, lam, grad);
  return check_launch("ic_theta_adjoint");
}

template <int n>
static int loss_n(const Group& g, double* part, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_loss_part<n>, dim3(g.C), dim3(kWave), 0, s, g.ph, g.Q, g.d_geom, g.d_gtab, part);
  hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(256), 0, s, part, g.C, out);
  return check_launch("loss");
}
template <int n>
static int loss_adj_n(const Group& g, const double* L, const double* gL, double* lam, hipStream_t s) {
  hipLaunchKernelGGL(k_loss_adj<n>, dim3(g.C), dim3(kWave), 0, s, g.ph, g.Q, g.d_geom, g.d_gtab, L, gL, lam);
  return check_launch("loss adjoint");
}

int launch_loss(const Group& g, double* part, double* out, hipStream_t s) {
  switch (g.n) {
    case 2: return loss_n<2>(g, part, out, s);
    case 3: return loss_n<3>(g, part, out, s);
    case 4: return loss_n<4>(g, part, out, s);
    case 5: return loss_n<5>(g, part, out, s);
    case 6: return loss_n<6>(g, part, out, s);
    case 7: return loss_n<7>(g, part, out, s);
    case 8: return loss_n<8>(g, part, out, s);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}
int launch_loss_adj(const Group& g, const double* L, const double* gL, double* lam, hipStream_t s) {
  switch (g.n) {
    case 2: return loss_adj_n<2>(g, L, gL, lam, s);
    case 3: return loss_adj_n<3>(g, L, gL, lam, s);
    case 4: return loss_adj_n<4>(g, L, gL, lam, s);
    case 5: return loss_adj_n<5>(g, L, gL, lam, s);
    case 6: return loss_adj_n<6>(g, L, gL, lam, s);
    case 7: return loss_adj_n<7>(g, L, gL, lam, s);
    case 8: return loss_adj_n<8>(g, L, gL, lam, s);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}

}  // namespace adg
