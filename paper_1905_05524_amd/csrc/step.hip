// ADER-DG step kernels for gfx950: corrector with the viscous Rusanov face
// flux (conforming, wall and 1:3 non-conforming faces), CFL time step, clock.
//
// Work decomposition.  A wavefront (64 lanes) owns CPW cells (CPW * n*n <=
// 64); a workgroup holds WPB independent wavefronts, each with its own LDS
// region, synchronised at wavefront level only.  In a cell, lane (slot, l)
// with l < n*n owns spatial node (j, i) = (l / n, l % n); in the face phase
// lane (slot, f, k) handles face f at node k.  CPW and WPB are template
// parameters picked by order, or by the caller's launch shape.
#include "step_internal.h"

namespace adg {

// LDS of the corrector, doubles per cell: sG [4][4][n], sL/sV [4][3][n] each,
// sGs [4][3][4][n].
template <int n, int CPW>
struct Lay {
  static constexpr int nn = n * n, sl = 4 * nn;
  static constexpr int corr_cell = 16 * n + 24 * n + 48 * n;
};

// ------------------------------------------------------------------ corrector
// Ghost state and flux at a no-slip wall: mirrored velocity, background
// density and pressure (interior ones without gravity), mass flux mirrored,
// momentum flux copied, energy flux 2 q_bg - F with the background
// conductive flux q_bg = kappa g / cp through horizontal walls.
// bg: the background at the face node.
__device__ inline void wall_ghost(const Phys& ph, int d, double zf, const double bg[2], const double Qi[4],
                                  const double Fi[4], double Qg[4], double Fg[4]) {
  const double u = Qi[1] / Qi[0], w = Qi[2] / Qi[0];
  double rb, pb;
  if (ph.gravity) { rb = bg[0]; pb = bg[1]; }
  else { rb = Qi[0]; pb = pressure(ph, Qi[0], Qi[1], Qi[2], Qi[3], zf); }
  const double geo = ph.gravity ? rb * (ph.g * zf) : 0.0;
  Qg[0] = rb;
  Qg[1] = -(rb * u);
  Qg[2] = -(rb * w);
  Qg[3] = pb / ph.gm1 + 0.5 * rb * (u * u + w * w) + geo;
  const double qbg = (ph.gravity && d == 1) ? ph.kappa * ph.g / ph.cp : 0.0;
  Fg[0] = -Fi[0];
  Fg[1] = Fi[1];
  Fg[2] = Fi[2];
  Fg[3] = 2.0 * qbg - Fi[3];
}

// |v| + c and lambda_v for the larger of the momenta ma, mb (one twice: the
// normal speed of a face): one reciprocal and one square root, where the two
// directions of a node apart took four divisions and two roots (|1/rho|: the
// velocity's magnitude also where a flow has driven rho below zero)
__device__ inline void eig(const Phys& ph, const double q[4], double ma, double mb, double z, double& lam, double& lv) {
  const double ir = recip(q[0]);
  const double ke = fma(q[1], q[1], q[2] * q[2]) * ir;                        // rho |v|^2
  const double p = ph.gm1 * (fma(-0.5, ke, q[3]) - q[0] * (ph.geff * z));
  lam = fmax(fabs(ma), fabs(mb)) * fabs(ir) + sqrt(ph.gamma * p * ir);
  lv = ph.lv_coef * ir;
}

// face data of cell cf, face f, node k: averaged state and normal flux
template <int n>
__device__ inline void load_face(const double* FD, int cf, int f, int k, double Q[4], double F[4]) {
  const double* fd = FD + (size_t)cf * 32 * n + f * 8 * n;
#pragma unroll
  for (int v = 0; v < 4; ++v) { Q[v] = fd[v * n + k]; F[v] = fd[4 * n + v * n + k]; }
}

// face polynomial of cell cf, face f, evaluated at node q of sub-face s
template <int n>
__device__ inline void prolong_face(const double* FD, const double* gt, int cf, int f, int s, int q, double Q[4],
                                    double F[4]) {
  const double* fd = FD + (size_t)cf * 32 * n + f * 8 * n;
  const double* P = gt + GTab::pk(n) + (s * n + q) * n;
#pragma unroll
  for (int v = 0; v < 4; ++v) { Q[v] = 0.0; F[v] = 0.0; }
#pragma unroll
  for (int m = 0; m < n; ++m) {
    const double p = P[m];
#pragma unroll
    for (int v = 0; v < 4; ++v) { Q[v] = fma(p, fd[v * n + m], Q[v]); F[v] = fma(p, fd[4 * n + v * n + m], F[v]); }
  }
}

// Per cell: lanes (slot, f, k) handle face f at node k.  The Rusanov speed s
// is one value per (sub-)face: max over the face nodes of both sides of the
// normal eigenvalue bound, plus the viscous penalty 2 eta max lambda_v with
// eta = (2N+1)/(h sqrt(pi/2)), h the (finer) cell size at the face.
// Conforming: the neighbour's face data; wall: ghost data; fine side of a
// 1:3 face: the coarse neighbour's face polynomial at this sub-face; coarse
// side: the three sub-face fluxes restricted by L2 projection.  Both sides of
// a face evaluate the identical expressions, so the fluxes agree bitwise.
template <int n, int CPW, int WPB, bool NC>
__global__ __launch_bounds__(kWave * WPB) void k_corrector(Phys ph, StepArgs a) {
  using L = Lay<n, CPW>;
  constexpr int nn = L::nn, sl = L::sl;
  extern __shared__ double lds[];
  constexpr bool by_lds = CPW > 1 && nn != 4 && nn != 16;   // maxima over a cell's nodes
  __shared__ double slam[by_lds ? WPB : 1][2][by_lds ? kWave : 1];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  double* wl = lds + (size_t)wave * CPW * L::corr_cell;
  const int cell0 = (blockIdx.x * WPB + wave) * CPW;
  const double* gt = a.gtab;
  const double eta0 = (2.0 * ph.N + 1.0) / 1.2533141373155002512;   // (2N+1)/sqrt(pi/2)

  // Q* of this lane's node, loaded first so that its latency overlaps the
  // face phase
  const int slot = lane / nn, l = lane % nn;
  const int c = cell0 + slot;
  const bool valid = slot < CPW && c < a.C;
  double qsv[4] = {0.0, 0.0, 0.0, 0.0};
  if (valid) {
    const double* qs = a.Qs + (size_t)c * sl;
#pragma unroll
    for (int v = 0; v < 4; ++v) qsv[v] = qs[v * nn + l];
  }

  // face role
  const int fslot = lane / (4 * n);
  const int f = (lane % (4 * n)) / n, k = lane % n;
  const int fc = cell0 + fslot;
  const bool fl = fslot < CPW && fc < a.C;
  double* fw = wl + (fslot < CPW ? fslot : 0) * L::corr_cell;
  double* sG = fw;                 // [4 faces][4 vars][n]
  double* sL = fw + 16 * n;        // [4][3][n]
  double* sV = sL + 12 * n;        // [4][3][n]
  double* sGs = sV + 12 * n;       // [4][3][4][n]
  const int d = f >> 1;
  const bool lower = (f & 1) == 0;   // face on the lower side: this cell is R
  int kind = kWall, nb1 = 0, nb2 = 0, nb3 = 0;
  double hf = 1.0, z0f = 0.0;
  // Rusanov flux G = S/2 - (s/2) J from the flux sums S and the jumps J of the
  // face (three sub-faces on the coarse side)
  constexpr int NF = NC ? 3 : 1;
  double Sf[NF][4], Jf[NF][4];
  auto sides = [&](int s, const double Qm[4], const double Fm[4], const double Qo[4], const double Fo[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      Sf[s][v] = Fm[v] + Fo[v];
      Jf[s][v] = lower ? Qm[v] - Qo[v] : Qo[v] - Qm[v];
    }
  };
  if (fl) {
    double Qm[4], Fm[4], Qo[4], Fo[4], l1, v1, l2, v2;
    const int* nb = a.nbr + (size_t)fc * 16 + f * 4;
    kind = nb[0]; nb1 = nb[1]; nb2 = nb[2]; nb3 = nb[3];
    hf = a.geom[4 * fc + 2]; z0f = a.geom[4 * fc + 1];
    if (!NC || kind != kCoarseSide) {
      const double zf = (d == 0) ? z0f + hf * gt[GTab::XI * n + k] : z0f + ((f & 1) ? hf : 0.0);
      load_face<n>(a.FD, fc, f, k, Qm, Fm);
      if (kind == kConforming) load_face<n>(a.FD, nb1, f ^ 1, k, Qo, Fo);
      else if (NC && kind == kFineSide) prolong_face<n>(a.FD, gt, nb1, f ^ 1, nb2, k, Qo, Fo);
      else wall_ghost(ph, d, zf, a.bg + 2 * ((size_t)fc * (n + 2) + (d == 0 ? k : n + (f & 1))), Qm, Fm, Qo, Fo);
      eig(ph, Qm, Qm[1 + d], Qm[1 + d], zf, l1, v1);
      eig(ph, Qo, Qo[1 + d], Qo[1 + d], zf, l2, v2);
      sides(0, Qm, Fm, Qo, Fo);
      sL[(f * 3) * n + k] = fmax(l1, l2);
      sV[(f * 3) * n + k] = fmax(v1, v2);
    } else if constexpr (NC) {
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        const int fine = s == 0 ? nb1 : (s == 1 ? nb2 : nb3);
        const double zf = (d == 0) ? z0f + hf * (s + gt[GTab::XI * n + k]) / 3.0 : z0f + ((f & 1) ? hf : 0.0);
        prolong_face<n>(a.FD, gt, fc, f, s, k, Qm, Fm);
        load_face<n>(a.FD, fine, f ^ 1, k, Qo, Fo);
        eig(ph, Qm, Qm[1 + d], Qm[1 + d], zf, l1, v1);
        eig(ph, Qo, Qo[1 + d], Qo[1 + d], zf, l2, v2);
        sides(s, Qm, Fm, Qo, Fo);
        sL[(f * 3 + s) * n + k] = fmax(l1, l2);
        sV[(f * 3 + s) * n + k] = fmax(v1, v2);
      }
    }
  }
  wave_sync();
  if (fl) {
    if (!NC || kind != kCoarseSide) {
      double lam = sL[(f * 3) * n], lv = sV[(f * 3) * n];
#pragma unroll
      for (int m = 1; m < n; ++m) { lam = fmax(lam, sL[(f * 3) * n + m]); lv = fmax(lv, sV[(f * 3) * n + m]); }
      const double s = lam + 2.0 * (eta0 / hf) * lv;
#pragma unroll
      for (int v = 0; v < 4; ++v) sG[(f * 4 + v) * n + k] = 0.5 * Sf[0][v] - 0.5 * s * Jf[0][v];
    } else if constexpr (NC) {
      const double hfine = hf / 3.0;
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        double lam = sL[(f * 3 + s) * n], lv = sV[(f * 3 + s) * n];
#pragma unroll
        for (int m = 1; m < n; ++m) { lam = fmax(lam, sL[(f * 3 + s) * n + m]); lv = fmax(lv, sV[(f * 3 + s) * n + m]); }
        const double sp = lam + 2.0 * (eta0 / hfine) * lv;
#pragma unroll
        for (int v = 0; v < 4; ++v) sGs[((f * 3 + s) * 4 + v) * n + k] = 0.5 * Sf[s][v] - 0.5 * sp * Jf[s][v];
      }
    }
  }
  wave_sync();
  if (NC && fl && kind == kCoarseSide) {
    // L2 restriction to the coarse face node m = k
    const double* Rk = gt + GTab::rk(n);
    double G[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int q = 0; q < n; ++q) {
        const double r = Rk[(s * n + k) * n + q];
#pragma unroll
        for (int v = 0; v < 4; ++v) G[v] = fma(r, sGs[((f * 3 + s) * 4 + v) * n + q], G[v]);
      }
#pragma unroll
    for (int v = 0; v < 4; ++v) sG[(f * 4 + v) * n + k] = G[v];
  }
  wave_sync();

  // node role: lifting and the next CFL candidate
  const double* sGc = wl + (slot < CPW ? slot : 0) * L::corr_cell;
  double lam_n = 0.0, lv_n = 0.0;
  if (valid) {
    const int jz = l / n, ix = l % n;
    const int sc = a.scen ? a.scen[c] : 0;
    const double dt = a.clock[4 * sc + 1];
    const double z0 = a.geom[4 * c + 1], h = a.geom[4 * c + 2];
    const double L0i = gt[GTab::L0 * n + ix], L1i = gt[GTab::L1 * n + ix];
    const double L0j = gt[GTab::L0 * n + jz], L1j = gt[GTab::L1 * n + jz];
    double* qo = a.Qout + (size_t)c * sl;
    const double scl = dt / h;
    double q[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double sx = L1i * sGc[(1 * 4 + v) * n + jz] - L0i * sGc[(0 * 4 + v) * n + jz];
      const double sz = L1j * sGc[(3 * 4 + v) * n + ix] - L0j * sGc[(2 * 4 + v) * n + ix];
      q[v] = qsv[v] - scl * (sx + sz);
      qo[v * nn + l] = q[v];
    }
    if (!ph.fixed_dt) {
      const double zz = z0 + h * gt[GTab::XI * n + jz];
      eig(ph, q, q[1], q[2], zz, lam_n, lv_n);
    }
  }
  if (!ph.fixed_dt) {
    // maxima of lambda and lambda_v over the nodes of each cell slot (a
    // contiguous lane range), then the CFL rule on the cell maxima
    double lm, vm;
    if constexpr (CPW == 1) {
      lm = wave_max(lam_n);   // lanes without a node hold 0
      vm = wave_max(lv_n);
    } else if constexpr (nn == 4) {
      lm = quad_max(lam_n);
      vm = quad_max(lv_n);
    } else if constexpr (nn == 16) {
      lm = row_max(lam_n);
      vm = row_max(lv_n);
    } else {
      slam[wave][0][lane] = lam_n;
      slam[wave][1][lane] = lv_n;
      wave_sync();
      lm = lam_n; vm = lv_n;
      if (valid && l == 0)
        for (int j = 1; j < nn; ++j) { lm = fmax(lm, slam[wave][0][lane + j]); vm = fmax(vm, slam[wave][1][lane + j]); }
    }
    if (valid && l == 0) {
      const double h = a.geom[4 * c + 2];
      const double o = 2.0 * ph.N + 1.0;
      a.dtc[c] = ph.cfl * h / (2.0 * o * (lm + 2.0 * vm * o / h));
    }
  }
  // a frozen time step: the clock advances here, with no reduction to wait
  // for (the corrector reads only dt, which does not change)
  if (a.advance && blockIdx.x == 0 && threadIdx.x == 0) {
    a.advance[0] += a.advance[1];
    a.advance[3] += 1.0;
  }
}

// per-cell CFL candidate from the current state (no update)
template <int n>
__global__ __launch_bounds__(kWave) void k_cell_dt(Phys ph, StepArgs a) {
  constexpr int nn = n * n;
  const int c = blockIdx.x;
  const int lane = threadIdx.x;
  const double z0 = a.geom[4 * c + 1], h = a.geom[4 * c + 2];
  double lam = 0.0, lvm = 0.0;
  if (lane < nn) {
    const int jz = lane / n;
    const double* Qc = a.Qin + (size_t)c * 4 * nn;
    double q[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) q[v] = Qc[v * nn + lane];
    const double z = z0 + h * a.gtab[GTab::XI * n + jz];
    eig(ph, q, q[1], q[2], z, lam, lvm);
  }
  lam = wave_max(lam);
  lvm = wave_max(lvm);
  if (lane == 0) {
    const double o = 2.0 * ph.N + 1.0;
    a.dtc[c] = ph.cfl * h / (2.0 * o * (lam + 2.0 * lvm * o / h));
  }
}

// Clock update, one workgroup per scenario: if advance, t += dt and
// steps += 1; if update, dt <- min of the CFL candidates of the scenario's
// cells [beg[s], end[s]) (min is exact, so the result is order independent).
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void k_clock(double* clock, const double* dtc, const int* beg,
                                                           const int* end, int C, int advance, int update) {
  __shared__ double sm[kReduceThreads / kWave];
  const int s = blockIdx.x, t = threadIdx.x;
  const int b0 = beg ? beg[s] : 0, b1 = end ? end[s] : C;
  // the clock is read before the reduction so that its latency overlaps it
  double t_old = 0.0, dt_old = 0.0, n_old = 0.0;
  if (t == 0) { t_old = clock[4 * s + 0]; dt_old = clock[4 * s + 1]; n_old = clock[4 * s + 3]; }
  double m = __builtin_inf();
  if (update) {
    // four independent loads in flight per thread
    int c = b0 + t;
    for (; c + 3 * kReduceThreads < b1; c += 4 * kReduceThreads) {
      const double a0 = dtc[c], a1 = dtc[c + kReduceThreads], a2 = dtc[c + 2 * kReduceThreads],
                   a3 = dtc[c + 3 * kReduceThreads];
      m = fmin(m, fmin(fmin(a0, a1), fmin(a2, a3)));
    }
    for (; c < b1; c += kReduceThreads) m = fmin(m, dtc[c]);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) m = fmin(m, __shfl_xor(m, o, kWave));
  if ((t & (kWave - 1)) == 0) sm[t / kWave] = m;
  __syncthreads();
  if (t == 0) {
    double r = sm[0];
    for (int k = 1; k < kReduceThreads / kWave; ++k) r = fmin(r, sm[k]);
    if (advance) { clock[4 * s + 0] = t_old + dt_old; clock[4 * s + 3] = n_old + 1.0; }
    if (update) clock[4 * s + 1] = r;
  }
}

// Minimum of every chunk of len candidates.
constexpr int kChunkThreads = 256;
__global__ __launch_bounds__(kChunkThreads) void k_chunk_min(const double* dtc, double* part, int C, int len) {
  __shared__ double sm[kChunkThreads / kWave];
  const int t = threadIdx.x;
  const long long b0 = (long long)blockIdx.x * len, b1 = min(b0 + len, (long long)C);
  double m = __builtin_inf();
  for (long long c = b0 + t; c < b1; c += kChunkThreads) m = fmin(m, dtc[c]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) m = fmin(m, __shfl_xor(m, o, kWave));
  if ((t & (kWave - 1)) == 0) sm[t / kWave] = m;
  __syncthreads();
  if (t == 0) {
    for (int k = 1; k < kChunkThreads / kWave; ++k) m = fmin(m, sm[k]);
    part[blockIdx.x] = m;
  }
}

// Background of the node rows, the bottom and the top of every cell, once per
// mesh (or regrid): the power function is 250 of the 2,000 to 8,700 vector
// instructions of a predictor's lane at n = 4 to 7, and a microsecond of the
// chain of a small mesh's step.
__global__ void k_background(Phys ph, int n, int C, const double* geom, const double* gtab, double* bg) {
  const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long long)C * (n + 2)) return;
  const int c = (int)(g / (n + 2)), k = (int)(g % (n + 2));
  const double z0 = geom[4 * c + 1], h = geom[4 * c + 2];
  double rb, pb;
  background(ph, k < n ? z0 + h * gtab[GTab::XI * n + k] : z0 + (k > n ? h : 0.0), rb, pb);
  bg[2 * g] = rb;
  bg[2 * g + 1] = pb;
}

// --------------------------------------------------------------- dispatchers
int launch_background(const Group& g, int C, hipStream_t s) {
  const long long tot = (long long)C * (g.n + 2);
  if (tot == 0) return ADG_OK;
  hipLaunchKernelGGL(k_background, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, g.ph, g.n, C, g.d_geom, g.d_gtab,
                     g.d_bg);
  return check_launch("background");
}

StepArgs make_args(const Group& g) {
  StepArgs a;
  a.Qin = g.Q; a.Qout = g.Q; a.Qs = g.Qs; a.FD = g.FD; a.dtc = g.dtc;
  a.clock = g.clock; a.scen = g.d_scen; a.geom = g.d_geom; a.bg = g.d_bg; a.nbr = g.d_nbr; a.gtab = g.d_gtab;
  a.C = g.C; a.iters = g.iters;
  a.iter_store = nullptr;
  a.advance = g.advance;
  return a;
}

template <int n, int CPW, int WPB>
static int launch_corr_t(const Group& g, hipStream_t s) {
  using L = Lay<n, CPW>;
  const size_t lds = sizeof(double) * (size_t)WPB * CPW * L::corr_cell;
  const int per_block = CPW * WPB;
  const int blocks = (g.C + per_block - 1) / per_block;
  if (blocks == 0) return ADG_OK;
  // meshes without 1:3 faces take the variant without their code paths
  if (g.nc)
    hipLaunchKernelGGL((k_corrector<n, CPW, WPB, true>), dim3(blocks), dim3(kWave * WPB), lds, s, g.ph,
                       make_args(g));
  else
    hipLaunchKernelGGL((k_corrector<n, CPW, WPB, false>), dim3(blocks), dim3(kWave * WPB), lds, s, g.ph,
                       make_args(g));
  return check_launch("corrector");
}

template <int n, int CPW>
static int corr_w(const Group& g, hipStream_t s) {
  switch (g.wpb) {
    case 1: return launch_corr_t<n, CPW, 1>(g, s);
    case 2: return launch_corr_t<n, CPW, 2>(g, s);
    case 4: return launch_corr_t<n, CPW, 4>(g, s);
    default: return fail(ADG_EINVAL, "waves per block must be 1, 2 or 4");
  }
}
// Cells per wavefront of a launch without a shape of its own: as many as have
// a lane for every node and every face node.  One cell for each wavefront
// takes 47 to 48 us for 200 x 200 cells, with the clock, at every n up to 6 (1.2
// ns a cell, the rate of the wavefronts); with them packed, 17 us at n = 2, 21 at
// n = 3, 26 at n = 4 and 35 at n = 5, near the time of their memory traffic, and
// no mesh of 81 to 3,600 cells gets slower.  At n = 6 and 7 (48 and 50 us) the
// traffic bounds one cell per wavefront already.
constexpr int corr_cells(int n) { return n == 2 ? 8 : n == 3 ? 5 : n == 4 ? 4 : n == 5 ? 2 : 1; }
// cells per wavefront of a launch shape: 1, 2 or 4 (while CPW * n^2 <= 64)
template <int n>
static int corr_n(const Group& g, hipStream_t s) {
  constexpr int nn = n * n;
  if (g.lv != 0) return launch_corr_t<n, corr_cells(n), 1>(g, s);
  if (g.cpw == 1) return corr_w<n, 1>(g, s);
  if constexpr (2 * nn <= kWave) { if (g.cpw == 2) return corr_w<n, 2>(g, s); }
  if constexpr (4 * nn <= kWave) { if (g.cpw == 4) return corr_w<n, 4>(g, s); }
  return fail(ADG_EINVAL, "cells per wavefront not supported for this order");
}
template <int n>
static int dt_n(const Group& g, hipStream_t s) {
  if (g.C == 0) return ADG_OK;
  hipLaunchKernelGGL(k_cell_dt<n>, dim3(g.C), dim3(kWave), 0, s, g.ph, make_args(g));
  return check_launch("cell_dt");
}

#define ADG_DISPATCH_N(fn, g, s)                                   \
  switch ((g).n) {                                                 \
    case 2: return fn<2>(g, s);                                    \
    case 3: return fn<3>(g, s);                                    \
    case 4: return fn<4>(g, s);                                    \
    case 5: return fn<5>(g, s);                                    \
    case 6: return fn<6>(g, s);                                    \
    case 7: return fn<7>(g, s);                                    \
    case 8: return fn<8>(g, s);                                    \
    default: return fail(ADG_EUNSUPPORTED, "order not supported"); \
  }

int launch_corrector(const Group& g, hipStream_t s) { ADG_DISPATCH_N(corr_n, g, s); }
int launch_cell_dt(const Group& g, hipStream_t s) { ADG_DISPATCH_N(dt_n, g, s); }

int launch_clock(double* clock, const double* dtc, double* part, const int* beg, const int* end, int nscen, int C,
                 int advance, int update, hipStream_t s) {
  if (nscen <= 0) return ADG_OK;
  // One mesh of many cells with room for the chunks' minima (part: the
  // candidates themselves stay, callers read them): one workgroup reads no more
  // than 50 GB/s, so 256 of them reduce chunks first.  Corrector and clock in one stage and in two:
  // 22,500 cells of n = 2 12.2 and 11.9 us (a step 32.1 and 32.5), 32,400 17.3
  // and 15.6, 62,500 26.6 and 22.5, 531,441 of n = 7 868 and 791.
  if (part && !beg && update && C > kOneStage) {
    const int len = (C + kChunks - 1) / kChunks, chunks = (C + len - 1) / len;
    hipLaunchKernelGGL(k_chunk_min, dim3(chunks), dim3(kChunkThreads), 0, s, dtc, part, C, len);
    dtc = part;
    C = chunks;
  }
  hipLaunchKernelGGL(k_clock, dim3(nscen), dim3(kReduceThreads), 0, s, clock, dtc, beg, end, C, advance, update);
  return check_launch("clock");
}

int max_cpw(int n) { return max_cpw_c(n); }

}  // namespace adg
