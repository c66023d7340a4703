// Space-time predictor for gfx950, one lane per (time level, row of nodes).
//
// Work decomposition.  n^2 lanes work on a cell and hold n nodes of the four
// variables each, in one of three layouts:
//   time columns  lane (j, i) holds the n time levels of node (j, i);
//   rows          lane (b, j) holds the n nodes of row j at time level b;
//   columns       lane (b, i) holds the n nodes of column i at level b.
// The contraction along the dimension that a lane holds runs in its
// registers, with the tables in scalar registers, and the layouts change
// through one LDS buffer per cell, [variable][level][j][i].  A Picard sweep
// is six stages of n independent nodes: iterate out (time columns), z
// gradients in place (columns) beside the x gradients (rows), fluxes (rows,
// in place), z divergence (columns) beside the x divergence (rows), their
// sum, residuals in (time columns) and the time solve.  The mass flux is the
// momentum, so the mass residual is the sum of two momentum gradients and
// three variables, not four, go through the divergences.
//
// What bounds it (counters at 243 x 243 cells, n = 7): the vector units are
// busy 70 % of the time (8,390 vector instructions per cell), the LDS 63 %; at
// 81 x 81 cells, with a nearly empty third round of wavefronts, 54 and 49 %.
// The kernel before it kept one node per lane and went through LDS for every
// contraction of one time level at a time (26 writes and 30 reads per node
// and level against 18 and 22 here, and 28 dependent LDS stages per sweep
// against 6).  Per launch, before and now: 81 x 81 cells n = 7 190 and
// 149 us, 243 x 243 1.47 and 1.17 ms; 81 x 81 n = 8 800 and 228 us, n = 6
// 137 and 88 us, n = 5 87 and 45 us, n = 4 58 and 21 us, n = 3 29 and
// 12 us, n = 2 17 and 9 us.
//
// LDS strides.  A probe of ds_read2_b64 and ds_write_b64 fits four passes of
// 16 lanes over 16 banks of one double: a read costs max(4, sum over the
// passes of the fullest bank) clocks, a write max(6.5, the same).  The
// strides below make the row and column accesses free of conflicts; at n = 6
// and 7 with one cell per wavefront lane 8 hi + lo does it for all three
// layouts (2e6 conflict cycles at 81 x 81 against 2.1e7 with lane 7 hi + lo,
// 166 against 190 us).
#include "step_internal.h"

namespace adg {

// Momentum and energy fluxes along x and z at one node (eqs. equation-set,
// eos, temperature, stress-tensor, heat-conduction-coeff,
// momentum-equation-split).  q: state; gx, gz: gradients in reference
// coordinates (the 1/h sits in mu, kap and gh).  The mass fluxes are the
// momenta themselves and are left out.  With a = rho du/dx etc. the
// divisions by rho collect in ir; the two shear fluxes mx w + sxz and
// mz u + sxz are one number.  Every product that meets a sum does so in an
// explicit fused operation: the kernels' results agree bit for bit.
__device__ inline void flux_xz(const FluxC& c, const double q[4], const double gx[4], const double gz[4],
                               double Fx[3], double Fz[3]) {
  const double rho = q[0], mx = q[1], mz = q[2], E = q[3];
  const double ir = recip(rho);
  const double u = mx * ir, w = mz * ir;
  const double ke = fma(mx, u, mz * w);                    // rho |v|^2
  const double p = fma(-c.hgm1, ke, c.gm1 * fma(-c.gz, rho, E));
  const double pm = p - c.pb;
  const double pir = p * ir;                               // R T
  const double ax = fma(-u, gx[0], gx[1]), az = fma(-u, gz[0], gz[1]);   // rho du
  const double cx = fma(-w, gx[0], gx[2]), cz = fma(-w, gz[0], gz[2]);   // rho dw
  const double hv = fma(0.5 * ir, ke, c.gz);
  const double dx = fma(-w, cx, fma(-u, ax, fma(-hv, gx[0], gx[3])));    // dp / gm1
  const double dz = fma(-c.gh, rho, fma(-w, cz, fma(-u, az, fma(-hv, gz[0], gz[3]))));
  const double m23 = c.mu23 * ir;
  const double exx = fma(-2.0, ax, cz), ezz = fma(-2.0, cz, ax);         // sxx = m23 exx, szz = m23 ezz
  const double sxz = -(c.mu * ir) * (az + cx);
  const double k = c.kap * ir;
  const double qx = fma(-pir, gx[0], c.gm1 * dx), qz = fma(-pir, gz[0], c.gm1 * dz);
  const double H = E + p;
  Fx[0] = fma(mx, u, fma(m23, exx, pm));
  Fx[1] = fma(mx, w, sxz);
  Fx[2] = fma(-k, qx, fma(w, sxz, u * fma(m23, exx, H)));
  Fz[0] = Fx[1];
  Fz[1] = fma(mz, w, fma(m23, ezz, pm));
  Fz[2] = fma(-k, qz, fma(u, sxz, w * fma(m23, ezz, H)));
}

// Instructions do not move across this line: it bounds how many loads the
// scheduler hoists, and so the registers they hold.
__device__ inline void fence_schedule() { __builtin_amdgcn_sched_barrier(0); }

// In-place derivative of the lane's columns of variables v0..3 and, from its
// rows q, the derivative along the rows (out of place for the gradients, in
// place of g for the divergences).  The next column is read while one is
// worked on.
template <int n, int VS, int JS, int v0>
__device__ __forceinline__ void derivatives(const EO<n>& D, double* colp, const double (&q)[4][n], double (&g)[4][n]) {
  double in[2][n], out[n];
  auto read = [&](int v) {
#pragma unroll
    for (int m = 0; m < n; ++m) in[v & 1][m] = colp[v * VS + m * JS];
  };
  read(v0);
#pragma unroll
  for (int v = v0; v < 4; ++v) {
    if (v < 3) read(v + 1);
    D.apply(in[v & 1], out);
#pragma unroll
    for (int m = 0; m < n; ++m) colp[v * VS + m * JS] = out[m];
    D.apply(q[v], out);
#pragma unroll
    for (int m = 0; m < n; ++m) g[v][m] = out[m];
    fence_schedule();
  }
}

// Cells per workgroup (CB), wavefronts per workgroup (WV) and LDS strides.
template <int n, int CB, int WV>
struct RowsLay {
  static constexpr int nn = n * n;
  // one cell per wavefront at n = 6, 7: lane 8 hi + lo; else lanes hi n + lo
  static constexpr bool grid8 = CB == 1 && WV == 1 && (n == 6 || n == 7);
  static_assert(grid8 || CB * nn <= kWave * WV, "a lane per time level and row");
  // strides of level, row and node within a variable; doubles per variable
  static constexpr int BS = grid8 ? 8 : n, JS = 1;
  static constexpr int IS = grid8 ? 55 : n == 8 ? 65 : n == 7 ? 49 : n == 6 ? 41 : n == 5 ? 25 : n == 4 ? 19 : n == 3 ? 10 : 4;
  static constexpr int VS = (n - 1) * (BS + JS + IS) + 1;
  // doubles per cell: the variables, or the three node slices of a single
  // level; with several cells the cell stride sets the banks of the next one
  static constexpr int cell0 = 4 * VS > 12 * nn ? 4 * VS : 12 * nn;
  static constexpr int cell = CB == 1 ? cell0 : n == 7 ? 1377 : n == 6 ? 964 : n == 5 ? 505 : n == 4 ? 292 : n == 3 ? 121 : cell0;
  static_assert(cell >= cell0, "the padded cell holds its arrays");
};

// Predictor of the CB cells starting at cell0 by one workgroup of WV
// wavefronts.  ms: doubles per cell of the density wave's source (n^3, or 0).
template <int n, int CB, int WV, bool PW>
__device__ __forceinline__ void predict_rows(const Phys& ph, const StepArgs& a, double* lds, int ms, int cell0) {
  using L = RowsLay<n, CB, WV>;
  constexpr int nn = L::nn, sl = 4 * nn, BS = L::BS, JS = L::JS, IS = L::IS, VS = L::VS;
  auto sync = [] {
    if constexpr (WV == 1) wave_sync();
    else __syncthreads();
  };
  const int t = threadIdx.x;
  const int slot = L::grid8 ? 0 : t / nn;
  const int h0 = L::grid8 ? t / 8 : (t % nn) / n, l0 = L::grid8 ? t % 8 : t % nn % n;
  const bool act = L::grid8 ? h0 < n && l0 < n : slot < CB;
  // the lane's (j, i), (b, j) or (b, i); idle lanes read along with lane 0
  const int hi = act ? h0 : 0, lo = act ? l0 : 0;
  if (CB > 1 && !act) return;
  const int r = hi * n + lo;                           // node of the time column
  const int cell = CB == 1 ? cell0 : cell0 + (act ? slot : 0);
  const bool valid = act && cell < a.C;
  const int cc = cell < a.C ? cell : a.C - 1;          // loads stay in bounds; only valid lanes store
  double* S = lds + (act ? slot : 0) * (L::cell + ms);
  const double* gt = a.gtab;
  double* rowp = S + hi * BS + lo * JS;                // the lane's row (stride IS)
  double* colp = S + hi * BS + lo * IS;                // the lane's column (stride JS)
  double* timp = S + hi * JS + lo * IS;                // the lane's time column (stride BS)

  const int s = a.scen ? a.scen[cc] : 0;
  const double t0 = a.clock[4 * s + 0], dt = a.clock[4 * s + 1];
  const double x0 = a.geom[4 * cc + 0], z0 = a.geom[4 * cc + 1], h = a.geom[4 * cc + 2];
  double ih = 1.0 / h;
  if constexpr (CB == 1) ih = uniform(ih);
  FluxC fc;
  fc.gm1 = ph.gm1;
  fc.hgm1 = 0.5 * ph.gm1;
  fc.mu = ph.mu * ih;
  fc.mu23 = fc.mu * (2.0 / 3.0);
  fc.kap = ph.kappa * ih * ph.iR;
  fc.gh = ph.geff * h;
  if constexpr (CB == 1) { fc.mu = uniform(fc.mu); fc.mu23 = uniform(fc.mu23); fc.kap = uniform(fc.kap); fc.gh = uniform(fc.gh); }
  // background at the node of the time column (row j = hi)
  const double zc = fma(h, gt[GTab::XI * n + hi], z0);
  const double* bg = a.bg + (size_t)cc * 2 * (n + 2);
  const double rbc = bg[2 * hi], pbc = bg[2 * hi + 1];
  const double* Qc = a.Qin + (size_t)cc * sl;
  double* smm = S + L::cell;                           // [n][nn] density wave's source

  double X[n][4];
#pragma unroll
  for (int v = 0; v < 4; ++v) X[0][v] = Qc[v * nn + r];

  // the density wave's energy source at the n time nodes (state-independent)
  if (!PW && ms) {
    WavePhase* lev = reinterpret_cast<WavePhase*>(S);   // of the time levels, from the lanes with hi = 0
    const double xi = gt[GTab::XI * n + lo], tb = xi * dt;
    if (act && hi == 0) lev[lo] = wave_phase(ph, ph.mms_u * tb, ph.mms_w * tb);
    sync();
    if (act) {
      const WavePhase w = wave_phase(ph, fma(-ph.mms_u, t0, fma(h, xi, x0)), fma(-ph.mms_w, t0, zc));
#pragma unroll
      for (int b = 0; b < n; ++b) smm[b * nn + r] = mms_source(ph, w, lev[b]);
    }
    sync();
  }

  // Where there is one level only (first sweep, volume term) the contractions
  // run as line jobs, one lane per (direction, variable, line), on slices
  // [v][j][i]: state at S, x parts at S + sl, z parts at S + 2 sl.
  constexpr bool all = CB == 1 && WV == 1;             // idle lanes take jobs too
  constexpr int JL = all ? kWave : nn;
  const int jl = all ? t : r;

  // first sweep: every level starts from Q^n, one residual serves all
  if (act) {
#pragma unroll
    for (int v = 0; v < 4; ++v) S[v * nn + r] = X[0][v];
  }
  sync();
  if (act || all) {
    const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
#pragma unroll 1
    for (int q = jl; q < 8 * n; q += JL) {
      const int dir = q >= 4 * n, k = q - dir * 4 * n, v = k / n, line = k % n;
      const int base = v * nn + (dir ? line : line * n), st = dir ? n : 1;
      double in[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) in[m] = S[base + m * st];
      D.apply(in, out);
      double* d = S + (1 + dir) * sl + base;
#pragma unroll
      for (int m = 0; m < n; ++m) d[m * st] = out[m];
    }
  }
  sync();
  double R[4] = {0.0, 0.0, 0.0, 0.0};
  if (act) {
    double gx[4], gz[4], Fx[3], Fz[3];
#pragma unroll
    for (int v = 0; v < 4; ++v) { gx[v] = S[sl + v * nn + r]; gz[v] = S[2 * sl + v * nn + r]; }
    fc.gz = ph.geff * zc;
    fc.pb = pbc;
    flux_xz(fc, X[0], gx, gz, Fx, Fz);
    R[0] = gx[1] + gz[2];
    R[2] = X[0][0] - rbc;
#pragma unroll
    for (int v = 1; v < 4; ++v) { S[sl + v * nn + r] = Fx[v - 1]; S[2 * sl + v * nn + r] = Fz[v - 1]; }
  }
  sync();
  if (act || all) {
    const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
#pragma unroll 1
    for (int q = jl; q < 6 * n; q += JL) {
      const int dir = q >= 3 * n, k = q - dir * 3 * n, v = 1 + k / n, line = k % n;
      const int st = dir ? n : 1;
      double* d = S + (1 + dir) * sl + v * nn + (dir ? line : line * n);
      double in[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) in[m] = d[m * st];
      D.apply(in, out);
#pragma unroll
      for (int m = 0; m < n; ++m) d[m * st] = out[m];
    }
  }
  sync();
  if (act) {
#pragma unroll
    for (int v = 1; v < 4; ++v) {
      const double div = S[sl + v * nn + r] + S[2 * sl + v * nn + r];
      R[v] = v == 2 ? fma(fc.gh, R[2], div) : div;   // -h times the gravity source
    }
  }
#pragma unroll
  for (int b = 0; b < n; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) X[b][v] = R[v];
  // background of the lane's row (j = lo)
  const double rbr = bg[2 * lo];
  fc.pb = bg[2 * lo + 1];
  fc.gz = ph.geff * fma(h, gt[GTab::XI * n + lo], z0);
  sync();

  double Qb[4] = {0.0, 0.0, 0.0, 0.0}, Fxa[3] = {0.0, 0.0, 0.0}, Fza[3] = {0.0, 0.0, 0.0};
  if (act) {
#pragma unroll 1
  for (int it = 0;; it = __builtin_amdgcn_readfirstlane(it + 1)) {
    // X holds the scaled residuals R' (time columns): manufactured sources,
    // then X <- Q^n - (dt/h) K1^{-1} W R' by forward and back substitution
    if constexpr (PW) {
      const double x = fma(h, gt[GTab::XI * n + lo], x0);
#pragma unroll
      for (int b = 0; b < n; ++b) {
        double Sm[4];
        paper_wave_source(ph, x, zc, fma(gt[GTab::XI * n + b], dt, t0), Sm);
#pragma unroll
        for (int v = 0; v < 4; ++v) X[b][v] = fma(-h, Sm[v], X[b][v]);
      }
    } else if (ms) {
#pragma unroll
      for (int b = 0; b < n; ++b) X[b][3] = fma(-h, smm[b * nn + r], X[b][3]);
    }
    {
      double qn[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) qn[v] = Qc[v * nn + r];
      const ctab lu = scalar_table(gt + GTab::lu(n));
      int o = 0;
#pragma unroll
      for (int i = 1; i < n; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) {
          const double l = lu[o++];
#pragma unroll
          for (int v = 0; v < 4; ++v) X[i][v] = fma(-l, X[j][v], X[i][v]);
        }
#pragma unroll
      for (int i = n - 1; i >= 0; --i) {
        const double d = lu[o++];
#pragma unroll
        for (int v = 0; v < 4; ++v) X[i][v] *= d;
#pragma unroll
        for (int j = i + 1; j < n; ++j) {
          const double u = lu[o++];
#pragma unroll
          for (int v = 0; v < 4; ++v) X[i][v] = fma(-u, X[j][v], X[i][v]);
        }
      }
      const double sdt = CB == 1 ? uniform(-dt * ih) : -dt * ih;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < n; ++i) X[i][v] = fma(sdt, X[i][v], qn[v]);
    }
    if (a.iter_store && cell < a.C) {
      double* st = a.iter_store + ((size_t)cell * a.iters + it) * n * sl;
#pragma unroll
      for (int b = 0; b < n; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) st[b * sl + v * nn + r] = X[b][v];
    }
    {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int b = 0; b < n; ++b) timp[v * VS + b * BS] = X[b][v];
    }
    if (it == a.iters - 1) break;
    sync();

    // one sweep: rows and columns of every level
    double q[4][n], g[4][n];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int i = 0; i < n; ++i) q[v][i] = rowp[v * VS + i * IS];
    sync();   // every row read before the columns are overwritten
    {
      const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
      derivatives<n, VS, JS, 0>(D, colp, q, g);       // gradients
    }
    sync();
    {
      double gz[4];
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const double qi[4] = {q[0][i], q[1][i], q[2][i], q[3][i]};
        const double gx[4] = {g[0][i], g[1][i], g[2][i], g[3][i]};
        double Fx[3], Fz[3];
#pragma unroll
        for (int v = 0; v < 4; ++v) gz[v] = rowp[v * VS + i * IS];
        flux_xz(fc, qi, gx, gz, Fx, Fz);
        {
          rowp[i * IS] = gx[1] + gz[2];                    // mass residual
#pragma unroll
          for (int v = 1; v < 4; ++v) rowp[v * VS + i * IS] = Fz[v - 1];
        }
#pragma unroll
        for (int v = 1; v < 4; ++v) g[v][i] = Fx[v - 1];
        q[0][i] -= rbr;
        fence_schedule();
      }
    }
    sync();
    {
      const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
      derivatives<n, VS, JS, 1>(D, colp, g, g);       // divergences
    }
    sync();
    {
#pragma unroll
      for (int v = 1; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < n; ++i) rowp[v * VS + i * IS] += v == 2 ? fma(fc.gh, q[0][i], g[v][i]) : g[v][i];
    }
    sync();
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int b = 0; b < n; ++b) X[b][v] = timp[v * VS + b * BS];
    sync();   // every time column read before the next iterate is written
  }

  // time averages on the last iterate (published above; read back, so that
  // no iterate is held in registers across the sweeps)
  sync();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    Qb[v] = 0.0;
#pragma unroll
    for (int b = 0; b < n; ++b) Qb[v] = fma(gt[GTab::W * n + b], timp[v * VS + b * BS], Qb[v]);
  }
  sync();
  {
    double q[4][n], g[4][n];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int i = 0; i < n; ++i) q[v][i] = rowp[v * VS + i * IS];
    sync();   // every row read before the columns are overwritten
    {
      const EO<n> D(scalar_table(gt + GTab::eo_d(n)));
      derivatives<n, VS, JS, 0>(D, colp, q, g);
    }
    sync();
    {
      double gz[4];
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const double qi[4] = {q[0][i], q[1][i], q[2][i], q[3][i]};
        const double gx[4] = {g[0][i], g[1][i], g[2][i], g[3][i]};
        double Fx[3], Fz[3];
#pragma unroll
        for (int v = 0; v < 4; ++v) gz[v] = rowp[v * VS + i * IS];
        flux_xz(fc, qi, gx, gz, Fx, Fz);
        {
#pragma unroll
          for (int v = 1; v < 4; ++v) rowp[v * VS + i * IS] = Fz[v - 1];
        }
#pragma unroll
        for (int v = 1; v < 4; ++v) g[v][i] = Fx[v - 1];
        fence_schedule();
      }
    }
    sync();
    {
#pragma unroll
      for (int v = 1; v < 4; ++v)
#pragma unroll
        for (int b = 0; b < n; ++b) Fza[v - 1] = fma(gt[GTab::W * n + b], timp[v * VS + b * BS], Fza[v - 1]);
    }
    sync();
    {
#pragma unroll
      for (int v = 1; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < n; ++i) rowp[v * VS + i * IS] = g[v][i];
    }
    sync();
    {
#pragma unroll
      for (int v = 1; v < 4; ++v)
#pragma unroll
        for (int b = 0; b < n; ++b) Fxa[v - 1] = fma(gt[GTab::W * n + b], timp[v * VS + b * BS], Fxa[v - 1]);
    }
    sync();
  }

  }

  // face data and volume term from the averaged state and fluxes
  if (act) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      S[v * nn + r] = Qb[v];
      S[sl + v * nn + r] = v == 0 ? Qb[1] : Fxa[v > 0 ? v - 1 : 0];
      S[2 * sl + v * nn + r] = v == 0 ? Qb[2] : Fza[v > 0 ? v - 1 : 0];
    }
  }
  sync();
  if (act || all) {
    const EO<n> W(scalar_table(gt + GTab::eo_dw(n)));
    const ctab e = scalar_table(gt);
#pragma unroll 1
    for (int q = jl; q < 8 * n; q += JL) {
      const int dir = q >= 4 * n, k = q - dir * 4 * n, v = k / n, line = k % n;
      const int base = v * nn + (dir ? line : line * n), st = dir ? n : 1;
      double* d = S + (1 + dir) * sl + base;
      double in[n], out[n], q0 = 0, q1 = 0, f0 = 0, f1 = 0;
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const double e0 = e[GTab::E0 * n + m], e1 = e[GTab::E1 * n + m];
        const double iq = S[base + m * st];
        in[m] = d[m * st];
        q0 = fma(e0, iq, q0); q1 = fma(e1, iq, q1);
        f0 = fma(e0, in[m], f0); f1 = fma(e1, in[m], f1);
      }
      W.apply(in, out);
#pragma unroll
      for (int m = 0; m < n; ++m) d[m * st] = out[m];
      if (cell >= a.C) continue;
      double* fd = a.FD + (size_t)cell * 32 * n;
      const int fl = 2 * dir, fu = 2 * dir + 1;
      fd[((fl * 2 + 0) * 4 + v) * n + line] = q0;
      fd[((fl * 2 + 1) * 4 + v) * n + line] = f0;
      fd[((fu * 2 + 0) * 4 + v) * n + line] = q1;
      fd[((fu * 2 + 1) * 4 + v) * n + line] = f1;
    }
  }
  sync();
  if (valid) {
    double Sb[4] = {0.0, 0.0, -ph.geff * (Qb[0] - bg[2 * hi]), 0.0};
    if (!PW && ms) {
#pragma unroll
      for (int b = 0; b < n; ++b) Sb[3] = fma(gt[GTab::W * n + b], smm[b * nn + r], Sb[3]);
    }
    if constexpr (PW) {
      const double x = fma(h, gt[GTab::XI * n + lo], x0);
#pragma unroll 1
      for (int b = 0; b < n; ++b) {
        double Sm[4];
        paper_wave_source(ph, x, zc, fma(gt[GTab::XI * n + b], dt, t0), Sm);
        const double wb = gt[GTab::W * n + b];
#pragma unroll
        for (int v = 0; v < 4; ++v) Sb[v] = fma(wb, Sm[v], Sb[v]);
      }
    }
    double* qs = a.Qs + (size_t)cell * sl;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      qs[v * nn + r] = fma(dt, fma(S[sl + v * nn + r] + S[2 * sl + v * nn + r], ih, Sb[v]), Qc[v * nn + r]);
  }
}

// Up to n = 7 the kernel is held to 168 VGPRs, three wavefronts per SIMD; at
// n = 8 two.  At n = 7 that spills some 20 of them outside the inner phases:
// meshes of up to 2048 cells, which have no third wavefront for a SIMD, take
// the variant that holds 183.  Two, three per SIMD at n = 7: 30 x 30 cells 31.6
// and 34.7 us, 45 x 45 51.1 and 52.5, 48 x 48 72.8 and 66.2, 243 x 243 1.28 and
// 1.17 ms.
template <int n, int CB, int WV, bool PW, int OCC>
__global__ __launch_bounds__(kWave * WV, OCC) void k_predict_rows(Phys ph, StepArgs a, int ms) {
  extern __shared__ double lds[];
  predict_rows<n, CB, WV, PW>(ph, a, lds, ms, blockIdx.x * CB);
}

template <int n, int CB, int WV, bool PW = false, int OCC = (n <= 7 ? 3 : 2)>
static int rows_t(const Group& g, double* store, hipStream_t s) {
  StepArgs a = make_args(g);
  a.iter_store = store;
  const int ms = g.ph.mms == 1 ? n * n * n : 0;
  const size_t lds = sizeof(double) * (size_t)CB * (RowsLay<n, CB, WV>::cell + ms);
  hipLaunchKernelGGL((k_predict_rows<n, CB, WV, PW, OCC>), dim3((g.C + CB - 1) / CB), dim3(kWave * WV), lds, s, g.ph, a,
                     ms);
  return check_launch("predictor (rows)");
}

// ------------------------------------------------- four wavefronts per cell
// For meshes that leave most SIMDs without a cell: one workgroup of four
// wavefronts per cell, wavefront w working on variable w in the contractions
// and the time solve, and on nodes w and w + 4 of every row in the fluxes.
// The gradients along x meet the fluxes in LDS too (three buffers instead
// of one), and the workgroup synchronises four times per sweep.  The same
// arithmetic per value as predict_rows: the results agree bit for bit.
constexpr int kSplit = 4;
template <int n>
struct SplitLay : RowsLay<n, 1, 1> {
  using L = RowsLay<n, 1, 1>;
  static constexpr int buf = 4 * L::VS;
  static constexpr int cell = 3 * buf;
  static_assert(buf >= 6 * L::nn && buf >= 4 * L::nn + 4 * n, "the density wave's phases fit behind the slices");
};

template <int n, bool PW>
__device__ __forceinline__ void predict_split(const Phys& ph, const StepArgs& a, double* lds, int cell) {
  using L = SplitLay<n>;
  constexpr int nn = L::nn, sl = 4 * nn, BS = L::BS, JS = L::JS, IS = L::IS, VS = L::VS, buf = L::buf;
  // the derivative table: up to n = 5 it stays in scalar registers, beyond it
  // is read again in every phase (kept, it spilled; both measured)
  auto eo_table = [](const double* g) {
    return n <= 5 ? (ctab)(g + GTab::eo_d(n)) : scalar_table(g + GTab::eo_d(n));
  };
  const int t = threadIdx.x, lane = t % kWave;
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  const int h0 = L::grid8 ? lane / 8 : lane / n, l0 = L::grid8 ? lane % 8 : lane % n;
  const bool act = h0 < n && l0 < n;
  const int hi = act ? h0 : 0, lo = act ? l0 : 0;   // (j, i), (b, j) or (b, i)
  const int r = hi * n + lo;
  double* XR = lds;              // iterate
  double* GX = lds + buf;        // gradients, fluxes and divergence along x
  double* GZ = lds + 2 * buf;    // the same along z
  const int rowo = hi * BS + lo * JS, colo = hi * BS + lo * IS, timo = hi * JS + lo * IS;
  const double* gt = a.gtab;
  const int s = a.scen ? a.scen[cell] : 0;
  const double t0 = a.clock[4 * s + 0], dt = a.clock[4 * s + 1];
  const double x0 = a.geom[4 * cell + 0], z0 = a.geom[4 * cell + 1], h = a.geom[4 * cell + 2];
  const double* Qc = a.Qin + (size_t)cell * sl;
  const double qn = Qc[w * nn + r];                 // this wavefront's variable at the time column's node
  const double ih = uniform(1.0 / h);
  FluxC fc;
  fc.gm1 = ph.gm1;
  fc.hgm1 = 0.5 * ph.gm1;
  fc.mu = uniform(ph.mu * ih);
  fc.mu23 = uniform(fc.mu * (2.0 / 3.0));
  fc.kap = uniform(ph.kappa * ih * ph.iR);
  fc.gh = uniform(ph.geff * h);
  const double zc = fma(h, gt[GTab::XI * n + hi], z0);
  // background at the time column's node (row hi) and of the lane's row (lo)
  const double* bg = a.bg + (size_t)cell * 2 * (n + 2);
  const double rbc = bg[2 * hi], pbc = bg[2 * hi + 1], rbr = bg[2 * lo], pbr = bg[2 * lo + 1];
  // manufactured sources of this wavefront's variable at the node's n times
  double Sm[n];
#pragma unroll
  for (int b = 0; b < n; ++b) Sm[b] = 0.0;
  if constexpr (PW) {
    const double x = fma(h, gt[GTab::XI * n + lo], x0);
#pragma unroll
    for (int b = 0; b < n; ++b) {
      double S4[4];
      paper_wave_source(ph, x, zc, fma(gt[GTab::XI * n + b], dt, t0), S4);
      Sm[b] = w == 0 ? S4[0] : w == 1 ? S4[1] : w == 2 ? S4[2] : S4[3];
    }
  }

  // first sweep: one residual serves all levels (slices [v][j][i])
  if (act) XR[w * nn + r] = qn;
  __syncthreads();
  // The density wave's source runs beside the first sweep, on the wavefronts
  // that have no part in it: the phases of the nodes along x and z and those of
  // the levels, through the free end of the buffers, then the levels' sources.
  const bool wave = !PW && ph.mms;
  double *phx = XR + 4 * nn, *phz = GX + 4 * nn, *phl = GZ + 4 * nn;   // [nn][2], [nn][2], [2][n][2]
  auto sources = [&](int b0, int b1) {
    const double xs = phx[2 * r], xc = phx[2 * r + 1], zs = phz[2 * r], zco = phz[2 * r + 1];
#pragma unroll
    for (int b = 0; b < n; ++b)
      if (b >= b0 && b < b1)
        Sm[b] = mms_source(ph, {xs, xc, zs, zco}, {phl[2 * b], phl[2 * b + 1], phl[2 * (n + b)], phl[2 * (n + b) + 1]});
  };
  {
    const EO<n> D(eo_table(gt));
    if (t < 8 * n) {
      const int dir = t >= 4 * n, k = t - dir * 4 * n, v = k / n, line = k % n;
      const int base = v * nn + (dir ? line : line * n), st = dir ? n : 1;
      double in[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) in[m] = XR[base + m * st];
      D.apply(in, out);
      double* d = (dir ? GZ : GX) + base;
#pragma unroll
      for (int m = 0; m < n; ++m) d[m * st] = out[m];
    } else if (wave && w > 0) {
      const int lev = lane & 31;   // w = 3: lanes 0.. the levels along x, 32.. along z
      const double xi = gt[GTab::XI * n + min(lev, n - 1)];
      double ang;
      if (w == 1) ang = ph.mms_kx * fma(-ph.mms_u, t0, fma(h, gt[GTab::XI * n + lo], x0));
      else if (w == 2) ang = ph.mms_kz * fma(-ph.mms_w, t0, zc);
      else ang = lane < 32 ? ph.mms_kx * (ph.mms_u * (xi * dt)) : ph.mms_kz * (ph.mms_w * (xi * dt));
      double sn, cs;
      sincos(ang, &sn, &cs);
      if (w < 3 ? act : lev < n) {
        double* o = w == 1 ? phx + 2 * r : w == 2 ? phz + 2 * r : phl + 2 * ((lane >> 5) * n + lev);
        o[0] = sn;
        o[1] = cs;
      }
    }
    __syncthreads();
    if (w == 0 && act) {
      double q[4], gx[4], gz[4], Fx[3], Fz[3];
#pragma unroll
      for (int v = 0; v < 4; ++v) { q[v] = XR[v * nn + r]; gx[v] = GX[v * nn + r]; gz[v] = GZ[v * nn + r]; }
      fc.gz = ph.geff * zc;
      fc.pb = pbc;
      flux_xz(fc, q, gx, gz, Fx, Fz);
      GX[r] = gx[1] + gz[2];
      GZ[r] = q[0] - rbc;
#pragma unroll
      for (int v = 1; v < 4; ++v) { GX[v * nn + r] = Fx[v - 1]; GZ[v * nn + r] = Fz[v - 1]; }
    } else if (wave && w == 3) {
      sources(0, (n + 1) / 2);
    }
    __syncthreads();
    if (t < 6 * n) {
      const int dir = t >= 3 * n, k = t - dir * 3 * n, v = 1 + k / n, line = k % n;
      const int st = dir ? n : 1;
      double* d = (dir ? GZ : GX) + v * nn + (dir ? line : line * n);
      double in[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) in[m] = d[m * st];
      D.apply(in, out);
#pragma unroll
      for (int m = 0; m < n; ++m) d[m * st] = out[m];
    } else if (wave && w == 3) {
      sources((n + 1) / 2, n);
    }
  }
  __syncthreads();
  double X[n];
  {
    const double div = GX[w * nn + r] + GZ[w * nn + r];
    const double R = w == 0 ? GX[r] : w == 2 ? fma(fc.gh, GZ[r], div) : div;   // -h times the gravity source
#pragma unroll
    for (int b = 0; b < n; ++b) X[b] = R;
  }
  fc.pb = pbr;
  fc.gz = ph.geff * fma(h, gt[GTab::XI * n + lo], z0);

  // gradients of the iterate: this wavefront's variable along x and z
  auto gradients = [&] {
    const EO<n> D(eo_table(gt));
    double in[n], im[n], out[n];
#pragma unroll
    for (int m = 0; m < n; ++m) { in[m] = XR[w * VS + rowo + m * IS]; im[m] = XR[w * VS + colo + m * JS]; }
    D.apply(in, out);
    if (act) {
#pragma unroll
      for (int m = 0; m < n; ++m) GX[w * VS + rowo + m * IS] = out[m];
    }
    D.apply(im, out);
    if (act) {
#pragma unroll
      for (int m = 0; m < n; ++m) GZ[w * VS + colo + m * JS] = out[m];
    }
  };
  // fluxes at this wavefront's nodes, over the gradients; with res the mass
  // residual and the density perturbation go to the free mass slots
  auto fluxes = [&](bool res) {
#pragma unroll
    for (int i = 0; i < n; i += kSplit) {
      if (i + w < n) {
        const int o = rowo + (i + w) * IS;
        double q[4], gx[4], gz[4], Fx[3], Fz[3];
#pragma unroll
        for (int v = 0; v < 4; ++v) { q[v] = XR[v * VS + o]; gx[v] = GX[v * VS + o]; gz[v] = GZ[v * VS + o]; }
        flux_xz(fc, q, gx, gz, Fx, Fz);
        if (act) {
          if (res) {
            GX[o] = gx[1] + gz[2];
            GZ[o] = q[0] - rbr;
          }
#pragma unroll
          for (int v = 1; v < 4; ++v) { GX[v * VS + o] = Fx[v - 1]; GZ[v * VS + o] = Fz[v - 1]; }
        }
      }
    }
  };

#pragma unroll 1
  for (int it = 0;; it = __builtin_amdgcn_readfirstlane(it + 1)) {
    // manufactured source, then the time solve of this wavefront's variable
    if (PW || (ph.mms && w == 3)) {
#pragma unroll
      for (int b = 0; b < n; ++b) X[b] = fma(-h, Sm[b], X[b]);
    }
    {
      const ctab lu = scalar_table(gt + GTab::lu(n));
      int o = 0;
#pragma unroll
      for (int i = 1; i < n; ++i)
#pragma unroll
        for (int j = 0; j < i; ++j) X[i] = fma(-lu[o++], X[j], X[i]);
#pragma unroll
      for (int i = n - 1; i >= 0; --i) {
        X[i] *= lu[o++];
#pragma unroll
        for (int j = i + 1; j < n; ++j) X[i] = fma(-lu[o++], X[j], X[i]);
      }
      const double sdt = uniform(-dt * ih);
#pragma unroll
      for (int i = 0; i < n; ++i) X[i] = fma(sdt, X[i], qn);
    }
    if (act) {
      if (a.iter_store) {
        double* st = a.iter_store + ((size_t)cell * a.iters + it) * n * sl;
#pragma unroll
        for (int b = 0; b < n; ++b) st[b * sl + w * nn + r] = X[b];
      }
#pragma unroll
      for (int b = 0; b < n; ++b) XR[w * VS + timo + b * BS] = X[b];
    }
    __syncthreads();
    gradients();
    __syncthreads();
    if (it == a.iters - 1) break;
    fluxes(true);
    __syncthreads();
    if (w > 0) {
      const EO<n> D(eo_table(gt));
        double in[n], im[n], out[n];
#pragma unroll
      for (int m = 0; m < n; ++m) { in[m] = GX[w * VS + rowo + m * IS]; im[m] = GZ[w * VS + colo + m * JS]; }
      D.apply(in, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) GX[w * VS + rowo + m * IS] = out[m];
      }
      D.apply(im, out);
      if (act) {
#pragma unroll
        for (int m = 0; m < n; ++m) GZ[w * VS + colo + m * JS] = out[m];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < n; ++b) {
      const int o = timo + b * BS;
      if (w == 0) X[b] = GX[o];
      else if (w == 2) X[b] = GZ[2 * VS + o] + fma(fc.gh, GZ[o], GX[2 * VS + o]);
      else X[b] = GZ[w * VS + o] + GX[w * VS + o];
    }
    // (the iterate's buffer, written next, holds no value read here; the
    // gradient buffers, whose mass slots other wavefronts read here, are written
    // after the barrier that publishes the iterate)
  }

  // time averages: of the state and, from the fluxes of the last iterate, of
  // the fluxes of this wavefront's variable
  fluxes(false);
  __syncthreads();
  double Qb = 0.0, Fxa = 0.0, Fza = 0.0;
#pragma unroll
  for (int b = 0; b < n; ++b) {
    const double wb = gt[GTab::W * n + b];
    const int o = w * VS + timo + b * BS;
    Qb = fma(wb, XR[o], Qb);
    Fxa = fma(wb, GX[o], Fxa);
    Fza = fma(wb, GZ[o], Fza);
  }
  __syncthreads();
  // averaged state and fluxes as slices; the mass fluxes are the momenta
  if (act) {
    XR[w * nn + r] = Qb;
    if (w > 0) { GX[w * nn + r] = Fxa; GZ[w * nn + r] = Fza; }
    if (w == 1) GX[r] = Qb;
    if (w == 2) GZ[r] = Qb;
  }
  __syncthreads();
  if (t < 8 * n) {
    const EO<n> W(scalar_table(gt + GTab::eo_dw(n)));
    const ctab e = scalar_table(gt);
    const int dir = t >= 4 * n, k = t - dir * 4 * n, v = k / n, line = k % n;
    const int base = v * nn + (dir ? line : line * n), st = dir ? n : 1;
    double* d = (dir ? GZ : GX) + base;
    double in[n], out[n], q0 = 0, q1 = 0, f0 = 0, f1 = 0;
#pragma unroll
    for (int m = 0; m < n; ++m) {
      const double e0 = e[GTab::E0 * n + m], e1 = e[GTab::E1 * n + m];
      const double iq = XR[base + m * st];
      in[m] = d[m * st];
      q0 = fma(e0, iq, q0); q1 = fma(e1, iq, q1);
      f0 = fma(e0, in[m], f0); f1 = fma(e1, in[m], f1);
    }
    W.apply(in, out);
#pragma unroll
    for (int m = 0; m < n; ++m) d[m * st] = out[m];
    double* fd = a.FD + (size_t)cell * 32 * n;
    const int fl = 2 * dir, fu = 2 * dir + 1;
    fd[((fl * 2 + 0) * 4 + v) * n + line] = q0;
    fd[((fl * 2 + 1) * 4 + v) * n + line] = f0;
    fd[((fu * 2 + 0) * 4 + v) * n + line] = q1;
    fd[((fu * 2 + 1) * 4 + v) * n + line] = f1;
  }
  __syncthreads();
  if (act) {
    double Sb = 0.0;
    if (w == 2) Sb = -ph.geff * (XR[r] - bg[2 * hi]);
    if (PW || (ph.mms && w == 3)) {
#pragma unroll
      for (int b = 0; b < n; ++b) Sb = fma(gt[GTab::W * n + b], Sm[b], Sb);
    }
    a.Qs[(size_t)cell * sl + w * nn + r] = fma(dt, fma(GX[w * nn + r] + GZ[w * nn + r], ih, Sb), qn);
  }
}

template <int n, bool PW>
__global__ __launch_bounds__(kWave * kSplit) void k_predict_split(Phys ph, StepArgs a) {
  extern __shared__ double lds[];
  predict_split<n, PW>(ph, a, lds, blockIdx.x);
}

template <int n>
static int split_n(const Group& g, double* store, hipStream_t s) {
  StepArgs a = make_args(g);
  a.iter_store = store;
  const size_t lds = sizeof(double) * SplitLay<n>::cell;
  if (g.ph.mms == 2)
    hipLaunchKernelGGL((k_predict_split<n, true>), dim3(g.C), dim3(kWave * kSplit), lds, s, g.ph, a);
  else
    hipLaunchKernelGGL((k_predict_split<n, false>), dim3(g.C), dim3(kWave * kSplit), lds, s, g.ph, a);
  return check_launch("predictor (split)");
}
// ----------------------------------------------------------------- dispatch
// Cells of a workgroup of one wavefront: 63 of 64 lanes at n = 3, all at
// n = 2, 4 and 8, 50 at n = 5 (36 and 49 with one cell at n = 6 and 7).
constexpr int wave_cells(int n) { return n == 2 ? 16 : n == 3 ? 7 : n == 4 ? 4 : n == 5 ? 2 : 1; }

// The kernel of a launch.  Measured per predictor launch (us):
//   four wavefronts per cell against one-wavefront workgroups: n = 7,
//     21x21 25.5 / 30.3, 27x27 31.4 / 34.8, 30x30 43.8 / 35.4; n = 6, 27x27
//     24.4 / 24.7, 30x30 28.8 / 24.8; n = 5, 15x15 13.2 / 15.8, 22x22
//     15.0 / 15.1 (16.4 / 17.0 with the density wave's source), 23x23
//     17.4 / 16.1; n = 4, 15x15 9.6 / 11.5, 20x20 10.1 / 10.7, 23x23
//     11.6 / 10.8; n = 3, 20x20 6.9 / 7.7, 27x27 7.9 / 7.7; n = 2, 31x31
//     7.0 / 8.3.  Three such workgroups share a CU at n = 6 and 7: up to 768
//     cells there (one round of the 256 CUs); up to 512 below, 1024 at n = 2.
//   n = 6, one cell per wavefront (36 lanes) against three cells on two
//     (108 of 128): 45x45 39.2 / 39.8, 55x55 53.0 / 44.8, 81x81 110 / 98;
//     seven cells on four (252 of 256) 243x243 674 / 653, as its larger
//     workgroups wait for each other.
//   n = 5, two cells on one wavefront against five on two (125 of 128
//     lanes): 55x55 27.8 / 29.2, 65x65 37.9 / 33.5, 81x81 52 / 45.
//   n = 7, five cells on four wavefronts (245 of 256 lanes) measured 1.44
//     against 1.21 ms at 243x243 (its workgroups leave two wavefronts per
//     SIMD, which wait for each other).
// A launch shape set by the caller chooses among the same kernels; results
// do not depend on the choice.
enum class Kernel { kSplit, kCell, kWave, kPacked };
static Kernel pick(const Group& g) {
  if (g.lv == 1) return Kernel::kSplit;
  if (g.lv == 0) {
    if (g.cpw == 1 && g.wpb == 1) return Kernel::kCell;
    return g.cpw == 1 ? Kernel::kPacked : Kernel::kWave;
  }
  if (g.C <= (g.n >= 6 ? 768 : g.n == 2 ? 1024 : 512)) return Kernel::kSplit;
  if (g.n == 6) return g.C <= 2048 ? Kernel::kCell : Kernel::kPacked;
  if (g.n == 5) return g.C <= 4096 ? Kernel::kWave : Kernel::kPacked;
  return Kernel::kWave;
}

// the launch shape of a group; one that runs the same kernel for a group without
void predictor_shape(const Group& g, int* cpw, int* wpb) {
  const Kernel k = pick(g);
  if (g.lv == 0) { *cpw = g.cpw; *wpb = g.wpb; return; }
  *cpw = k == Kernel::kSplit ? 0 : k == Kernel::kWave ? max_cpw_c(g.n) : 1;
  *wpb = k == Kernel::kPacked ? 2 : 1;
}

template <int n>
static int predict_n(const Group& g, double* store, hipStream_t s) {
  if (g.C == 0) return ADG_OK;
  const Kernel k = pick(g);
  if (k == Kernel::kSplit) return split_n<n>(g, store, s);
  // the paper's manufactured solution runs one cell per wavefront
  if (g.ph.mms == 2) return rows_t<n, 1, 1, true>(g, store, s);
  if constexpr (n == 7) { if (g.C <= 2048) return rows_t<n, 1, 1, false, 2>(g, store, s); }
  if (k == Kernel::kCell) return rows_t<n, 1, 1>(g, store, s);
  if constexpr (n == 5) { if (k == Kernel::kPacked) return rows_t<n, 5, 2>(g, store, s); }
  if constexpr (n == 6) { if (k == Kernel::kPacked) return rows_t<n, 3, 2>(g, store, s); }
  return rows_t<n, wave_cells(n), 1>(g, store, s);
}

int launch_predictor(const Group& g, double* store, hipStream_t s) {
  switch (g.n) {
    case 2: return predict_n<2>(g, store, s);
    case 3: return predict_n<3>(g, store, s);
    case 4: return predict_n<4>(g, store, s);
    case 5: return predict_n<5>(g, store, s);
    case 6: return predict_n<6>(g, store, s);
    case 7: return predict_n<7>(g, store, s);
    case 8: return predict_n<8>(g, store, s);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}

// ------------------------------------------------- persistent batch predictor
// One persistent launch per order group: a grid of resident wavefronts that
// take work items (one wavefront's cells) from the group's device counter
// until none are left, each running predict_rows.
// The last wavefront to finish resets the counter pair for the next launch
// (every wavefront of the grid reaches that point: the loop ends when the
// counter passes the last item).  The batch sizes each order's grid by its
// share of the modelled work, so that the orders, launched side by side,
// finish together.
template <int n>
__global__ __launch_bounds__(kWave, (n <= 7 ? 3 : 2)) void k_predict_queue(Phys ph, StepArgs a, int ms,
                                                                           unsigned* counter, unsigned nwaves) {
  constexpr int CB = wave_cells(n);
  extern __shared__ double lds[];
  const unsigned items = (unsigned)((a.C + CB - 1) / CB);
  for (;;) {
    unsigned item = 0;
    if (threadIdx.x == 0) item = atomicAdd(&counter[0], 1u);
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= items) break;
    // an opaque copy of the buffer pointers per item, so that the body's
    // table and state loads stay inside the loop (hoisted, they would stay
    // live across the whole body)
    StepArgs ai = a;
    asm volatile("" : "+s"(ai.gtab), "+s"(ai.geom), "+s"(ai.Qin), "+s"(ai.clock));
    predict_rows<n, CB, 1, false>(ph, ai, lds, ms, (int)item * CB);
    wave_sync();
  }
  if (threadIdx.x == 0) {
    const unsigned done = atomicAdd(&counter[1], 1u);
    if (done + 1 == nwaves) {
      atomicExch(&counter[0], 0u);
      atomicExch(&counter[1], 0u);
    }
  }
}

template <int n>
static size_t queue_lds(int ms) { return sizeof(double) * (size_t)wave_cells(n) * (RowsLay<n, wave_cells(n), 1>::cell + ms); }

template <int n>
static int queue_n(const Group& g, unsigned* counter, int nwaves, hipStream_t s) {
  const int ms = g.ph.mms == 1 ? n * n * n : 0;
  hipLaunchKernelGGL(k_predict_queue<n>, dim3(nwaves), dim3(kWave), queue_lds<n>(ms), s, g.ph, make_args(g), ms, counter,
                     (unsigned)nwaves);
  return check_launch("persistent predictor");
}

int launch_predictor_queue(const Group& g, unsigned* counter, int nwaves, hipStream_t s) {
  if (g.C == 0 || nwaves < 1) return ADG_OK;
  if (g.ph.mms == 2) return fail(ADG_EUNSUPPORTED, "the persistent batch predictor has no manufactured-solution source");
  switch (g.n) {
    case 2: return queue_n<2>(g, counter, nwaves, s);
    case 3: return queue_n<3>(g, counter, nwaves, s);
    case 4: return queue_n<4>(g, counter, nwaves, s);
    case 5: return queue_n<5>(g, counter, nwaves, s);
    case 6: return queue_n<6>(g, counter, nwaves, s);
    case 7: return queue_n<7>(g, counter, nwaves, s);
    case 8: return queue_n<8>(g, counter, nwaves, s);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}

// resident wavefronts per CU of the persistent predictor of order n-1
template <int n>
static int queue_occ(int* per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_predict_queue<n>, kWave, queue_lds<n>(0)) == hipSuccess
             ? ADG_OK
             : fail(ADG_EHIP, "occupancy query failed");
}
int predictor_queue_occupancy(int n, int* per_cu) {
  switch (n) {
    case 2: return queue_occ<2>(per_cu);
    case 3: return queue_occ<3>(per_cu);
    case 4: return queue_occ<4>(per_cu);
    case 5: return queue_occ<5>(per_cu);
    case 6: return queue_occ<6>(per_cu);
    case 7: return queue_occ<7>(per_cu);
    case 8: return queue_occ<8>(per_cu);
    default: return fail(ADG_EUNSUPPORTED, "order not supported");
  }
}

}  // namespace adg
