// Internal definitions of the gfx950 ADER-DG library: constant tables,
// physics parameters in kernel-argument form, the mesh handle, and the
// pointwise physics as device functions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <unordered_map>
#include <vector>

#include "adg.h"

namespace adg {

constexpr int kMaxN = 8;          // nodes per direction supported (order 7)
constexpr int kWave = 64;         // CDNA wavefront size

// Basis tables for n nodes, passed by value as a kernel argument so that every
// entry read with a compile-time index becomes a scalar (SGPR) operand.
template <int n>
struct Tab {
  double D[n][n];    // D[i][m] = phi_m'(xi_i)
  double P[n][n];    // time predictor matrix K1^{-1} W
  double Dw[n][n];   // volume term: Dw[i][m] = w_m D[m][i] / w_i
  double w[n];
  double e0[n], e1[n];
};

// Tables in global memory (one per handle), read with lane-dependent or
// runtime indices:
//   xi[n], w[n], L0[n] = e0/w, L1[n] = e1/w, e0[n], e1[n],
//   Pk[3][n][n]  sub-face k prolongation phi_m((k+xi_q)/3) at [k][q][m],
//   Rk[3][n][n]  restriction (w_q/3) phi_m((k+xi_q)/3)/w_m at [k][m][q],
//   D[n][n], Pt[n][n] (time matrix transposed: Pt[b][a] = P[a][b]), Dw[n][n],
//   even-odd forms of D and Dw (see EvenOdd below),
//   LU[n*n]: the time matrix K1 = L U (unit lower L, no pivoting: for
//   Gauss-Legendre nodes the factors stay bounded, |U_ii| >= 1 up to n = 8)
//   stored in the order the in-place solve of K1 y = W r reads it, with the
//   weights moved into the factors (the forward substitution works on
//   z_i / w_i): for each row i > 0, L[i][j] w_j / w_i for j < i; then for each
//   row i from n-1 down to 0, w_i / U_ii then U[i][i+1..n-1] / U_ii.
struct GTab {
  static constexpr int XI = 0, W = 1, L0 = 2, L1 = 3, E0 = 4, E1 = 5;
  static __host__ __device__ inline int pk(int n) { return 6 * n; }
  static __host__ __device__ inline int rk(int n) { return 6 * n + 3 * n * n; }
  static __host__ __device__ inline int d(int n) { return 6 * n + 6 * n * n; }
  static __host__ __device__ inline int pt(int n) { return 6 * n + 7 * n * n; }
  static __host__ __device__ inline int dw(int n) { return 6 * n + 8 * n * n; }
  static __host__ __device__ inline int eo_size(int n) { return 2 * (n / 2) * (n / 2) + 2 * (n / 2); }
  static __host__ __device__ inline int eo_d(int n) { return 6 * n + 9 * n * n; }
  static __host__ __device__ inline int eo_dw(int n) { return 6 * n + 9 * n * n + eo_size(n); }
  static __host__ __device__ inline int lu(int n) { return 6 * n + 9 * n * n + 2 * eo_size(n); }
  static __host__ __device__ inline int size(int n) { return 6 * n + 10 * n * n + 2 * eo_size(n); }
};

// Even-odd form of an n x n matrix T with T[n-1-i][n-1-m] = -T[i][m] (the
// Gauss-Legendre derivative matrix and the volume matrix are centro-
// antisymmetric), h = n/2, mid = (n-1)/2 for odd n:
//   A[i][m] = (T[i][m] - T[i][n-1-m]) / 2,  B[i][m] = (T[i][m] + T[i][n-1-m]) / 2
//   (i, m < h), C[i] = T[i][mid], M[m] = T[mid][m] (odd n only).
// With e_m = x_m + x_{n-1-m}, o_m = x_m - x_{n-1-m}: S_i = sum_m A[i][m] o_m,
// T_i = sum_m B[i][m] e_m + C[i] x_mid, (T x)_i = S_i + T_i,
// (T x)_{n-1-i} = S_i - T_i, (T x)_mid = sum_m M[m] o_m.  Stored as
// A[h][h], B[h][h], C[h], M[h].

struct Phys {
  double gamma, gm1, R, iR, cp, Pr, mu, kappa, g, p0, theta;
  double cp_over_R, R_over_cp, ex_coef;   // ex_coef = g/(cp theta)
  double lv_coef;                         // lambda_v = lv_coef / rho
  double mms_amp, mms_u, mms_w, mms_kx, mms_kz, mms_p;
  double cfl;
  double geff;                            // g with gravity on, 0 otherwise
  int gravity, mms, fixed_dt, N;
};

enum FaceKind { kConforming = 0, kWall = 1, kFineSide = 2, kCoarseSide = 3 };

// Everything a kernel launch needs for one set of cells of one order: the
// cells of one mesh, or of all scenarios of one order in a batch.
struct Group {
  int n = 0, N = 0, iters = 0, C = 0;
  Phys ph{};
  // handle-owned device tables
  double* d_geom = nullptr;   // [C][4] x0, z0, h, 0; the background table behind it
  double* d_bg = nullptr;     // [C][n + 2][2] background density and pressure: node rows, bottom, top
  int* d_nbr = nullptr;       // [C][4 faces][4] kind, a, b, c (cell indices local to the group)
  double* d_gtab = nullptr;   // GTab layout
  int* d_scen = nullptr;      // [C] scenario index into clock (NULL: all 0)
  // caller-owned buffers bound by set_state
  double* Q = nullptr;        // [C][4][n][n]
  double* Qs = nullptr;       // [C][4][n][n]
  double* FD = nullptr;       // [C][4][2][4][n]
  double* dtc = nullptr;      // [C]
  double* dtmin = nullptr;    // chunk minima of dtc, or NULL (reduced in one stage)
  double* clock = nullptr;    // [S][4]
  // launch shape: cells per wavefront, wavefronts per workgroup
  int cpw = 1, wpb = 1;
  // predictor kernel: -1 automatic (by order and cells, pick() in
  // predict.hip), 0 chosen by the launch shape, 1 four wavefronts per cell
  int lv = -1;
  // handle-owned scratch of the TV statistics over many cells: per-workgroup
  // partials (count, mean, M2) and the thresholds (kTvPartDoubles doubles)
  double* d_part = nullptr;
  // corrector launches: a clock the corrector advances itself (frozen time
  // step, one mesh), or NULL
  double* advance = nullptr;
  int nc = 0;                 // the mesh has 1:3 non-conforming faces
};

// TV statistics over many cells: at most kStatParts per-workgroup partials
constexpr int kStatParts = 512;
// The minimum of more than kOneStage time-step candidates is taken in two
// stages: of kChunks chunks, whose minima go to the end of the workspace, then of
// those.  The section's doubles for C candidates:
constexpr int kChunks = 256, kOneStage = 24576;
constexpr size_t chunk_minima(size_t C) { return C > kOneStage ? kChunks : 0; }
constexpr int kTvPartDoubles = 3 * kStatParts + 3;

// Host copies of the basis of one order.
struct HostBasis {
  int n = 0;
  std::vector<double> xi, w, D, P, Dw, e0, e1, gtab;
};

// Leaves by (level, i, j) on a mesh of nx x nz coarse cells with levels
// 0..L: one dense table per level while the boxes of all levels number at
// most kDenseBoxes (16 MB of ints), else a hash map keyed by the same box
// number (unique: nx * nz <= 2^26 coarse cells and L <= 8 give fewer than
// 2^62 boxes).  Lookups outside the grid of their level find nothing.
struct LeafIndex {
  static constexpr long long kDenseBoxes = 1LL << 22;
  struct Level { long long nx, nz, off; };   // boxes along x and z, start of the level's table
  int L;
  bool dense = false;
  std::vector<Level> lev;
  std::vector<int> tab;
  std::unordered_map<long long, int> map;
  LeafIndex(int nx, int nz, int L_, size_t n_leaves) : L(L_), lev(L_ + 1) {
    long long total = 0, s = 1;
    for (int l = 0; l <= L; ++l, s *= 3) {
      lev[l] = {nx * s, nz * s, total};
      total += lev[l].nx * lev[l].nz;
    }
    dense = total <= kDenseBoxes;
    if (dense) tab.assign((size_t)total, -1);
    else map.reserve(n_leaves * 2);
  }
  bool in_grid(int l, int i, int j) const {
    return l >= 0 && l <= L && i >= 0 && j >= 0 && i < lev[l].nx && j < lev[l].nz;
  }
  long long slot(int l, int i, int j) const { return lev[l].off + (long long)j * lev[l].nx + i; }
  // records leaf c at (l, i, j); false if the box is outside the grid or
  // holds a leaf already
  bool insert(int l, int i, int j, int c) {
    if (!in_grid(l, i, j)) return false;
    if (!dense) return map.emplace(slot(l, i, j), c).second;
    int& t = tab[(size_t)slot(l, i, j)];
    if (t >= 0) return false;
    t = c;
    return true;
  }
  int find(int l, int i, int j) const {
    if (!in_grid(l, i, j)) return -1;
    if (!dense) {
      auto it = map.find(slot(l, i, j));
      return it == map.end() ? -1 : it->second;
    }
    return tab[(size_t)slot(l, i, j)];
  }
};

// Host mesh: leaves, geometry and face table.
struct HostMesh {
  int C = 0;
  std::vector<int> lev, ci, cj;
  std::vector<double> geom;   // [C][4]
  std::vector<int> nbr;       // [C][16]
};

}  // namespace adg

struct adg_mesh {
  adg_params prm;
  // device the handle's tables live on, and that device's static scratch
  // (device address, resolved at init; NULL if the lookup failed)
  int dev = 0;
  void* static_scratch = nullptr;
  int static_scratch_rc = 0;
  adg_mesh_desc desc{};
  adg::HostBasis basis;
  adg::HostMesh hm;
  adg::Group g;
  // bound (caller-owned)
  double* Q = nullptr;
  void* ws = nullptr;
  double* clock = nullptr;
  // workspace partition (byte offsets)
  size_t off_qs = 0, off_fd = 0, off_dtc = 0, off_health = 0, off_min = 0, ws_bytes = 0;
  // pending regrid (from adg_regrid_plan): new leaves, transfer operations
  // and the new mesh tables
  bool plan_ready = false;
  std::vector<int> plan_lev, plan_ci, plan_cj, plan_ops;
  adg::HostMesh plan_mesh;
  // grow-only device buffers of the regrid: transfer operations (ints) and
  // the capacity, in cells, of the geometry and neighbour tables
  int* d_ops = nullptr;
  size_t ops_cap = 0;
  int cells_cap = 0;
  // pinned host staging of the regrid's uploads (grow-only, bytes)
  void* h_stage = nullptr;
  size_t stage_cap = 0;
};

namespace adg {

void set_error(const std::string& msg);
int fail(int code, const std::string& msg);
int check_launch(const char* what);

// Gauss-Legendre basis of n nodes and its device tables (computed in long
// double, stored in double).
void build_basis(int n, HostBasis& B);
// persistent predictor of one order group (predict_rows on work items
// from counter [2], nwaves resident wavefronts), and its resident
// wavefronts per CU
int launch_predictor_queue(const Group& g, unsigned* counter, int nwaves, hipStream_t s);
int predictor_queue_occupancy(int n, int* per_cu);
// device address of the allocation-free step's static scratch on device dev
// (the current device); looked up once per device
int static_scratch_address(int dev, void** ptr);
// parameter checks shared by the 2D and 3D handles
int validate_params(const adg_params* p);
Phys make_phys(const adg_params& p);

template <int n>
inline Tab<n> tab_of(const HostBasis& B) {
  Tab<n> T;
  for (int i = 0; i < n; ++i) {
    T.w[i] = B.w[i]; T.e0[i] = B.e0[i]; T.e1[i] = B.e1[i];
    for (int j = 0; j < n; ++j) {
      T.D[i][j] = B.D[i * n + j]; T.P[i][j] = B.P[i * n + j]; T.Dw[i][j] = B.Dw[i * n + j];
    }
  }
  return T;
}

// wavefront-scope barrier for LDS hand-offs between lanes of one wavefront:
// LDS operations of a wavefront execute in order, so a compiler fence and a
// wave barrier are enough.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- physics
// Hydrostatic background of constant potential temperature:
// Exner pi = 1 - g z/(cp theta), p = p0 pi^(cp/R), rho = p/(R theta pi).
__device__ inline void background(const Phys& ph, double z, double& rb, double& pb) {
  if (!ph.gravity) { rb = 0.0; pb = 0.0; return; }
  double pi = 1.0 - ph.ex_coef * z;
  pb = ph.p0 * pow(pi, ph.cp_over_R);
  rb = pb / (ph.R * ph.theta * pi);
}

__device__ inline double pressure(const Phys& ph, double rho, double mx, double mz, double E, double z) {
  const double geo = rho * (ph.geff * z);   // 0 without gravity
  return ph.gm1 * (E - 0.5 * (mx * mx + mz * mz) / rho - geo);
}

// Reciprocal of a positive normal double: the hardware estimate refined by
// two Newton steps r <- r + r (1 - x r) (quadratic convergence; the result
// is within an ulp or so of 1/x, not necessarily correctly rounded).
__device__ inline double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// Phases of the manufactured advected density wave, kx (x - u t) and
// kz (z - w t): sine and cosine along x, then along z.
struct WavePhase {
  double sx, cx, sz, cz;
};
__device__ inline WavePhase wave_phase(const Phys& ph, double X, double Z) {
  WavePhase p;
  sincos(ph.mms_kx * X, &p.sx, &p.cx);
  sincos(ph.mms_kz * Z, &p.sz, &p.cz);
  return p;
}
// Energy source of the wave (T = p/(R rho), S_E = -kappa Lap T) at a point with
// phases a, a time later in which the phases decrease by b: n time levels cost
// one pair of sines for the point and one for each level of a cell, not two
// for each of the cell's n^3 nodes in space and time.
__device__ inline double mms_source(const Phys& ph, const WavePhase& a, const WavePhase& b) {
  const double sx = fma(a.sx, b.cx, -(a.cx * b.sx)), cx = fma(a.cx, b.cx, a.sx * b.sx);
  const double sz = fma(a.sz, b.cz, -(a.cz * b.sz)), cz = fma(a.cz, b.cz, a.sz * b.sz);
  double rho = fma(ph.mms_amp * sx, sz, 1.0);
  double rx = ph.mms_amp * ph.mms_kx * cx * sz;
  double rz = ph.mms_amp * ph.mms_kz * sx * cz;
  double lap = -fma(ph.mms_kx, ph.mms_kx, ph.mms_kz * ph.mms_kz) * ph.mms_amp * sx * sz;
  double ir = recip(rho);
  double lapT = ph.mms_p * ph.iR * fma(-lap * ir, ir, 2.0 * fma(rx, rx, rz * rz) * ir * ir * ir);
  return -ph.kappa * lapT;
}

// The paper's manufactured solution (CFD scenarios, eq.
// manufactured-solution): with phase xi = k (x + z) - om t, k = pi/5,
// om = 2 pi, the fields rho = 1 + sin(xi)/2, p = 1/gamma + cos(xi)/10,
// u = w = sin(xi)/4 depend on xi alone; d/dx = d/dz = k d/dxi and
// d/dt = -om d/dxi.
constexpr double kWaveK = 0.62831853071795864769;   // pi / 5
constexpr double kWaveOm = 6.28318530717958647693;  // 2 pi
__device__ inline void paper_wave_state(const Phys& ph, double x, double z, double t, double q[4]) {
  double sn, cs;
  sincos(kWaveK * (x + z) - kWaveOm * t, &sn, &cs);
  const double rho = 1.0 + 0.5 * sn, p = 1.0 / ph.gamma + 0.1 * cs, u = 0.25 * sn;
  q[0] = rho; q[1] = rho * u; q[2] = rho * u;
  q[3] = p / ph.gm1 + rho * u * u;
}
// Source that makes the wave solve the equation set without gravity,
// S = dQ/dt + div F, from the derivatives of the fields along xi (primes):
// the stress tensor gives sigma_xx = sigma_zz = -(2/3) mu k u',
// sigma_xz = -2 mu k u'; the heat flux -kappa k T' with T = p/(R rho), whose
// second derivative follows from differentiating R rho T = p twice.  (Fused
// operations spelt out: the predictors that call it agree bit for bit.)
__device__ inline void paper_wave_source(const Phys& ph, double x, double z, double t, double S[4]) {
  constexpr double k = kWaveK, om = kWaveOm;
  double sn, cs;
  sincos(fma(k, x + z, -(om * t)), &sn, &cs);
  const double rho = fma(0.5, sn, 1.0), r1 = 0.5 * cs, r2 = -0.5 * sn;
  const double p = fma(0.1, cs, 1.0 / ph.gamma), p1 = -0.1 * sn;
  const double u = 0.25 * sn, u1 = 0.25 * cs, u2 = -0.25 * sn;
  const double ir = 1.0 / rho;
  const double m1 = fma(r1, u, rho * u1);              // (rho u)'
  const double h1 = fma(r1, u, 2.0 * rho * u1);        // (rho u^2)' / u
  const double E = fma(rho * u, u, p / ph.gm1), E1 = fma(u, h1, p1 / ph.gm1);
  const double H1 = fma(u1, E + p, u * fma(-0.1, sn, E1));   // (u (E + p))', p' = -sin(xi)/10
  const double T = p * ir * ph.iR;
  const double T1 = fma(p1, ph.iR, -(r1 * T)) * ir;
  const double T2 = fma(-2.0 * r1, T1, fma(-0.1 * cs, ph.iR, -(r2 * T))) * ir;
  const double kk = k * k;
  S[0] = fma(2.0 * k, m1, -(om * r1));
  S[1] = fma((-8.0 / 3.0) * ph.mu * kk, u2, fma(k, fma(2.0 * u, h1, p1), -(om * m1)));
  S[2] = S[1];
  S[3] = fma(-2.0 * ph.kappa * kk, T2,
             fma((-16.0 / 3.0) * ph.mu * kk, fma(u1, u1, u * u2), fma(2.0 * k, H1, -(om * E1))));
}

// Square root, correctly rounded.  Goldschmidt's coupled iteration for the root
// g and the half reciprocal h from the hardware estimate of 1/sqrt(x), then two
// Newton corrections of g with the residual x - g^2 formed by one fused
// multiply-add (Markstein, Computation of elementary functions on the IBM RISC
// System/6000 processor, 1990).  Below 2^-767 that residual would lose bits to
// underflow: those numbers, negative ones, infinity and NaN (by one comparison
// of the high word) take the library's root, which scales its argument.  12
// instructions and a branch that wavefronts of ordinary states jump over,
// instead of 20.
__device__ inline double root(double x) {
  constexpr unsigned lo = 0x10000000u, inf = 0x7ff00000u;   // high words of 2^-767 and infinity
  if ((unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) - lo >= inf - lo) return sqrt(x);
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return fma(fma(-g, g, x), h, g);
}

// Lane exchange within rows of 16 lanes through the data-parallel primitives
// (no LDS round trip).
template <int ctrl>
__device__ inline double dpp(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ inline double lane_value(double v, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// max over groups of 4 lanes, of 16 lanes, and over the wavefront: lane xor 1
// and 2 (quad permutations), mirrors within 8 and 16 lanes, then the four rows
__device__ inline double quad_max(double v) {
  v = fmax(v, dpp<0xB1>(v));
  return fmax(v, dpp<0x4E>(v));
}
__device__ inline double row_max(double v) {
  v = quad_max(v);
  v = fmax(v, dpp<0x141>(v));
  return fmax(v, dpp<0x140>(v));
}
__device__ inline double wave_max(double v) {
  v = row_max(v);
  return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

}  // namespace adg
