// Jacobian and residual assembly on the GPU.
//
// Residual of component c in cell i (eqs. (3)/(5) with backward Euler,
// eq. (10), and TPFA fluxes, eq. (11)):
//   R_c,i = [ V (acc_c(x) - acc_c(x_old)) / dt + sum_faces F_c,ij - q_c,i ] / s_c
// with F_c,ij = T_ij lam_c,up (Phi_i - Phi_j) the mass flow from i to j,
// Phi = p - rho g z (z depth), upstream = higher potential (ties, within
// 1e-9 bar, go to the lower-index cell of the face), face density the mean
// of the two cells, and q from eq. (6) (Peaceman index, BHP constraint).
// s_c = rho_c V mean(phi) / dt.  The output right-hand side is -R.
//
// Two kernels: a cell-centric kernel in which every cell evaluates its fluid
// state (phase densities and mobilities with their derivatives) and its faces
// and writes its whole block row (no atomics: the face flow is computed
// identically from both sides); and a per-perforation well kernel.  Built
// without FP contraction so that both sides of a face round identically.
#include <cmath>

#include "internal.h"

namespace {

constexpr double G_ACC = 9.80665;
constexpr double BAR = 1.0e5;
constexpr double CP = 1.0e-3;
constexpr double DAY = 86400.0;
constexpr double TIE_BAR = 1.0e-9;

template <int MODEL>
struct Traits;
template <>
struct Traits<1> {   // single-phase (water) test model
  static constexpr int B = 1, NP = 1, NT = 1;
  __host__ __device__ static constexpr int row(int) { return 0; }
  __host__ __device__ static constexpr int phase(int) { return 0; }
  __host__ __device__ static constexpr bool dep(int, int) { return true; }
};
template <>
struct Traits<2> {
  static constexpr int B = 2, NP = 2, NT = 2;
  __host__ __device__ static constexpr int row(int t) { return t; }
  __host__ __device__ static constexpr int phase(int t) { return t; }
  __host__ __device__ static constexpr bool dep(int, int) { return true; }
};
template <>
struct Traits<3> {
  static constexpr int B = 3, NP = 3, NT = 4;
  // terms: oil comp. in oil phase, water, dissolved gas in oil phase, free gas
  __host__ __device__ static constexpr int row(int t) { return t == 3 ? 2 : t; }
  __host__ __device__ static constexpr int phase(int t) { return t == 2 ? 0 : (t == 3 ? 2 : t); }
  // water does not depend on the third unknown, free gas not on S_w
  __host__ __device__ static constexpr bool dep(int t, int u) { return !(t == 1 && u == 2) && !(t == 3 && u == 1); }
};
static_assert(Traits<3>::phase(0) == 0 && Traits<3>::phase(1) == 1 && Traits<3>::phase(2) == 0 &&
                  Traits<3>::phase(3) == 2 && Traits<3>::row(2) == 2 && Traits<3>::row(3) == 2,
              "black-oil term table");

template <int MODEL>
struct CellState {
  static constexpr int B = Traits<MODEL>::B, NP = Traits<MODEL>::NP, NT = Traits<MODEL>::NT;
  double acc[B], dacc[B][B];
  double rho[NP], drho[NP];
  double drho_o2 = 0.0;   // black oil: d rho_oil-phase / d x2 (undersaturated cells)
  double lam[NT], dlam[NT][B];
  double lt, dlt[B];
};

double pvt_eval(const FluidDev& f, int row, double p) {
  int seg = -1;
  for (int q = 0; q < f.npvt; ++q) seg += f.pvt[0][q] <= p ? 1 : 0;
  seg = seg < 0 ? 0 : (seg > f.npvt - 2 ? f.npvt - 2 : seg);
  return f.pvt[row][seg] + f.slope[row][seg] * (p - f.pvt[0][seg]);
}

// x / s given rs = RN(1 / s): two residual corrections of x rs, the second
// of which rounds correctly (Markstein, IBM J. Res. Dev. 34, 1990) for every
// quotient in the normal range, and the hardware's fix-up of the special ones
// (zeros, infinities: a residual would be inf - inf or 0 inf); six operations
// instead of the dozen of a division, for the many quotients by the same few
// denominators.
__device__ inline double div_by(double x, double s, double rs) {
  double q = x * rs;
  q = __builtin_fma(__builtin_fma(-q, s, x), rs, q);
  q = __builtin_fma(__builtin_fma(-q, s, x), rs, q);
  return __builtin_amdgcn_div_fixup(q, s, x);
}

// The PVT table in LDS: nodes, then value and slope of each row's segments
// (a lane's segment is its own, so the look-ups are not scalar loads).
struct PvtLds {
  double p[CPR_MAX_PVT];
  double2 row[6][CPR_MAX_PVT];

  __device__ void load(const FluidDev& f) {
    for (int q = threadIdx.x; q < 6 * CPR_MAX_PVT; q += blockDim.x)
      row[q / CPR_MAX_PVT][q % CPR_MAX_PVT] =
          make_double2(f.pvt[q / CPR_MAX_PVT][q % CPR_MAX_PVT], f.slope[q / CPR_MAX_PVT][q % CPR_MAX_PVT]);
    for (int q = threadIdx.x; q < CPR_MAX_PVT; q += blockDim.x) p[q] = f.pvt[0][q];
  }
  // right-hand segment at a node, end segments extended
  __device__ int segment(const FluidDev& f, double at) const {
    int seg = -1;
    for (int q = 0; q < f.npvt; ++q) seg += f.pvt[0][q] <= at ? 1 : 0;
    return seg < 0 ? 0 : (seg > f.npvt - 2 ? f.npvt - 2 : seg);
  }
  __device__ double value(int r, int seg, double at, double& slope) const {
    const double2 v = row[r][seg];
    slope = v.y;
    return v.x + slope * (at - p[seg]);
  }
};

__device__ inline void clip01(double a, double& v, double& inside) {
  inside = (a > 0.0 && a < 1.0) ? 1.0 : 0.0;
  v = a < 0.0 ? 0.0 : (a > 1.0 ? 1.0 : a);
}

__device__ inline void corey(double sw, double swc, double sor, double& krw, double& dkrw,
                             double& kro, double& dkro) {
  const double den = 1.0 - swc - sor, rden = 1.0 / den;
  double a, ia, o, io;
  clip01(div_by(sw - swc, den, rden), a, ia);
  clip01(div_by(1.0 - sor - sw, den, rden), o, io);
  krw = a * a;
  dkrw = div_by(2.0 * a * ia, den, rden);
  kro = o * o;
  dkro = div_by(-2.0 * o * io, den, rden);
}

template <int MODEL>
__device__ inline void cell_state(const FluidDev& f, const PvtLds& pvt, double poro, const double* xv,
                                  CellState<MODEL>& s) {
  double p = xv[0];
  double pref = f.p_ref;
  double phi = poro * (1.0 + f.c_r * (p - pref));
  double dphi = poro * f.c_r;
  double rho_w = f.rho_w_ref * exp(f.c_w * (p - pref));
  double drho_w = f.c_w * rho_w;
  double mu_w = f.mu_w * CP;
  if constexpr (MODEL == 1) {
    s.acc[0] = phi * rho_w;
    s.dacc[0][0] = dphi * rho_w + phi * drho_w;
    s.rho[0] = rho_w; s.drho[0] = drho_w;
    s.lam[0] = rho_w / mu_w;
    s.dlam[0][0] = drho_w / mu_w;
    s.lt = 1.0 / mu_w;
    s.dlt[0] = 0.0;
  } else if constexpr (MODEL == 2) {
    double sw = xv[1];
    double so = 1.0 - sw;
    double rho_o = f.rho_o_ref * exp(f.c_o * (p - pref));
    double drho_o = f.c_o * rho_o;
    double mu_o = f.mu_o * CP;
    double krw, dkrw, kro, dkro;
    corey(sw, f.s_wc, f.s_or, krw, dkrw, kro, dkro);
    s.acc[0] = phi * so * rho_o;
    s.acc[1] = phi * sw * rho_w;
    s.dacc[0][0] = so * (dphi * rho_o + phi * drho_o);
    s.dacc[0][1] = -phi * rho_o;
    s.dacc[1][0] = sw * (dphi * rho_w + phi * drho_w);
    s.dacc[1][1] = phi * rho_w;
    s.rho[0] = rho_o; s.drho[0] = drho_o;
    s.rho[1] = rho_w; s.drho[1] = drho_w;
    const double rmo = 1.0 / mu_o, rmw = 1.0 / mu_w;
    s.lam[0] = div_by(rho_o * kro, mu_o, rmo);
    s.dlam[0][0] = div_by(drho_o * kro, mu_o, rmo);
    s.dlam[0][1] = div_by(rho_o * dkro, mu_o, rmo);
    s.lam[1] = div_by(rho_w * krw, mu_w, rmw);
    s.dlam[1][0] = div_by(drho_w * krw, mu_w, rmw);
    s.dlam[1][1] = div_by(rho_w * dkrw, mu_w, rmw);
    s.lt = div_by(krw, mu_w, rmw) + div_by(kro, mu_o, rmo);
    s.dlt[0] = 0.0;
    s.dlt[1] = dkrw / mu_w + dkro / mu_o;
  } else {
    // third unknown: S_g >= 0 (saturated), -p_b < 0 (undersaturated: no free
    // gas, Rs and mu_o at p_b, B_o = B_o(p_b) exp(-c_o (p - p_b)))
    double sw = xv[1], x2 = xv[2];
    const bool sat = x2 >= 0.0;
    double sg = sat ? x2 : 0.0;
    double dsg = sat ? 1.0 : 0.0;
    double pb = sat ? p : -x2;
    double so = 1.0 - sw - sg;
    double drs_b, dbo_b, dmuo_b, dbg, dmug;
    const int sb = pvt.segment(f, pb), sp = pvt.segment(f, p);
    double rs = pvt.value(1, sb, pb, drs_b);
    double bo_b = pvt.value(2, sb, pb, dbo_b);
    double muo = pvt.value(3, sb, pb, dmuo_b);
    double bg = pvt.value(4, sp, p, dbg);
    double mug = pvt.value(5, sp, p, dmug);
    double e = sat ? 1.0 : exp(-f.c_o * (p - pb));
    double bo = bo_b * e;
    double rs_p = sat ? drs_b : 0.0, rs_2 = sat ? 0.0 : -drs_b;
    double bo_p = sat ? dbo_b : -f.c_o * bo;
    double bo_2 = sat ? 0.0 : -(dbo_b * e + f.c_o * bo);
    double mu_p = sat ? dmuo_b : 0.0, mu_2 = sat ? 0.0 : -dmuo_b;
    muo *= CP; mu_p *= CP; mu_2 *= CP; mug *= CP; dmug *= CP;
    double rsc_o = f.rho_o_sc, rsc_g = f.rho_g_sc;
    const double bo2 = bo * bo, rbo = 1.0 / bo, rbo2 = 1.0 / bo2, bg2 = bg * bg;
    double rho_oo = div_by(rsc_o, bo, rbo);
    double rho_oo_p = div_by(-rsc_o * bo_p, bo2, rbo2);
    double rho_oo_2 = div_by(-rsc_o * bo_2, bo2, rbo2);
    double rho_og = div_by(rsc_g * rs, bo, rbo);
    double rho_og_p = div_by(rsc_g * (rs_p * bo - rs * bo_p), bo2, rbo2);
    double rho_og_2 = div_by(rsc_g * (rs_2 * bo - rs * bo_2), bo2, rbo2);
    double rho_g = rsc_g / bg;
    double drho_g = -rsc_g * dbg / bg2;
    // relative permeabilities: Corey water / oil-water, quadratic gas, Stone II oil
    double krw, dkrw, krow, dkrow;
    corey(sw, f.s_wc, f.s_or, krw, dkrw, krow, dkrow);
    double g, ig, h, ih;
    const double rsg = 1.0 / f.sg_den;
    clip01(div_by(sg, f.sg_den, rsg), g, ig);
    clip01(div_by(f.sg_den - sg, f.sg_den, rsg), h, ih);
    double krg = g * g, dkrg = div_by(2.0 * g * ig, f.sg_den, rsg);
    double krog = h * h, dkrog = div_by(-2.0 * h * ih, f.sg_den, rsg);
    double raw = (krow + krw) * (krog + krg) - krw - krg;
    bool pos = raw > 0.0;
    double kro = pos ? raw : 0.0;
    double dkro_w = pos ? (dkrow + dkrw) * (krog + krg) - dkrw : 0.0;
    double dkro_g = pos ? (krow + krw) * (dkrog + dkrg) - dkrg : 0.0;
    dkrg *= dsg;      // per unit of x2
    dkro_g *= dsg;
    s.acc[0] = phi * so * rho_oo;
    s.acc[1] = phi * sw * rho_w;
    s.acc[2] = phi * (so * rho_og + sg * rho_g);
    s.dacc[0][0] = so * (dphi * rho_oo + phi * rho_oo_p);
    s.dacc[0][1] = -phi * rho_oo;
    s.dacc[0][2] = -phi * rho_oo * dsg + phi * so * rho_oo_2;
    s.dacc[1][0] = sw * (dphi * rho_w + phi * drho_w);
    s.dacc[1][1] = phi * rho_w;
    s.dacc[1][2] = 0.0;
    s.dacc[2][0] = dphi * (so * rho_og + sg * rho_g) + phi * (so * rho_og_p + sg * drho_g);
    s.dacc[2][1] = -phi * rho_og;
    s.dacc[2][2] = phi * (-rho_og * dsg + so * rho_og_2 + rho_g * dsg);
    s.rho[0] = rho_oo + rho_og; s.drho[0] = rho_oo_p + rho_og_p;
    s.drho_o2 = rho_oo_2 + rho_og_2;
    s.rho[1] = rho_w; s.drho[1] = drho_w;
    s.rho[2] = rho_g; s.drho[2] = drho_g;
    // mass mobilities rho k_r / mu of each (component, phase) term
    const double rmw = 1.0 / mu_w, rmo = 1.0 / muo, rmg = 1.0 / mug;
    auto oil = [&](int t, double rho, double rho_p, double rho_2) {
      const double m = rho * kro;
      s.lam[t] = div_by(m, muo, rmo);
      s.dlam[t][0] = div_by(rho_p * kro - div_by(m * mu_p, muo, rmo), muo, rmo);
      s.dlam[t][1] = div_by(rho * dkro_w, muo, rmo);
      s.dlam[t][2] = div_by(rho_2 * kro + rho * dkro_g - div_by(m * mu_2, muo, rmo), muo, rmo);
    };
    oil(0, rho_oo, rho_oo_p, rho_oo_2);
    oil(2, rho_og, rho_og_p, rho_og_2);
    s.lam[1] = div_by(rho_w * krw, mu_w, rmw);
    s.dlam[1][0] = div_by(drho_w * krw, mu_w, rmw);
    s.dlam[1][1] = div_by(rho_w * dkrw, mu_w, rmw);
    s.dlam[1][2] = 0.0;
    s.lam[3] = div_by(rho_g * krg, mug, rmg);
    s.dlam[3][0] = div_by(drho_g * krg - div_by(rho_g * krg * dmug, mug, rmg), mug, rmg);
    s.dlam[3][1] = 0.0;
    s.dlam[3][2] = div_by(rho_g * dkrg, mug, rmg);
    s.lt = div_by(krw, mu_w, rmw) + div_by(kro, muo, rmo) + div_by(krg, mug, rmg);
    s.dlt[0] = -kro * mu_p / (muo * muo) - krg * dmug / (mug * mug);
    s.dlt[1] = dkrw / mu_w + dkro_w / muo;
    s.dlt[2] = dkro_g / muo - kro * mu_2 / (muo * muo) + dkrg / mug;
  }
}

// What a face needs of the cells on its two sides.
template <int MODEL>
struct FaceState {
  static constexpr int B = Traits<MODEL>::B, NP = Traits<MODEL>::NP, NT = Traits<MODEL>::NT;
  static constexpr int COUNT = 1 + 2 * NP + NT + NT * B + (MODEL == 3 ? 1 - 2 : 0);   // stored values (dep)
  double p, rho[NP], drho[NP], lam[NT], dlam[NT][B];
  double dro2 = 0.0;   // black oil: d rho_oil-phase / d x2

  __device__ void set(double p0, const CellState<MODEL>& s) {
    p = p0;
    for (int q = 0; q < NP; ++q) {
      rho[q] = s.rho[q];
      drho[q] = s.drho[q];
    }
    for (int q = 0; q < NT; ++q) {
      lam[q] = s.lam[q];
      for (int u = 0; u < B; ++u) dlam[q][u] = s.dlam[q][u];
    }
    if constexpr (MODEL == 3) dro2 = s.drho_o2;
  }
  // value v (0 <= v < COUNT), for storage as planes
  template <typename F>
  __device__ void each(F&& f) {
    int v = 0;
    f(v++, p);
    for (int q = 0; q < NP; ++q) f(v++, rho[q]);
    for (int q = 0; q < NP; ++q) f(v++, drho[q]);
    for (int q = 0; q < NT; ++q) f(v++, lam[q]);
    for (int q = 0; q < NT; ++q)
      for (int u = 0; u < B; ++u)
        if (Traits<MODEL>::dep(q, u)) f(v++, dlam[q][u]);
    if constexpr (MODEL == 3) f(v++, dro2);
  }
};

// Flow of each (component, phase) term through a face from its lower-index
// cell to its upper-index one, with its derivatives in the unknowns of both.
template <int MODEL>
struct FaceFlow {
  static constexpr int B = Traits<MODEL>::B, NT = Traits<MODEL>::NT;
  double F[NT], dlo[NT][B], dhi[NT][B];
};

template <int MODEL>
__device__ inline void face_flow(const FaceState<MODEL>& lo, const FaceState<MODEL>& hi, double T, double dzf,
                                 FaceFlow<MODEL>& o) {
  constexpr int B = Traits<MODEL>::B, NP = Traits<MODEL>::NP, NT = Traits<MODEL>::NT;
  // x2 derivative of the oil-phase potential difference (undersaturated cells)
  const double dd2lo = -0.5 * G_ACC * dzf * lo.dro2;
  const double dd2hi = -0.5 * G_ACC * dzf * hi.dro2;
  double dphi[NP], ddlo[NP], ddhi[NP];
  bool uplo[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    dphi[q] = (lo.p - hi.p) * BAR - 0.5 * (lo.rho[q] + hi.rho[q]) * G_ACC * dzf;
    ddlo[q] = BAR - 0.5 * G_ACC * dzf * lo.drho[q];
    ddhi[q] = -BAR - 0.5 * G_ACC * dzf * hi.drho[q];
    uplo[q] = dphi[q] >= -TIE_BAR * BAR;
  }
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const int ph = Traits<MODEL>::phase(q);
    const double lam_up = uplo[ph] ? lo.lam[q] : hi.lam[q];
    o.F[q] = T * lam_up * dphi[ph];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (!Traits<MODEL>::dep(q, u)) continue;
      o.dlo[q][u] = T * (uplo[ph] ? lo.dlam[q][u] : 0.0) * dphi[ph];
      o.dhi[q][u] = T * (uplo[ph] ? 0.0 : hi.dlam[q][u]) * dphi[ph];
    }
    o.dlo[q][0] += T * lam_up * ddlo[ph];
    o.dhi[q][0] += T * lam_up * ddhi[ph];
    if (MODEL == 3 && ph == 0) {
      o.dlo[q][B - 1] += T * lam_up * dd2lo;
      o.dhi[q][B - 1] += T * lam_up * dd2hi;
    }
  }
}

// Residual and block rows.  A workgroup owns TX x TY columns and marches down
// kz planes of them, one thread a column: each thread evaluates the state of
// its cell one plane ahead (and the workgroup those of the four sides of its
// tile), the states of the current plane meet in LDS for the x and y faces,
// and a z face's flow is carried to the next plane instead of being formed
// again.  So a cell's state is evaluated (TX TY + 2 (TX + TY)) / (TX TY) times
// and never goes to memory; with the states in planes of their own, the
// kernel read them 1,380 bytes a cell beyond the caches (five rows of
// neighbours, none of them still in an XCD's L2) and was bound by that.  Now
// 536 bytes are written and about 85 read per cell, and what bounds it is the
// latency of FP64 chains between the barriers with two workgroups per CU (256
// registers a thread, 60 KB of LDS): VALU issue in a third of the wave cycles.
// The loops over axes and evaluations stay rolled, so that the code fits the
// instruction cache.  Rows of TX = 64 natural cells are 32 consecutive cells
// of either colour, so each store covers whole cache lines.  NAT: x_old, x
// and rhs in natural order, else colour-split; the sums run in direction
// order, one term after the other, whichever side of a face forms its flow.
// The call at MODEL 3: 1592 to 911 us at 256x256x64, 234 to 155 at
// 128x128x32; MODEL 2: 233 to 129 at 60x220x85.
template <int MODEL, int TX, int TY, bool NAT>
__global__ __launch_bounds__(TX * TY) void cell_kernel(FluidDev f, Lay L, int kz, double dz, double top, double vol,
                                                       double dt, double s0, double s1, double s2,
                                                       const double* __restrict__ poro, const double* __restrict__ tp,
                                                       const double* __restrict__ xold, const double* __restrict__ x,
                                                       double* __restrict__ lt, double* __restrict__ J,
                                                       double* __restrict__ rhs) {
  static_assert(2 * (TX + TY) <= TX * TY, "one side cell per thread");
  constexpr int B = Traits<MODEL>::B, NT = Traits<MODEL>::NT;
  using FS = FaceState<MODEL>;
  constexpr int LX = TX + 2, NC = LX * (TY + 2);
  extern __shared__ double sm[];   // [FS::COUNT][NC]
  __shared__ PvtLds pvt;
  if (MODEL == 3) pvt.load(f);
  const size_t n = L.n;
  const int ntx = (L.nx + TX - 1) / TX, nty = (L.ny + TY - 1) / TY;
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const int bx = blk % ntx, by = (blk / ntx) % nty, bz = blk / (ntx * nty);
  const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  const int i = bx * TX + tx, j = by * TY + ty;
  const int k0 = bz * kz, k1 = k0 + kz < L.nz ? k0 + kz : L.nz;
  const bool mine = i < L.nx && j < L.ny;
  const double scale[3] = {s0, s1, s2};
  const double rscale[3] = {1.0 / s0, B > 1 ? 1.0 / s1 : 0.0, B > 2 ? 1.0 / s2 : 0.0};
  const double rdt = 1.0 / dt;
  auto at = [&](int a, int b, int k, int t) {   // cell (a, b, k), colour-split index t, in x_old, x and rhs
    return NAT ? (size_t)a + (size_t)L.nx * (b + (size_t)L.ny * k) : (size_t)t;
  };
  auto put = [&](int c, FS& s) { s.each([&](int v, double& d) { sm[v * NC + c] = d; }); };
  auto get = [&](int c, FS& s) { s.each([&](int v, double& d) { d = sm[v * NC + c]; }); };
  // the side cell of the tile this thread evaluates as well (tid < 2 (TX + TY))
  int si = 0, sj = 0, sc = -1;
  if (tid < 2 * TX) {
    si = bx * TX + tid % TX;
    sj = tid < TX ? by * TY - 1 : by * TY + TY;
    sc = (tid < TX ? 0 : TY + 1) * LX + tid % TX + 1;
  } else if (tid < 2 * (TX + TY)) {
    const int q = tid - 2 * TX;
    sj = by * TY + q % TY;
    si = q < TY ? bx * TX - 1 : bx * TX + TX;
    sc = (q % TY + 1) * LX + (q < TY ? 0 : TX + 1);
  }
  if (si < 0 || si >= L.nx || sj < 0 || sj >= L.ny) sc = -1;
  const int own = (ty + 1) * LX + tx + 1;
  // one entry of block (d, r, u) of cell t
  auto store = [&](int d, int r, int u, int t, double v) {
    J[tix(7 * B * B, (d * B + r) * B + u, t)] = div_by(v, scale[r], rscale[r]);
  };
  __syncthreads();

  double R[B], Jd[B][B];   // current plane; before it, the accumulation terms of the coming one
  FaceFlow<MODEL> below;   // flow through the face between the current plane and the one before
  for (int k = k0 > 0 ? k0 - 2 : -1; k < k1; ++k) {
    const bool full = k >= k0 && mine;                         // a cell of this march
    const bool have = k >= 0 && k >= k0 - 1 && mine;           // its state is in LDS
    const int t = k >= 0 && mine ? lay_index(L, i, j, k) : 0;
    const bool more = k + 1 < L.nz, march = k + 1 >= k0 && k + 1 < k1;   // the coming plane: exists, is of this march
    // every load of the iteration before its stores: a wait for a load is a
    // wait for the stores issued before it
    double xv[B], xw[B], xo[B], pv, pw, tx0, tx1, ty0, ty1, tz;
    {
      // side cell (xv, pv) and own cell (xw, pw, xo) of the coming plane
      const bool s_ = more && march && sc >= 0, o_ = more && mine;
      const int ts = s_ ? lay_index(L, si, sj, k + 1) : 0, to = o_ ? lay_index(L, i, j, k + 1) : 0;
      const size_t es = s_ ? at(si, sj, k + 1, ts) : 0, eo = o_ ? at(i, j, k + 1, to) : 0;
      pv = poro[ts];
      pw = poro[to];
      for (int u = 0; u < B; ++u) {
        xv[u] = x[u * n + es];
        xw[u] = x[u * n + eo];
        xo[u] = xold[u * n + eo];
      }
      tx0 = tp[full && i > 0 ? lay_index(L, i - 1, j, k) : t];
      tx1 = tp[t];
      ty0 = tp[n + (full && j > 0 ? lay_index(L, i, j - 1, k) : t)];
      ty1 = tp[n + t];
      tz = tp[2 * n + t];
    }
    if (full) {
#pragma unroll 1
      for (int axis = 0; axis < 2; ++axis) {
        const int step = axis ? LX : 1;
        double Jo[B][B];
#pragma unroll
        for (int plus = 0; plus < 2; ++plus) {
          for (int r = 0; r < B; ++r)
            for (int u = 0; u < B; ++u) Jo[r][u] = 0.0;
          const int c = axis ? j : i, last = (axis ? L.ny : L.nx) - 1;
          if (plus ? c < last : c > 0) {
            FS lo, hi;
            get(plus ? own : own - step, lo);
            get(plus ? own + step : own, hi);
            FaceFlow<MODEL> q;
            face_flow<MODEL>(lo, hi, axis ? (plus ? ty1 : ty0) : (plus ? tx1 : tx0), 0.0, q);
#pragma unroll
            for (int m = 0; m < NT; ++m) {
              const int row = Traits<MODEL>::row(m);
              if (plus) R[row] += q.F[m]; else R[row] -= q.F[m];
#pragma unroll
              for (int u = 0; u < B; ++u) {
                if (!Traits<MODEL>::dep(m, u)) continue;
                if (plus) {
                  Jd[row][u] += q.dlo[m][u];
                  Jo[row][u] += q.dhi[m][u];
                } else {
                  Jo[row][u] -= q.dlo[m][u];
                  Jd[row][u] -= q.dhi[m][u];
                }
              }
            }
          }
          const int d = 2 * axis + 1 + plus;
          for (int r = 0; r < B; ++r)
            for (int u = 0; u < B; ++u) store(d, r, u, t, Jo[r][u]);
        }
      }
      double Jo[B][B];
      for (int r = 0; r < B; ++r)
        for (int u = 0; u < B; ++u) Jo[r][u] = 0.0;
      if (k > 0) {
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          const int row = Traits<MODEL>::row(m);
          R[row] -= below.F[m];
#pragma unroll
          for (int u = 0; u < B; ++u) {
            if (!Traits<MODEL>::dep(m, u)) continue;
            Jo[row][u] -= below.dlo[m][u];
            Jd[row][u] -= below.dhi[m][u];
          }
        }
      }
      for (int r = 0; r < B; ++r)
        for (int u = 0; u < B; ++u) store(5, r, u, t, Jo[r][u]);
    }
    __syncthreads();   // the plane's states have been read
    CellState<MODEL> cs;
    FS next;
    if (more) {
#pragma unroll 1
      for (int w = 0; w < 2; ++w) {   // the side cell, then the own
        if (w == 0 ? sc >= 0 && march : mine) {
          cell_state<MODEL>(f, pvt, pv, xv, cs);
          next.set(xv[0], cs);
          if (w == 0) put(sc, next);
        }
        for (int u = 0; u < B; ++u) xv[u] = xw[u];
        pv = pw;
      }
    }
    if (have) {
      double Jo[B][B];
      for (int r = 0; r < B; ++r)
        for (int u = 0; u < B; ++u) Jo[r][u] = 0.0;
      if (more) {
        FS lo;
        get(own, lo);
        const double z_self = top + (k + 0.5) * dz, z_nb = top + (k + 1 + 0.5) * dz;
        face_flow<MODEL>(lo, next, tz, z_self - z_nb, below);
        if (full) {
#pragma unroll
          for (int m = 0; m < NT; ++m) {
            const int row = Traits<MODEL>::row(m);
            R[row] += below.F[m];
#pragma unroll
            for (int u = 0; u < B; ++u) {
              if (!Traits<MODEL>::dep(m, u)) continue;
              Jd[row][u] += below.dlo[m][u];
              Jo[row][u] += below.dhi[m][u];
            }
          }
        }
      }
      if (full) {
        const size_t e = at(i, j, k, t);
        for (int r = 0; r < B; ++r) {
          rhs[r * n + e] = -div_by(R[r], scale[r], rscale[r]);
          for (int u = 0; u < B; ++u) {
            store(6, r, u, t, Jo[r][u]);
            store(0, r, u, t, Jd[r][u]);
          }
        }
      }
    }
    if (more && mine) {
      put(own, next);
      if (march) {   // accumulation terms of the coming plane
        const int tn = lay_index(L, i, j, k + 1);
        lt[tn] = cs.lt;
        CellState<MODEL> so;
        cell_state<MODEL>(f, pvt, pw, xo, so);
        for (int r = 0; r < B; ++r) {
          R[r] = div_by(vol * (cs.acc[r] - so.acc[r]), dt, rdt);
          for (int u = 0; u < B; ++u) Jd[r][u] = div_by(vol * cs.dacc[r][u], dt, rdt);
        }
      }
    }
    __syncthreads();
  }
}

// One thread per perforated cell (cells are distinct; checked at creation).
// A perforation of a rate-controlled well takes the BHP from the unknowns
// (x[b n + well]) and also records its border entries: B = dR_cell/dp_h,
// C = dR_w/dx_cell (scaled like the controlled component's rows), and the
// controlled component's mass rate and its derivative in p_h (unscaled) for
// the well equation.
template <int MODEL>
__global__ void well_kernel(FluidDev f, Lay L, int nperf, const Perf* __restrict__ perfs,
                            const RateWell* __restrict__ rwells, double s0, double s1, double s2,
                            const double* __restrict__ poro, const double* __restrict__ x,
                            double* __restrict__ J, double* __restrict__ rhs, double* __restrict__ bord,
                            double* __restrict__ pq, int nat) {
  constexpr int B = Traits<MODEL>::B, NT = Traits<MODEL>::NT;
  __shared__ PvtLds pvt;
  if (MODEL == 3) pvt.load(f);
  __syncthreads();
  int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nperf) return;
  const size_t n = L.n;
  Perf pf = perfs[w];
  int t = pf.cell;
  size_t e = t;   // the cell in x and rhs (nat: in natural order)
  if (nat) {
    int i, j, k;
    lay_coords(L, t, i, j, k);
    e = i + (size_t)L.nx * (j + (size_t)L.ny * k);
  }
  double xv[B];
  for (int u = 0; u < B; ++u) xv[u] = x[u * n + e];
  CellState<MODEL> s;
  cell_state<MODEL>(f, pvt, poro[t], xv, s);
  const double scale[3] = {s0, s1, s2};
  const double ph = pf.rw >= 0 ? x[(size_t)B * n + pf.rw] : pf.bhp;
  double dh = ph - xv[0];
  double q[B], dq[B][B], dqh[B];
  for (int r = 0; r < B; ++r) {
    q[r] = 0.0;
    dqh[r] = 0.0;
    for (int u = 0; u < B; ++u) dq[r][u] = 0.0;
  }
  if (pf.kind == CPR_WELL_INJECTOR) {
    // water injector: total mobility of the cell, water density
    constexpr int WR = MODEL == 1 ? 0 : 1;   // water row and phase
    double rho = s.rho[WR], drho = s.drho[WR];
    double drive = dh * BAR - rho * G_ACC * pf.dzh;
    q[WR] = pf.wi * rho * s.lt * drive;
    dqh[WR] = pf.wi * rho * s.lt * BAR;
    for (int u = 0; u < B; ++u) {
      double v = pf.wi * rho * s.dlt[u] * drive;
      if (u == 0) {
        v += pf.wi * drho * s.lt * drive;
        v += pf.wi * rho * s.lt * (-BAR - drho * G_ACC * pf.dzh);
      }
      dq[WR][u] = v;
    }
  } else {
    for (int tt = 0; tt < NT; ++tt) {
      int c = Traits<MODEL>::row(tt), ph_ = Traits<MODEL>::phase(tt);
      double rho = s.rho[ph_], drho = s.drho[ph_];
      double drive = dh * BAR - rho * G_ACC * pf.dzh;
      q[c] += pf.wi * s.lam[tt] * drive;
      dqh[c] += pf.wi * s.lam[tt] * BAR;
      for (int u = 0; u < B; ++u) {
        double v = pf.wi * s.dlam[tt][u] * drive;
        if (u == 0) v += pf.wi * s.lam[tt] * (-BAR - drho * G_ACC * pf.dzh);
        if (MODEL == 3 && u == 2 && ph_ == 0) v += pf.wi * s.lam[tt] * (-s.drho_o2 * G_ACC * pf.dzh);
        dq[c][u] += v;
      }
    }
  }
  for (int r = 0; r < B; ++r) {
    rhs[r * n + e] += q[r] / scale[r];
    for (int u = 0; u < B; ++u) J[tix(7 * B * B, r * B + u, t)] -= dq[r][u] / scale[r];
  }
  if (pf.rw >= 0) {
    const int c = rwells[pf.rw].comp;
    double* bq = bord + (size_t)w * 6;
    for (int r = 0; r < 3; ++r) {
      bq[r] = r < B ? -dqh[r] / scale[r] : 0.0;
      bq[3 + r] = r < B ? dq[c][r] / scale[c] : 0.0;
    }
    pq[2 * w] = q[c];
    pq[2 * w + 1] = dqh[c];
  }
}

// Well equation of each rate-controlled well, summed over its perforations
// in order: R_w = (sum q_c - target) / s_c, D = sum dq_c/dp_h / s_c; the
// right-hand side tail receives -R_w.
__global__ void rate_well_kernel(int b, int n, int nrate, const RateWell* __restrict__ rwells,
                                 const double* __restrict__ pq, double s0, double s1, double s2,
                                 double* __restrict__ bordD, double* __restrict__ rhs) {
  int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nrate) return;
  const double scale[3] = {s0, s1, s2};
  const RateWell R = rwells[w];
  const double sc = scale[R.comp];
  double acc = -R.target, d = 0.0;
  for (int q = R.p0; q < R.p1; ++q) {
    acc += pq[2 * q];
    d += pq[2 * q + 1];
  }
  rhs[(size_t)b * n + w] = -(acc / sc);
  bordD[w] = d / sc;
}

__global__ void trans_kernel(Lay L, double dx, double dy, double dz, const double* __restrict__ perm,
                             double* __restrict__ tp) {
  const double MD = 9.869233e-16;
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= L.n) return;
  const size_t n = L.n;
  int i = t % L.nx, jk = t / L.nx;
  int j = jk % L.ny, k = jk / L.ny;
  int c = lay_index(L, i, j, k);
  const int nbr[3] = {i + 1 < L.nx ? t + 1 : -1, j + 1 < L.ny ? t + L.nx : -1,
                      k + 1 < L.nz ? t + L.nx * L.ny : -1};
  const double area[3] = {dy * dz, dx * dz, dx * dy};
  const double dd[3] = {dx, dy, dz};
  for (int a = 0; a < 3; ++a) {
    double T = 0.0;
    if (nbr[a] >= 0) {
      double ka = perm[a * n + t] * MD, kb = perm[a * n + nbr[a]] * MD;
      double s = ka + kb;
      T = s > 0.0 ? 2.0 * area[a] * ka * kb / (dd[a] * s) : 0.0;
    }
    tp[a * n + c] = T;
  }
}

}  // namespace

void launch_transmissibility(const Lay& L, const cpr_grid_t& g, const double* perm_nat,
                             double* tp, hipStream_t s) {
  trans_kernel<<<div_up(L.n, 256), 256, 0, s>>>(L, g.dx, g.dy, g.dz, perm_nat, tp);
}

namespace {

// The tile is 32 x 8 columns, or 64 x 4 where that leaves fewer threads
// without a cell (128 against 164 us at 96x70x50, where 64 pads the rows;
// 148 against 141 at 60x220x85, where 32 pads the columns; equal at
// 128x128x32).  A march is as long as leaves the device two rounds of two
// workgroups per CU, at most 16 planes (each march evaluates up to two planes
// beyond its own).
template <int MODEL, int TX, int TY, bool NAT>
int launch_cells(cpr_ctx* ctx, const double* xold, const double* x, double dt, const double (&sc)[3], double* rhs) {
  const Lay& L = ctx->lay;
  constexpr int lds = FaceState<MODEL>::COUNT * (TX + 2) * (TY + 2) * (int)sizeof(double);
  CPR_TRY(hipFuncSetAttribute((const void*)cell_kernel<MODEL, TX, TY, NAT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              lds));
  const long tiles = (long)div_up(L.nx, TX) * div_up(L.ny, TY);
  int kz = (int)(tiles * L.nz / 1024);
  kz = kz < 1 ? 1 : kz > 16 ? 16 : kz;
  prof_begin(ctx, CPR_KCLASS_ASSEMBLE);
  cell_kernel<MODEL, TX, TY, NAT><<<(unsigned)(tiles * div_up(L.nz, kz)), TX * TY, lds, ctx->stream>>>(
      ctx->fl, L, kz, ctx->grid.dz, ctx->grid.top, ctx->cell_vol, dt, sc[0], sc[1], sc[2], ctx->poro, ctx->tp, xold, x,
      ctx->lt, ctx->J, rhs);
  prof_end(ctx, CPR_KCLASS_ASSEMBLE);
  return CPR_OK;
}

template <int MODEL, bool NAT>
int assemble_model(cpr_ctx* ctx, const double* xold, const double* x, double dt, const double (&sc)[3], double* rhs) {
  const Lay& L = ctx->lay;
  hipStream_t s = ctx->stream;
  const long wide = (long)div_up(L.nx, 64) * 64 * div_up(L.ny, 4) * 4;
  const long narrow = (long)div_up(L.nx, 32) * 32 * div_up(L.ny, 8) * 8;
  const int rc = wide < narrow ? launch_cells<MODEL, 64, 4, NAT>(ctx, xold, x, dt, sc, rhs)
                               : launch_cells<MODEL, 32, 8, NAT>(ctx, xold, x, dt, sc, rhs);
  if (rc != CPR_OK) return rc;
  const int np = (int)ctx->perfs.size();
  if (np)
    well_kernel<MODEL><<<div_up(np, 64), 64, 0, s>>>(ctx->fl, L, np, ctx->perfs_d, ctx->rwells_d, sc[0], sc[1], sc[2],
                                                     ctx->poro, x, ctx->J, rhs, ctx->bord, ctx->pq, NAT);
  if (ctx->nrate)
    rate_well_kernel<<<div_up(ctx->nrate, 64), 64, 0, s>>>(ctx->b, L.n, ctx->nrate, ctx->rwells_d, ctx->pq, sc[0],
                                                          sc[1], sc[2], ctx->bord_d, rhs);
  return CPR_OK;
}

template <bool NAT>
int assemble_order(cpr_ctx* ctx, const double* xold, const double* x, double dt_days, double* rhs) {
  const double dt = dt_days * DAY;
  double sc[3] = {0, 0, 0};
  for (int c = 0; c < ctx->b; ++c) sc[c] = ctx->rho_scale[c] * ctx->cell_vol * ctx->phibar / dt;
  if (ctx->fl.model == 1) return assemble_model<1, NAT>(ctx, xold, x, dt, sc, rhs);
  if (ctx->fl.model == 2) return assemble_model<2, NAT>(ctx, xold, x, dt, sc, rhs);
  return assemble_model<3, NAT>(ctx, xold, x, dt, sc, rhs);
}

}  // namespace

int launch_assemble(cpr_ctx* ctx, const double* xold, const double* x, double dt_days, double* rhs, bool nat) {
  return nat ? assemble_order<true>(ctx, xold, x, dt_days, rhs) : assemble_order<false>(ctx, xold, x, dt_days, rhs);
}

double host_pvt(const FluidDev& f, int row, double p) { return pvt_eval(f, row, p); }
