// Extended GRMHD (Implicit Solver and Extended Theory section, EGRMHD
// subsection, after Chandra et al. 2015 in the rescaled variables of Foucart
// et al. 2016).  Two zone-centred variables join the eight of ideal GRMHD:
//   X0 = q  (tau_R / (chi rho Theta^2))^(1/2),   the rescaled heat flux,
//   X1 = dP (tau_R / (nu rho Theta))^(1/2),      the rescaled anisotropy,
// Theta = (gam - 1) u / rho.  The stress-energy tensor gains
//   q bh^mu u_nu + q bh_nu u^mu - dP (bh^mu bh_nu - h^mu_nu / 3),
// bh = b / |b|, h^mu_nu = delta^mu_nu + u^mu u_nu (nothing where b^2 = 0),
// and each X obeys
//   d_mu(sqrt(-g) X u^mu) = sqrt(-g) [-(X - X_target) / tau_R + (X / 2) div u],
// with the targets of the Chandra et al. closure
//   q_target  = -rho chi bh^mu (d_mu Theta + Theta a_mu),  a_mu = u^nu nabla_nu u_mu,
//   dP_target = 3 rho nu (bh^mu bh^nu nabla_mu u_nu - div u / 3),
// rescaled like the variables and taken from centred spatial differences of
// the stage's explicit state (time derivatives left out).  div u =
// d_t u^t + d_i(sqrt(-g) u^i) / sqrt(-g): the spatial part explicit, the
// time part (u^t - u^t(step start)) / h implicit like the relaxation and the
// X multiplying div u.
//
// A predictor-corrector stage (h = dt/2, then h = dt from the step's state
// again with the predicted state's explicit rates) runs six launches: the
// ghost fill of X, the face fluxes of all ten variables (ideal LLF speeds),
// the Flux-CT EMFs (the ideal kernel), the targets pass (X targets and the
// spatial div u), the update pass that forms each zone's explicit
// right-hand sides U^n + h L (ten slots), and the implicit pass: per zone
// the implicit solver's Newton on the five hydro prims, with the two X
// equations, linear in X for a given hydro state, solved for X inside
// every residual evaluation.
//
// FP64 throughout, every operation rounded on its own in the order written;
// quotients and roots by plain_div and plain_sqrt, whose bits are those of the
// correctly rounded ones.
//
// Included inside the anonymous namespace of grmhd.hip.

#include "newton_group.hpp"

constexpr int NXV = 2;  // extra variables per zone (stored as a pair per zone: index 2 c + n)

// Physical heat flux q and anisotropy dP of the rescaled variables x.
__device__ __forceinline__ void emhd_unscale(const Dev& g, const double p[NVAR], const double x[NXV], double& q,
                                             double& dP) {
#pragma clang fp contract(off)
  const double theta = plain_div((g.gam - 1.0) * p[UU], p[RHO]), itau = plain_rcp(g.tau);
  q = x[0] * theta * plain_sqrt(quotient(g.chi * p[RHO], g.tau, itau));
  dP = x[1] * plain_sqrt(quotient(g.nu * p[RHO] * theta, g.tau, itau));
}

// Row mu of the extended mixed stress-energy tensor.
__device__ __forceinline__ void tmunu_row_emhd(const double p[NVAR], const Fluid<double>& f, double gam, double q,
                                               double dP, int mu, double T[4]) {
#pragma clang fp contract(off)
  fplain::tmunu_row(p, f, gam, mu, T);
  if (!(f.bsq > 0.0) || (q == 0.0 && dP == 0.0)) return;
  const double sb = plain_sqrt(f.bsq), isb = plain_rcp(sb), third = 1.0 / 3.0;
  const double bm = quotient(f.bcon[mu], sb, isb);
#pragma unroll
  for (int nu = 0; nu < 4; nu++) {
    const double bn = quotient(f.bcov[nu], sb, isb);
    const double h = (mu == nu ? 1.0 : 0.0) + f.ucon[mu] * f.ucov[nu];
    T[nu] = ((T[nu] + q * bm * f.ucov[nu]) + q * bn * f.ucon[mu]) - dP * (bm * bn - quotient(h, 3.0, third));
  }
}

// Conserved variables (d = 0) or fluxes along x^d of the ten variables:
// sqrt(-g) (rho u^d, T^d_t + rho u^d, T^d_i, b^k u^d - b^d u^k, X u^d).
__device__ __forceinline__ void prim_to_flux_emhd(const Dev& g, const double p[NVAR], const double x[NXV],
                                                  const Fluid<double>& f, const PointMetric<double>& m, int d,
                                                  double F[NVAR + NXV]) {
#pragma clang fp contract(off)
  double q, dP;
  emhd_unscale(g, p, x, q, dP);
  double T[4];
  tmunu_row_emhd(p, f, g.gam, q, dP, d, T);
  F[RHO] = (m.gdet * p[RHO]) * f.ucon[d];
  F[UU] = m.gdet * (T[0] + p[RHO] * f.ucon[d]);
  F[U1] = m.gdet * T[1];
  F[U2] = m.gdet * T[2];
  F[U3] = m.gdet * T[3];
  if (d == 0) {
    F[B1] = m.gdet * p[B1];
    F[B2] = m.gdet * p[B2];
    F[B3] = m.gdet * p[B3];
  } else {
    F[B1] = m.gdet * (f.bcon[1] * f.ucon[d] - f.bcon[d] * f.ucon[1]);
    F[B2] = m.gdet * (f.bcon[2] * f.ucon[d] - f.bcon[d] * f.ucon[2]);
    F[B3] = m.gdet * (f.bcon[3] * f.ucon[d] - f.bcon[d] * f.ucon[3]);
  }
#pragma unroll
  for (int n = 0; n < NXV; n++) F[NVAR + n] = (m.gdet * x[n]) * f.ucon[d];
}

// Ghost zones of the extra variables: the maps of k_bc, no sign flips (both
// are scalars under the polar reflection).
__global__ void __launch_bounds__(BLOCK) k_bc_extra(Dev g, double* X) {
  long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= ghost_count(g)) return;
  int i, j, k;
  ghost_index(g, t, i, j, k);
  bool f1 = false, f2 = false, f3 = false;
  const int si = bc_map(i, g.n1, g.bc[0], g.bc[1], f1);
  const int sj = bc_map(j, g.n2, g.bc[2], g.bc[3], f2);
  const int sk = bc_map(k, g.n3, g.bc[4], g.bc[5], f3);
  if (si == i && sj == j && sk == k) return;  // frozen
  const long src = zid(g, si, sj, sk), dst = zid(g, i, j, k);
  Pair<double>* q = (Pair<double>*)X;
  q[dst] = q[src];
}

// The caller's extra variables [2][padded] into the state and the stage
// buffer (which carries the same frozen ghosts), and the state back out.
__global__ void __launch_bounds__(BLOCK) k_load_extra(long nz, const double* __restrict__ src, double* __restrict__ X,
                                                      double* __restrict__ X1) {
  const long c = blockIdx.x * (long)BLOCK + threadIdx.x;
  if (c >= nz) return;
  const Pair<double> x{src[c], src[nz + c]};
  ((Pair<double>*)X)[c] = x;
  ((Pair<double>*)X1)[c] = x;
}
__global__ void __launch_bounds__(BLOCK) k_read_extra(long nz, const double* __restrict__ X, double* __restrict__ dst) {
  const long c = blockIdx.x * (long)BLOCK + threadIdx.x;
  if (c >= nz) return;
  const Pair<double> x = ((const Pair<double>*)X)[c];
  dst[c] = x.a;
  dst[nz + c] = x.b;
}

// WENO5 on the zone values (12 times the smoothness indicators, the candidates
// over a common denominator, a correctly rounded quotient), where the ideal
// step works on differences.  A torus's atmosphere holds tens to thousands of
// zones whose implicit solve does not converge; there the step amplifies a
// changed last bit of a face state or of dt to 1e-3 of the prims.  Extended
// GRMHD therefore rounds as it always has (here, zone_rate_ordered, and the
// sums of every kernel below), so that a run repeats the runs before it.
namespace wv {
#pragma clang fp contract(off)
__device__ __forceinline__ void indicators(double a, double b, double c, double d, double e, double eps, double& s0,
                                           double& s1, double& s2) {
  const double eps12 = 12.0 * eps;
  const double t0 = fma(-2.0, b, a + c), u0 = fma(-4.0, b, fma(3.0, c, a));
  const double t1 = fma(-2.0, c, b + d), u1 = b - d;
  const double t2 = fma(-2.0, d, c + e), u2 = fma(-4.0, d, fma(3.0, c, e));
  s0 = fma(13.0 * t0, t0, fma(3.0 * u0, u0, eps12));
  s1 = fma(13.0 * t1, t1, fma(3.0 * u1, u1, eps12));
  s2 = fma(13.0 * t2, t2, fma(3.0 * u2, u2, eps12));
  s0 *= s0;
  s1 *= s1;
  s2 *= s2;
}
__device__ __forceinline__ double weno5(double a, double b, double c, double d, double e, double eps) {
  double s0, s1, s2;
  indicators(a, b, c, d, e, eps, s0, s1, s2);
  const double w0 = s1 * s2, w1 = 6.0 * (s0 * s2), w2 = 3.0 * (s0 * s1);
  const double p0 = fma(11.0, c, fma(-7.0, b, 2.0 * a));
  const double p1 = fma(2.0, d, fma(5.0, c, -b));
  const double p2 = fma(5.0, d, fma(2.0, c, -e));
  const double den = 6.0 * ((w0 + w1) + w2);
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  r = fma(fma(-den, r, 1.0), r, r);
  return quotient(fma(w0, p0, fma(w1, p1, w2 * p2)), den, r);
}
}  // namespace wv
// Far edge of a zone for the two variables of pair index c, the zones behind
// it s apart on the side away from the edge: the left state of a face comes
// from the zones below it (s > 0, c the zone below), the right state is the
// same expression on the mirrored stencil (s < 0, c the zone above).
template <int RECON>
__device__ __forceinline__ void recon_edge(const Pair<double>* __restrict__ q, long c, long s, double eps, double& a,
                                           double& b) {
  const Pair<double> m1 = q[c - s], z = q[c], p1 = q[c + s];
  if (RECON == GRMHD_RECON_MC) {
    a = mc_left(m1.a, z.a, p1.a);
    b = mc_left(m1.b, z.b, p1.b);
  } else {
    const Pair<double> m2 = q[c - 2 * s], p2 = q[c + 2 * s];
    a = wv::weno5(m2.a, m1.a, z.a, p1.a, p2.a, eps);
    b = wv::weno5(m2.b, m1.b, z.b, p1.b, p2.b, eps);
  }
}

// LLF flux of the ten variables through the lower D-face of zone (i, j, k),
// the face metric from tab; pole faces get zero.  The normal field's flux is
// not stored (Flux-CT reads only the tangential ones).
template <int D, int RECON>
__device__ __forceinline__ void emhd_face(const Dev& g, const double* __restrict__ P,
                                          const double* __restrict__ X, const double* __restrict__ tab,
                                          double* __restrict__ F, double* __restrict__ FX, int i, int j,
                                          int k) {
#pragma clang fp contract(off)
  const long c = zid(g, i, j, k);
  if (pole_face<D>(g, j)) {
    const double zero[NVAR] = {};
    store_flux<D>(F, g.nz, c, zero, g.stream);
    ((Pair<double>*)FX)[c] = Pair<double>{0.0, 0.0};
    return;
  }
  const long s = D == 1 ? 1 : (D == 2 ? (long)g.s1 : g.plane);
  PointMetric<double> m;
  load_metric<double>(tab, g.plane, pid(g, i, j), m);
  // one side at a time: F_L + F_R in S, U_R - U_L in J
  double S[NVAR + NXV] = {}, J[NVAR + NXV] = {}, cmax = 0.0;
#pragma unroll 1
  for (int side = 0; side < 2; side++) {
    const long z = side ? c : c - s, t = side ? -s : s;
    double q[NVAR], x[NXV];
#pragma unroll
    for (int v = 0; v < NVAR; v += 2)
      recon_edge<RECON>((const Pair<double>*)P + (v >> 1) * g.nz, z, t, g.weno_eps, q[v], q[v + 1]);
    recon_edge<RECON>((const Pair<double>*)X, z, t, g.weno_eps, x[0], x[1]);
    Fluid<double> f;
    fplain::fluid_state(q, m, f);
    double Fd[NVAR + NXV], Ut[NVAR + NXV], cp, cm;
    prim_to_flux_emhd(g, q, x, f, m, D, Fd);
    prim_to_flux_emhd(g, q, x, f, m, 0, Ut);
#pragma unroll
    for (int v = 0; v < NVAR + NXV; v++)
      if (v != B1 + D - 1) {
        S[v] = S[v] + Fd[v];
        J[v] = Ut[v] - J[v];
      }
    fplain::char_speeds(q, f, m, g.gam, D, cp, cm);
    if (cp > cmax) cmax = cp;
    if (-cm > cmax) cmax = -cm;
  }
  double f[NVAR + NXV];
#pragma unroll
  for (int v = 0; v < NVAR + NXV; v++)
    if (v != B1 + D - 1) f[v] = 0.5 * S[v] - 0.5 * cmax * J[v];
  store_flux<D>(F, g.nz, c, f, g.stream);
  ((Pair<double>*)FX)[c] = Pair<double>{f[NVAR], f[NVAR + 1]};
}

// All three face directions in one launch, partitioned as k_flux_all.  Bound by
// FP64 arithmetic (about 3000 operations per WENO5 face).  One side's states at
// a time, in a loop that is not unrolled: both at once need more than the 256
// registers of two waves per SIMD (64^3 torus, WENO5: 151 us with 396 bytes of
// scratch, 76 us so, with 154 registers and three waves).
template <int RECON>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_flux_emhd(Dev g, Sched b1, Sched b2, Sched b3, unsigned nb1, unsigned nb2, unsigned nb3,
            const double* __restrict__ P, const double* __restrict__ X, const double* __restrict__ tabF1,
            const double* __restrict__ tabF2, const double* __restrict__ tabC, double* __restrict__ F1,
            double* __restrict__ F2, double* __restrict__ F3, double* __restrict__ FX1,
            double* __restrict__ FX2, double* __restrict__ FX3) {
  const unsigned b = blockIdx.x;
  int i, j, k;
  if (b < nb1) {
    if (sched_index(b1, b, nb1, i, j, k)) emhd_face<1, RECON>(g, P, X, tabF1, F1, FX1, i, j, k);
  } else if (b < nb1 + nb2) {
    if (sched_index(b2, b - nb1, nb2, i, j, k)) emhd_face<2, RECON>(g, P, X, tabF2, F2, FX2, i, j, k);
  } else {
    if (sched_index(b3, b - nb1 - nb2, nb3, i, j, k)) emhd_face<3, RECON>(g, P, X, tabC, F3, FX3, i, j, k);
  }
}

// Targets X_target and the spatial part of div u at zone (i, j, k) from the
// ghost-filled prims P; p, f, m: the zone's prims, fluid state and metric.
// Axes with one zone contribute no differences.
__device__ __forceinline__ void emhd_targets(const Dev& g, const double* __restrict__ P,
                                             const double* __restrict__ tabC, const double* __restrict__ conn,
                                             int i, int j, int k, const double p[NVAR], const Fluid<double>& f,
                                             const PointMetric<double>& m, double Xt[NXV], double& divu_sp) {
#pragma clang fp contract(off)
  const long c = zid(g, i, j, k), q2 = pid(g, i, j);
  const double gam = g.gam;
  const double th0 = (gam - 1.0) * p[UU] / p[RHO];
  // d_a Theta, d_a u_nu and d_a (sqrt(-g) u^a)
  double dth[3], du[3][4], dgu[3];
  const int n[3] = {g.n1, g.n2, g.n3};
  const double dx[3] = {g.dx1, g.dx2, g.dx3};
#pragma unroll
  for (int a = 0; a < 3; a++) {
    dth[a] = dgu[a] = 0.0;
#pragma unroll
    for (int nu = 0; nu < 4; nu++) du[a][nu] = 0.0;
    if (n[a] == 1) continue;
    const long s = a == 0 ? 1 : (a == 1 ? (long)g.s1 : g.plane);
    const long qs = a == 0 ? 1 : (a == 1 ? (long)g.s1 : 0);
    double pp[NVAR], pm[NVAR];
    load8(P, g.nz, c + s, pp);
    load8(P, g.nz, c - s, pm);
    PointMetric<double> mp, mm;
    load_metric<double>(tabC, g.plane, q2 + qs, mp);
    load_metric<double>(tabC, g.plane, q2 - qs, mm);
    Fluid<double> sp, sm;
    fplain::fluid_state(pp, mp, sp);
    fplain::fluid_state(pm, mm, sm);
    const double thp = (gam - 1.0) * pp[UU] / pp[RHO];
    const double thm = (gam - 1.0) * pm[UU] / pm[RHO];
    const double h2 = 2.0 * dx[a];
    dth[a] = (thp - thm) / h2;
#pragma unroll
    for (int nu = 0; nu < 4; nu++) du[a][nu] = (sp.ucov[nu] - sm.ucov[nu]) / h2;
    dgu[a] = (mp.gdet * sp.ucon[a + 1] - mm.gdet * sm.ucon[a + 1]) / h2;
  }
  divu_sp = ((dgu[0] + dgu[1]) + dgu[2]) / m.gdet;
  Xt[0] = Xt[1] = 0.0;
  if (!(f.bsq > 0.0)) return;
  auto cn = [&](int l, int mu, int nu) { return conn[(l * 10 + sidx(mu, nu)) * g.plane + q2]; };
  double bh[4];
#pragma unroll
  for (int mu = 0; mu < 4; mu++) bh[mu] = f.bcon[mu] / sqrt(f.bsq);
  // a_nu = u^i d_i u_nu - Gamma^l_{m nu} u^m u_l
  double acc[4];
#pragma unroll
  for (int nu = 0; nu < 4; nu++) {
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; a++) s += f.ucon[a + 1] * du[a][nu];
#pragma unroll
    for (int l = 0; l < 4; l++)
#pragma unroll
      for (int mu = 0; mu < 4; mu++) s -= cn(l, mu, nu) * f.ucon[mu] * f.ucov[l];
    acc[nu] = s;
  }
  double gq = 0.0;  // bh^mu (d_mu Theta + Theta a_mu)
#pragma unroll
  for (int a = 0; a < 3; a++) gq += bh[a + 1] * dth[a];
#pragma unroll
  for (int nu = 0; nu < 4; nu++) gq += th0 * bh[nu] * acc[nu];
  double bbu = 0.0;  // bh^mu bh^nu nabla_mu u_nu
#pragma unroll
  for (int a = 0; a < 3; a++)
#pragma unroll
    for (int nu = 0; nu < 4; nu++) bbu += bh[a + 1] * bh[nu] * du[a][nu];
#pragma unroll
  for (int mu = 0; mu < 4; mu++)
#pragma unroll
    for (int nu = 0; nu < 4; nu++)
#pragma unroll
      for (int l = 0; l < 4; l++) bbu -= bh[mu] * bh[nu] * cn(l, mu, nu) * f.ucov[l];
  const double rho = p[RHO];
  if (g.chi > 0.0) Xt[0] = -gq * sqrt(g.chi * rho * g.tau) / th0;
  if (g.nu > 0.0) Xt[1] = 3.0 * (bbu - divu_sp / 3.0) * sqrt(g.nu * rho * g.tau / th0);
}

// Targets pass of a stage: X_target of every interior zone to xt (the
// update pass reads them there and overwrites them with the X right-hand
// sides, zone by zone) and the spatial div u to divu.
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_targets_emhd(Dev g, Sched box, const double* __restrict__ Pin, const double* __restrict__ tabC,
               const double* __restrict__ conn, double* __restrict__ xt, double* __restrict__ divu) {
  int i, j, k;
  if (!sched_index(box, blockIdx.x, gridDim.x, i, j, k)) return;
  const long c = zid(g, i, j, k);
  double p[NVAR];
  load8(Pin, g.nz, c, p);
  PointMetric<double> m;
  load_metric<double>(tabC, g.plane, pid(g, i, j), m);
  Fluid<double> f;
  fplain::fluid_state(p, m, f);
  double Xt[NXV], dsp;
  emhd_targets(g, Pin, tabC, conn, i, j, k, p, f, m, Xt, dsp);
  ((Pair<double>*)xt)[c] = Pair<double>{Xt[0], Xt[1]};
  divu[c] = dsp;
}

// Update pass of a stage: per interior zone the explicit right-hand sides
// of the ten variables, U^n + h (-flux divergence + geometric source) for
// the eight ideal slots (the field from the edge EMFs as in update_zone)
// and U^n_X + h (-flux divergence + sqrt(-g) X_target / tau_R) for X (the
// targets as the targets pass left them in xrhs), to ustar and xrhs.
// STAGE 1 (h = dt/2) also keeps U^n of the stage input in V, VX and its u^t
// in utn; STAGE 2 (h = dt) reads them.  dt from dt_dev when given.
template <int STAGE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_update_emhd(Dev g, Sched box, const double* __restrict__ Pin, const double* __restrict__ Xin,
              double* __restrict__ V, double* __restrict__ VX, double* __restrict__ utn,
              const double* __restrict__ F1, const double* __restrict__ F2, const double* __restrict__ F3,
              const double* __restrict__ FX1, const double* __restrict__ FX2, const double* __restrict__ FX3,
              const double* __restrict__ E1, const double* __restrict__ E2, const double* __restrict__ E3,
              const double* __restrict__ tabC, const double* __restrict__ conn, double dt,
              const double* __restrict__ dt_dev, double* __restrict__ ustar, double* __restrict__ xrhs,
              unsigned long long* nopen) {
#pragma clang fp contract(off)
  if (blockIdx.x == 0 && threadIdx.x == 0) *nopen = 0;   // for the implicit pass
  int i, j, k;
  if (!sched_index(box, blockIdx.x, gridDim.x, i, j, k)) return;
  if (dt_dev) dt = *dt_dev;
  const long c = zid(g, i, j, k), nz = g.nz, si = 1, sj = g.s1, sk = g.plane;
  const long q2 = pid(g, i, j);
  double p[NVAR], x[NXV];
  load8(Pin, nz, c, p);
#pragma unroll
  for (int n = 0; n < NXV; n++) x[n] = Xin[2 * c + n];
  PointMetric<double> m;
  load_metric<double>(tabC, g.plane, q2, m);
  Fluid<double> f;
  fplain::fluid_state(p, m, f);
  double qh, dPh;
  emhd_unscale(g, p, x, qh, dPh);

  double L[NVAR];
  {
    // sqrt(-g) T^k_l Gamma^l_{nu k} with the extended T, sums over k, then l
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      double Tk[4];
      tmunu_row_emhd(p, f, g.gam, qh, dPh, kk, Tk);
#pragma unroll
      for (int nu = 0; nu < 4; nu++)
#pragma unroll
        for (int l = 0; l < 4; l++) s[nu] += Tk[l] * conn[(l * 10 + sidx(nu, kk)) * g.plane + q2];
    }
    const double r1 = plain_rcp(g.dx1), r2 = plain_rcp(g.dx2), r3 = plain_rcp(g.dx3);
    double lo[5], hi[5];
    load_flux5(F1, nz, c, lo);
    load_flux5(F1, nz, c + si, hi);
#pragma unroll
    for (int v = 0; v < 5; v++) L[v] = quotient(hi[v] - lo[v], g.dx1, r1);
    load_flux5(F2, nz, c, lo);
    load_flux5(F2, nz, c + sj, hi);
#pragma unroll
    for (int v = 0; v < 5; v++) L[v] = L[v] + quotient(hi[v] - lo[v], g.dx2, r2);
    load_flux5(F3, nz, c, lo);
    load_flux5(F3, nz, c + sk, hi);
#pragma unroll
    for (int v = 0; v < 5; v++) L[v] = -(L[v] + quotient(hi[v] - lo[v], g.dx3, r3)) + (v == RHO ? 0.0 : m.gdet * s[v - 1]);
    ct_field_rate(g, E1, E2, E3, c, L);
  }
  double LX[NXV];
#pragma unroll
  for (int n = 0; n < NXV; n++) {
    const long o = 2 * c + n;
    const double d1 = (FX1[o + 2 * si] - FX1[o]) / g.dx1;
    const double d2 = (FX2[o + 2 * sj] - FX2[o]) / g.dx2;
    const double d3 = (FX3[o + 2 * sk] - FX3[o]) / g.dx3;
    LX[n] = -((d1 + d2) + d3) + m.gdet * xrhs[o] / g.tau;
  }
  double U0[NVAR + NXV];
  if (STAGE == 1) {
    prim_to_flux_emhd(g, p, x, f, m, 0, U0);
    store8(V, nz, c, U0);
#pragma unroll
    for (int n = 0; n < NXV; n++) VX[2 * c + n] = U0[NVAR + n];
    utn[c] = f.ucon[0];
  } else {
    load8(V, nz, c, U0);
#pragma unroll
    for (int n = 0; n < NXV; n++) U0[NVAR + n] = VX[2 * c + n];
  }
  const double h = STAGE == 1 ? 0.5 * dt : dt;
#pragma unroll
  for (int v = 0; v < NVAR; v++) L[v] = U0[v] + h * L[v];
  store8(ustar, nz, c, L);
#pragma unroll
  for (int n = 0; n < NXV; n++) xrhs[2 * c + n] = U0[NVAR + n] + h * LX[n];
}

// Implicit pass of a stage: per interior zone, the hydro prims and X whose
// ten conserved variables equal the right-hand sides plus h times the
// implicit X sources.  Given the hydro state the X equations read
//   sqrt(-g) X (u^t + h / tau_R - (h / 2) div u) = xrhs,
//   div u = divu + (u^t - u^t_n) / h,
// solved for X inside every residual; the Newton runs on the five hydro
// prims from the stage input (the guess), the field is xrhs's B /
// sqrt(-g).  On failure the zone keeps the guess's hydro prims and X (the
// field still updated) and is counted.
struct ImplicitZone {
  PointMetric<double> m;
  double Us[NVAR], Ux[NXV], B[3], dsp, ut_n, h, ih, htau, scale, iscale;

  __device__ __forceinline__ void load(const Dev& g, long c, int i, int j, const double* __restrict__ ustar,
                                       const double* __restrict__ xrhs, const double* __restrict__ divu,
                                       const double* __restrict__ utn, const double* __restrict__ tabC, double step) {
#pragma clang fp contract(off)
    load8(ustar, g.nz, c, Us);
#pragma unroll
    for (int n = 0; n < NXV; n++) Ux[n] = xrhs[2 * c + n];
    dsp = divu[c];
    ut_n = utn[c];
    h = step;
    load_metric<double>(tabC, g.plane, pid(g, i, j), m);
#pragma unroll
    for (int k = 0; k < 3; k++) B[k] = Us[B1 + k] / m.gdet;
    ih = plain_rcp(h);
    htau = h * m.gdet / g.tau;
    scale = 0.0;
#pragma unroll
    for (int kk = 0; kk < 5; kk++)
      if (fabs(Us[kk]) > scale) scale = fabs(Us[kk]);
    iscale = plain_rcp(scale);
  }
  __device__ __forceinline__ bool solvable() const { return scale > 0.0 && isfinite(scale); }
  // X of a hydro state with fluid state fz
  __device__ __forceinline__ void xsolve(const Fluid<double>& fz, double Xz[NXV]) const {
#pragma clang fp contract(off)
    const double ut = fz.ucon[0];
    const double du = dsp + quotient(ut - ut_n, h, ih);
    const double coef = m.gdet * ut + htau - 0.5 * h * m.gdet * du;
    const double ic = plain_rcp(coef);
#pragma unroll
    for (int n = 0; n < NXV; n++) Xz[n] = quotient(Ux[n], coef, ic);
  }
  __device__ __forceinline__ void residual(const Dev& g, const double xx[5], double R[5]) const {
#pragma clang fp contract(off)
    const double gd = m.gdet;
    const double Pz[NVAR] = {xx[0], xx[1], xx[2], xx[3], xx[4], B[0], B[1], B[2]};
    Fluid<double> fz;
    fplain::fluid_state(Pz, m, fz);
    double Xz[NXV];
    xsolve(fz, Xz);
    double q, dP;
    emhd_unscale(g, Pz, Xz, q, dP);
    double T[4];
    tmunu_row_emhd(Pz, fz, g.gam, q, dP, 0, T);
    double U[5];
    U[RHO] = (gd * Pz[RHO]) * fz.ucon[0];
    U[UU] = gd * (T[0] + Pz[RHO] * fz.ucon[0]);
    U[U1] = gd * T[1];
    U[U2] = gd * T[2];
    U[U3] = gd * T[3];
#pragma unroll
    for (int kk = 0; kk < 5; kk++) R[kk] = quotient(U[kk] - Us[kk], scale, iscale);
  }
  // Stores the solution from the root xs, or the guess; the zone's prims in
  // out.
  __device__ __forceinline__ void store(bool ok, const double xs[5], const double* __restrict__ Pin,
                                        const double* __restrict__ Xin, long nz, long c, double* __restrict__ Pout,
                                        double* __restrict__ Xout, unsigned long long* fails, double out[NVAR]) const {
    double xo[NXV];
    if (ok) {
      const double Pn[NVAR] = {xs[0], xs[1], xs[2], xs[3], xs[4], B[0], B[1], B[2]};
      Fluid<double> fz;
      fplain::fluid_state(Pn, m, fz);
      xsolve(fz, xo);
#pragma unroll
      for (int n = 0; n < NXV; n++)
        if (!isfinite(xo[n])) ok = false;
    }
    if (ok) {
#pragma unroll
      for (int v = 0; v < 5; v++) out[v] = xs[v];
    } else {
      load8(Pin, nz, c, out);
#pragma unroll
      for (int n = 0; n < NXV; n++) xo[n] = Xin[2 * c + n];
      atomicAdd(&fails[C_FAILS], 1ull);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) out[B1 + k] = B[k];
    store8(Pout, nz, c, out);
#pragma unroll
    for (int n = 0; n < NXV; n++) Xout[2 * c + n] = xo[n];
  }
};

// Zones whose Newton is still open after this many iterations go to the
// second kernel (64^3 torus, two steps: 2623 us with 3, 1892 with 4, 1632 with 5,
// 1721 with 6; 1951 in one kernel).
constexpr int EMHD_HEAD = 5;
struct OpenZone {
  int c, block;   // padded index; workgroup of the first kernel
};

// First kernel of the pass, a lane per zone.  Bound by FP64 arithmetic, some 30
// residuals per zone: shared reciprocals and the quotients without range
// handling took a residual from ~550 to ~300 instructions (64^3 torus: 387 -> 250
// us per launch).  Three waves per SIMD (168 registers) spill: 6 % slower step.
// A zone that has not converged after EMHD_HEAD iterations leaves its iterate in
// Pout and goes to the list (open, fails[C_OPEN] entries).  With RATE the
// CFL-rate partials of the new prims (ideal signal speeds), over the update's
// schedule.
template <int STAGE, bool RATE>
__global__ void __launch_bounds__(BLOCK)
k_implicit_emhd(Dev g, Sched box, const double* __restrict__ Pin, const double* __restrict__ Xin,
                const double* __restrict__ ustar, const double* __restrict__ xrhs,
                const double* __restrict__ divu, const double* __restrict__ utn, double* __restrict__ Pout,
                double* __restrict__ Xout, const double* __restrict__ tabC, double dt,
                const double* __restrict__ dt_dev, unsigned long long* fails,
                double* __restrict__ rate_partial, OpenZone* __restrict__ open) {
#pragma clang fp contract(off)
  __shared__ double jac[25 * BLOCK];
  int i, j, k;
  const bool in = sched_index(box, blockIdx.x, gridDim.x, i, j, k);
  if (dt_dev) dt = *dt_dev;
  double r = 0.0;
  if (in) {
    const long c = zid(g, i, j, k), nz = g.nz;
    ImplicitZone z;
    z.load(g, c, i, j, ustar, xrhs, divu, utn, tabC, STAGE == 1 ? 0.5 * dt : dt);
    double gs[NVAR], xs[5];
    load8(Pin, nz, c, gs);
    int how = NEWTON_FAILED;
    if (z.solvable())
      how = newton_hydro(g, gs, [&](const double xx[5], double R[5]) { z.residual(g, xx, R); }, xs, jac + threadIdx.x,
                         g.maxit < EMHD_HEAD ? g.maxit : EMHD_HEAD);
    double out[NVAR];
    if (how == NEWTON_OPEN) {
#pragma unroll
      for (int v = 0; v < 5; v++) Pout[vx(v, nz, c)] = xs[v];
      open[atomicAdd(&fails[C_OPEN], 1ull)] = OpenZone{(int)c, (int)blockIdx.x};
    } else {
      z.store(how == NEWTON_ROOT, xs, Pin, Xin, nz, c, Pout, Xout, fails, out);
      if (RATE) r = zone_rate_ordered(g, out, z.m);
    }
  }
  if (RATE) {
    double sm = 0.0;
    block_reduce(r, sm);
    if (threadIdx.x == 0) rate_partial[blockIdx.x] = r;
  }
}

// Second kernel: the listed zones, eight lanes each (newton_hydro_group).  A
// zone that does not converge runs to the iteration limit; with a lane per zone
// its chain of some 15 residuals an iteration set the time of the whole pass.
constexpr int EMHD_TAIL_BLOCKS = 512;
template <int STAGE, bool RATE>
__global__ void __launch_bounds__(BLOCK)
k_implicit_emhd_open(Dev g, const double* __restrict__ Pin, const double* __restrict__ Xin,
                     const double* __restrict__ ustar, const double* __restrict__ xrhs,
                     const double* __restrict__ divu, const double* __restrict__ utn, double* __restrict__ Pout,
                     double* __restrict__ Xout, const double* __restrict__ tabC, double dt,
                     const double* __restrict__ dt_dev, unsigned long long* fails,
                     double* __restrict__ rate_partial, const OpenZone* __restrict__ open) {
#pragma clang fp contract(off)
  __shared__ double jac[25 * BLOCK];
  const long n = (long)fails[C_OPEN], nz = g.nz;
  if (dt_dev) dt = *dt_dev;
  for (long e = (blockIdx.x * (long)BLOCK + threadIdx.x) >> 3; e < n; e += (long)EMHD_TAIL_BLOCKS * (BLOCK / 8)) {
    const OpenZone o = open[e];
    const long c = o.c;
    const int r = o.c / g.s1, i = o.c % g.s1 - NG, j = r % g.s2 - NG;
    ImplicitZone z;
    z.load(g, c, i, j, ustar, xrhs, divu, utn, tabC, STAGE == 1 ? 0.5 * dt : dt);
    double xs[5];
#pragma unroll
    for (int v = 0; v < 5; v++) xs[v] = Pout[vx(v, nz, c)];
    const int how = newton_hydro_group(g, [&](const double xx[5], double R[5]) { z.residual(g, xx, R); }, xs,
                                       jac + threadIdx.x, EMHD_HEAD);
    if ((threadIdx.x & 7u) == 0) {
      double out[NVAR];
      z.store(how == NEWTON_ROOT, xs, Pin, Xin, nz, c, Pout, Xout, fails, out);
      // (rates are not negative: their bits order as they do)
      if (RATE)
        atomicMax((unsigned long long*)rate_partial + o.block,
                  __builtin_bit_cast(unsigned long long, zone_rate_ordered(g, out, z.m)));
    }
  }
}
