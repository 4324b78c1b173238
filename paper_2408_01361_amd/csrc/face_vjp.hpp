// Reverse-mode derivatives for the adjoint, of one face state (its flux
// along D, conserved variables and two fast signal speeds) and of one zone's
// local terms (its geometric source and conserved variables): given the
// adjoints of those outputs, the adjoint of the prims q and of the adiabatic
// index.  One forward evaluation (zone_state), then one reverse sweep through
// it in the opposite order; and the Jacobian of the conserved variables, a
// column at a time.
//
// All of it on the library's structured metric (the entries that are
// identically zero are not in the sums), in terms of contractions with the
// output's adjoint -- a row T^mu_nu with adjoint X^nu needs X.u and X.b only --
// and with reciprocals that zone_state forms once; the speeds' sweep through
// their quadratic divides by its slope only.
//
// Included by adjoint.hpp (and by host tests) after physics.hpp, where the
// library's names are visible.
#pragma once

#pragma clang fp contract(off)

// Adjoints accumulated by the reverse sweeps: the four-velocity and the
// magnetic four-vector (both components), the fields, rho, u, the adiabatic
// index, w = rho + u + p + b^2, p + b^2/2, p and b^2.
struct FluidAdj {
  double u[4], l[4], b[4], k[4], B[3], rho, uu, gam, w, ptot, pg, bsq;
};
__device__ __forceinline__ void adj_zero(FluidAdj& a) {
#pragma unroll
  for (int x = 0; x < 4; x++) a.u[x] = a.l[x] = a.b[x] = a.k[x] = 0.0;
  a.B[0] = a.B[1] = a.B[2] = 0.0;
  a.rho = a.uu = a.gam = a.w = a.ptot = a.pg = a.bsq = 0.0;
}

// out_a += g_ab v^b
__device__ __forceinline__ void add_lowered(const PointMetric<double>& m, const double v[4], double out[4]) {
  const double gt1 = m.gcov[sidx(0, 1)], gt3 = m.gcov[sidx(0, 3)], g13 = m.gcov[sidx(1, 3)];
  out[0] += fma(m.gcov[sidx(0, 0)], v[0], fma(gt1, v[1], gt3 * v[3]));
  out[1] += fma(gt1, v[0], fma(m.gcov[sidx(1, 1)], v[1], g13 * v[3]));
  out[2] = fma(m.gcov[sidx(2, 2)], v[2], out[2]);
  out[3] += fma(gt3, v[0], fma(g13, v[1], m.gcov[sidx(3, 3)] * v[3]));
}

// Row e (u^e = ue, b^e = be) of sqrt(-g) (rho u^e, T^e_t + rho u^e, T^e_i),
// T^e_nu = w u^e u_nu + ptot delta^e_nu - b^e b_nu, with adjoints Y; X[e] is
// the entry that multiplies ptot.
__device__ __forceinline__ void adj_row(int e, const double Y[NVAR], double g, double rho, double ue, double be,
                                        const ZoneState& z, FluidAdj& a) {
  const double X[4] = {g * Y[UU], g * Y[U1], g * Y[U2], g * Y[U3]};
  const double rb = fma(g, Y[RHO], X[0]);   // adjoint of rho u^e
  const double xl = fma(X[0], z.l0, fma(X[1], z.l1, fma(X[2], z.l2, X[3] * z.l3)));
  const double xk = fma(X[0], z.k0, fma(X[1], z.k1, fma(X[2], z.k2, X[3] * z.k3)));
  const double wu = z.w * ue;
  a.rho = fma(rb, ue, a.rho);
  a.w = fma(ue, xl, a.w);
  a.u[e] += fma(rb, rho, z.w * xl);
  a.b[e] -= xk;
#pragma unroll
  for (int n = 0; n < 4; n++) {
    a.l[n] = fma(wu, X[n], a.l[n]);
    a.k[n] = fma(-be, X[n], a.k[n]);
  }
  a.ptot += X[e];
}

// The common tail of the reverse sweeps: from the adjoints of the state's
// quantities to those of the prims (qb) and of the adiabatic index (gamb).
__device__ __forceinline__ void fluid_rev(const double q[NVAR], const PointMetric<double>& m, double gam,
                                          const ZoneState& z, FluidAdj& a, double qb[NVAR], double& gamb) {
  const double Bp[3] = {q[B1], q[B2], q[B3]};
  const double u[4] = {z.ut, z.u1, z.u2, z.u3}, l[4] = {z.l0, z.l1, z.l2, z.l3};
  const double b[4] = {z.bt, z.b1, z.b2, z.b3}, k[4] = {z.k0, z.k1, z.k2, z.k3};
  // ptot = pg + bsq/2, w = rho + u + pg + bsq, pg = (gam - 1) u
  a.pg += a.ptot + a.w;
  a.bsq += fma(0.5, a.ptot, a.w);
  qb[RHO] = a.rho + a.w;
  qb[UU] = fma(a.pg, gam - 1.0, a.uu + a.w);
  gamb = fma(a.pg, q[UU], a.gam);
  // bsq = b^a b_a = g_ab b^a b^b (its two halves are equal), b_a = g_ab b^b
#pragma unroll
  for (int x = 0; x < 4; x++) a.b[x] = fma(2.0 * a.bsq, k[x], a.b[x]);
  add_lowered(m, a.k, a.b);
  // b^i = (B^i + bt u^i) / u^t, b^t = bt
  double bt_b = a.b[0];
#pragma unroll
  for (int i = 1; i < 4; i++) {
    const double f = a.b[i] * z.iut;
    a.B[i - 1] += f;
    bt_b = fma(f, u[i], bt_b);
    a.u[i] = fma(f, z.bt, a.u[i]);
    a.u[0] = fma(-f, b[i], a.u[0]);
  }
  // bt = B^i u_i
#pragma unroll
  for (int i = 1; i < 4; i++) {
    a.B[i - 1] = fma(bt_b, l[i], a.B[i - 1]);
    a.l[i] = fma(bt_b, Bp[i - 1], a.l[i]);
  }
  add_lowered(m, a.l, a.u);
  // u^t = gamma / alpha, u^1 = v^1 - gamma alpha g^{t1}; gamma =
  // sqrt(1 + g_ij v^i v^j)
  const double ia = inverse_lapse(m.alpha, m.gcon[sidx(0, 0)]);
  const double gb = fma(a.u[0], ia, -(a.u[1] * m.alpha) * m.gcon[sidx(0, 1)]);
  const double h = gb * (z.iut * ia);   // gamma_b / gamma
  const double g13 = m.gcov[sidx(1, 3)];
  qb[U1] = fma(h, fma(m.gcov[sidx(1, 1)], q[U1], g13 * q[U3]), a.u[1]);
  qb[U2] = fma(h, m.gcov[sidx(2, 2)] * q[U2], a.u[2]);
  qb[U3] = fma(h, fma(g13, q[U1], m.gcov[sidx(3, 3)] * q[U3]), a.u[3]);
  qb[B1] = a.B[0];
  qb[B2] = a.B[1];
  qb[B3] = a.B[2];
}

// The fast speeds along D: roots v = (b +- s)/A of A v^2 - 2 b v + C = 0 (the
// coefficients of fast_speed, with its power-of-two scale).
struct SpeedQuadratic {
  double A, b, C, s, m, sc;
};
template <int D>
__device__ __forceinline__ SpeedQuadratic speed_quadratic(const double q[NVAR], const PointMetric<double>& m,
                                                          double gam, const ZoneState& z) {
  const double ud = D == 1 ? z.u1 : (D == 2 ? z.u2 : z.u3);
  const double ctd = D == 1 ? m.gcon[sidx(0, 1)] : 0.0;
  const double n0 = fma(gam, z.pg, z.bsq);
  const double m0 = fma(gam * (2.0 - gam), q[UU], q[RHO]);
  SpeedQuadratic r;
  r.sc = unit_scale(n0 + m0);
  const double n = n0 * r.sc;
  r.m = m0 * r.sc;
  const double mut = r.m * z.ut;
  r.A = fma(mut, z.ut, -n * m.gcon[sidx(0, 0)]);
  r.b = fma(mut, ud, -n * ctd);
  r.C = fma(r.m * ud, ud, -n * m.gcon[sidx(D, D)]);
  const double disc = fma(r.b, r.b, -(r.A * r.C));
  double h;
  r.s = disc > 1e-280 ? face_sqrt(disc, h) : 0.0;
  return r;
}
// Adjoint vb of the root v = (b + sg s)/A: v follows from the quadratic, dv =
// -(v^2 dA - 2 v db + dC) / (2 sg s), where v^2 dA - 2 v db + dC =
// (v u^t - u^D)^2 dm + 2 m (v u^t - u^D)(v du^t - du^D) - (v^2 g^tt -
// 2 v g^tD + g^DD) dn.  A discriminant that is not positive counts as the
// constant zero (v = b/A).
template <int D>
__device__ __forceinline__ void speed_rev(const double q[NVAR], const PointMetric<double>& m, double gam,
                                          const ZoneState& z, const SpeedQuadratic& r, double sg, double vb,
                                          FluidAdj& a) {
  const double ud = D == 1 ? z.u1 : (D == 2 ? z.u2 : z.u3);
  const double ctt = m.gcon[sidx(0, 0)], ctd = D == 1 ? m.gcon[sidx(0, 1)] : 0.0, cdd = m.gcon[sidx(D, D)];
  const bool flat = !(r.s > 0.0);
  const double v = (r.b + sg * r.s) * face_rcp(r.A);
  const double kap = flat ? vb * face_rcp(r.A) : vb * face_rcp(-2.0 * sg * r.s);
  const double y = fma(v, z.ut, -ud), vt = fma(v, ctt, -ctd);
  const double mb = flat ? -y * z.ut : y * y;
  const double nb = flat ? vt : -fma(v, vt, fma(-v, ctd, cdd));
  const double tb = flat ? r.m * fma(-2.0 * v, z.ut, ud) : 2.0 * r.m * (v * y);
  const double db = flat ? r.m * z.ut : -2.0 * r.m * y;
  const double ks = kap * r.sc, mk = ks * mb, nk = ks * nb;
  a.u[0] = fma(kap, tb, a.u[0]);
  a.u[D] = fma(kap, db, a.u[D]);
  // n = gam p + b^2, m = rho + gam (2 - gam) u
  a.pg = fma(gam, nk, a.pg);
  a.bsq += nk;
  a.rho += mk;
  a.uu = fma(gam * (2.0 - gam), mk, a.uu);
  a.gam += fma(z.pg, nk, (2.0 - 2.0 * gam) * q[UU] * mk);
}

// Flux (row D, adjoint Fb) and conserved variables (row 0, Ub).
template <int D>
__device__ __forceinline__ void rows_rev(const double q[NVAR], const PointMetric<double>& m, const ZoneState& z,
                                         const double Fb[NVAR], const double Ub[NVAR], FluidAdj& a) {
  const double g = m.gdet;
  const double u[4] = {z.ut, z.u1, z.u2, z.u3}, b[4] = {z.bt, z.b1, z.b2, z.b3};
  adj_row(D, Fb, g, q[RHO], u[D], b[D], z, a);
  adj_row(0, Ub, g, q[RHO], z.ut, z.bt, z, a);
  // field slots: F[B_k] = g (b^k u^D - b^D u^k), U[B_k] = g B^k
#pragma unroll
  for (int k = 1; k < 4; k++) {
    if (k != D) {
      const double y = g * Fb[B1 + k - 1];
      a.b[k] = fma(y, u[D], a.b[k]);
      a.u[D] = fma(y, b[k], a.u[D]);
      a.b[D] = fma(-y, u[k], a.b[D]);
      a.u[k] = fma(-y, b[D], a.u[k]);
    }
    a.B[k - 1] = fma(g, Ub[B1 + k - 1], a.B[k - 1]);
  }
}

// One face state: flux along D (adjoint Fb), conserved variables (Ub) and
// the two fast speeds, the larger (cpb) and the smaller root (cmb).  (For the
// tests; the face kernel takes face_state_vjp below.)
template <int D>
__device__ __forceinline__ void state_vjp(const double q[NVAR], const PointMetric<double>& m, double gam,
                                          const double Fb[NVAR], const double Ub[NVAR], double cpb,
                                          double cmb, double qb[NVAR], double& gamb) {
  ZoneState z;
  zone_state(q, m, gam, z);
  FluidAdj a;
  adj_zero(a);
  const SpeedQuadratic r = speed_quadratic<D>(q, m, gam, z);
  const double sg = r.A < 0.0 ? -1.0 : 1.0;
  speed_rev<D>(q, m, gam, z, r, sg, cpb, a);
  speed_rev<D>(q, m, gam, z, r, -sg, cmb, a);
  rows_rev<D>(q, m, z, Fb, Ub, a);
  fluid_rev(q, m, gam, z, a, qb, gamb);
}

// The same with the adjoint vb of the speed of larger magnitude alone (the
// larger root on a tie): what a Lax-Friedrichs flux depends on.  That root is
// (b + sg s)/A with sg the sign of b, its own sign that of sg A: A is negative
// in states whose density or internal energy the reconstruction undershot.
template <int D>
__device__ __forceinline__ void face_state_vjp(const double q[NVAR], const PointMetric<double>& m, double gam,
                                               const double Fb[NVAR], const double Ub[NVAR], double vb,
                                               double qb[NVAR], double& gamb) {
  ZoneState z;
  zone_state(q, m, gam, z);
  FluidAdj a;
  adj_zero(a);
  const SpeedQuadratic r = speed_quadratic<D>(q, m, gam, z);
  const double sa = r.A < 0.0 ? -1.0 : 1.0;
  const double sg = r.b < 0.0 || (r.b == 0.0 && r.A < 0.0) ? -1.0 : 1.0;
  speed_rev<D>(q, m, gam, z, r, sg, sa * sg * vb, a);
  rows_rev<D>(q, m, z, Fb, Ub, a);
  fluid_rev(q, m, gam, z, a, qb, gamb);
}

// One zone: the geometric source (zone_source; adjoints S1b, S2b of its two
// components, d(n) the metric-derivative pair of entry n) and, when Ub is not
// null, the conserved variables (adjoint Ub).
template <typename Deriv>
__device__ __forceinline__ void zone_terms_vjp(const double q[NVAR], const PointMetric<double>& m, double gam, Deriv d,
                                               double S1b, double S2b, const double* Ub, double qb[NVAR],
                                               double& gamb) {
  ZoneState z;
  zone_state(q, m, gam, z);
  FluidAdj a;
  adj_zero(a);
  const double u[4] = {z.ut, z.u1, z.u2, z.u3}, b[4] = {z.bt, z.b1, z.b2, z.b3};
  const double y1 = m.gdet * S1b, y2 = m.gdet * S2b;
#pragma unroll
  for (int x = 0; x < 4; x++)
#pragma unroll
    for (int y = x; y < 4; y++) {
      if (x2_offdiag(sidx(x, y))) continue;
      const Pair<double> e = d(dgs_entry(sidx(x, y)));
      const double Tb = fma(y1, e.a, y2 * e.b), Tw = Tb * z.w;
      a.w = fma(Tb * u[x], u[y], a.w);
      if (!(x == 0 && y == 3)) a.ptot = fma(Tb, m.gcon[sidx(x, y)], a.ptot);
      a.u[x] = fma(Tw, u[y], a.u[x]);
      a.u[y] = fma(Tw, u[x], a.u[y]);
      a.b[x] = fma(-Tb, b[y], a.b[x]);
      a.b[y] = fma(-Tb, b[x], a.b[y]);
    }
  if (Ub) {
    adj_row(0, Ub, m.gdet, q[RHO], z.ut, z.bt, z, a);
#pragma unroll
    for (int k = 0; k < 3; k++) a.B[k] = fma(m.gdet, Ub[B1 + k], a.B[k]);
  }
  fluid_rev(q, m, gam, z, a, qb, gamb);
}

// The same from the connection, Gamma^l_{mn} at l * 10 + sidx(m, n), for
// sources of all four components (Sb; those along t and x3 vanish with the
// metric's derivatives): d_nu g_kl = g_km Gamma^m_{nu l} + g_lm Gamma^m_{nu k}.
// (For the tests, which have the connection's dual-number products.)
__device__ __forceinline__ void zone_vjp(const double q[NVAR], const PointMetric<double>& m, double gam,
                                         const double cn[40], const double Sb[4], const double* Ub,
                                         double qb[NVAR], double& gamb) {
  auto dg = [&](int nu, int k, int l) {
    double s = 0.0;
    for (int r = 0; r < 4; r++)
      s += m.gcov[sidx(k, r)] * cn[r * 10 + sidx(nu, l)] + m.gcov[sidx(l, r)] * cn[r * 10 + sidx(nu, k)];
    return k == l ? 0.5 * s : s;
  };
  Pair<double> e[NDGT / 2];
  for (int k = 0; k < 4; k++)
    for (int l = k; l < 4; l++)
      if (!x2_offdiag(sidx(k, l))) e[dgs_entry(sidx(k, l))] = Pair<double>{dg(1, k, l), dg(2, k, l)};
  zone_terms_vjp(q, m, gam, [&](int n) { return e[n]; }, Sb[1], Sb[2], Ub, qb, gamb);
}

// Columns of the Jacobian of the conserved variables' hydro rows, dU_a / dP_c
// over sqrt(-g): from the change of the state's quantities along one prim.
__device__ __forceinline__ void cons_column(const ZoneState& z, double rho, double drho, double dut, double dw,
                                            double dptot, const double dl[4], double dbt, const double dk[4],
                                            double J[5]) {
  const double dwu = fma(dw, z.ut, z.w * dut), wu = z.w * z.ut;
  const double dru = fma(drho, z.ut, rho * dut);
  const double l[4] = {z.l0, z.l1, z.l2, z.l3}, k[4] = {z.k0, z.k1, z.k2, z.k3};
  J[RHO] = dru;
#pragma unroll
  for (int n = 0; n < 4; n++) {
    const double t = fma(dwu, l[n], fma(wu, dl[n], -fma(dbt, k[n], z.bt * dk[n])));
    J[UU + n] = n == 0 ? t + dptot + dru : t;
  }
}
// Along the velocity u~^c, c = 1..3.
__device__ __forceinline__ void cons_column_velocity(int c, const double q[NVAR], const PointMetric<double>& m,
                                                     const ZoneState& z, double J[5]) {
  const double ia = inverse_lapse(m.alpha, m.gcon[sidx(0, 0)]);
  const double g13 = m.gcov[sidx(1, 3)];
  const double gv = c == 1   ? fma(m.gcov[sidx(1, 1)], q[U1], g13 * q[U3])
                    : c == 2 ? m.gcov[sidx(2, 2)] * q[U2]
                             : fma(g13, q[U1], m.gcov[sidx(3, 3)] * q[U3]);
  const double dg = gv * (z.iut * ia);   // (g v)_c / gamma
  double du[4] = {dg * ia, -(dg * m.alpha) * m.gcon[sidx(0, 1)], 0.0, 0.0};
  du[c] += 1.0;
  double dl[4] = {0.0, 0.0, 0.0, 0.0}, dk[4] = {0.0, 0.0, 0.0, 0.0};
  add_lowered(m, du, dl);
  const double dbt = fma(q[B1], dl[1], fma(q[B2], dl[2], q[B3] * dl[3]));
  const double u[4] = {z.ut, z.u1, z.u2, z.u3}, b[4] = {z.bt, z.b1, z.b2, z.b3};
  double db[4] = {dbt, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 1; i < 4; i++) db[i] = fma(dbt, u[i], fma(z.bt, du[i], -b[i] * du[0])) * z.iut;
  add_lowered(m, db, dk);
  const double hb = fma(db[0], z.k0, fma(db[1], z.k1, fma(db[2], z.k2, db[3] * z.k3)));   // d(b^2)/2
  cons_column(z, q[RHO], 0.0, du[0], 2.0 * hb, hb, dl, dbt, dk, J);
}
// Along the field B^c, c = 1..3.
__device__ __forceinline__ void cons_column_field(int c, const double q[NVAR], const PointMetric<double>& m,
                                                  const ZoneState& z, double J[5]) {
  const double u[4] = {z.ut, z.u1, z.u2, z.u3};
  const double dbt = c == 1 ? z.l1 : (c == 2 ? z.l2 : z.l3);
  double db[4] = {dbt, 0.0, 0.0, 0.0}, dk[4] = {0.0, 0.0, 0.0, 0.0};
  const double dl[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 1; i < 4; i++) db[i] = fma(dbt, u[i], i == c ? 1.0 : 0.0) * z.iut;
  add_lowered(m, db, dk);
  const double hb = fma(db[0], z.k0, fma(db[1], z.k1, fma(db[2], z.k2, db[3] * z.k3)));
  cons_column(z, q[RHO], 0.0, 0.0, 2.0 * hb, hb, dl, dbt, dk, J);
}
