// Recovery of the primitive variables from the conserved ones, per zone:
// the 1D_W Newton solve, the Kastaun et al. bracketed recovery and the
// implicit solver's Newton-Raphson, with the dispatcher the update calls.
// Device code written so that it also compiles as plain C++ on the host
// (the sanitizer test builds it there): it uses only Dev's scalar fields,
// the per-point physics and <math.h>.
//
// Included inside the anonymous namespace of grmhd.hip.

// ---------------------------------------------------------------- U -> P --

// The conserved variables in the frame of the normal observer n_mu =
// (-alpha, 0, 0, 0): D = alpha U_rho/sqrt(-g), Q_mu = alpha T^t_mu, Bn^i =
// alpha B^i (B^i = U_B/sqrt(-g), into P), Q.n, Bn^2, Q.Bn, and the part of Q
// orthogonal to n, Qt^i = (g^{ij} + n^i n^j) Q_j.  Its square is taken as
// Q.Q + (Q.n)^2 with the rounded Q.n, whose error then cancels in what the
// residual forms from the two (Q_i Qt^i leaves u 15 % further from the exact
// root).  Metric entries that are identically zero (x2_offdiag, g^{t3}) are
// left out.
struct NormalFrame {
  double D, Qn, Qt2, QB, Bsq;
  double Bn[3], Qt[3];
};
__device__ __forceinline__ NormalFrame normal_frame(const PointMetric<double>& m, const double U[NVAR],
                                                    double P[NVAR]) {
#pragma clang fp contract(off)
  NormalFrame f;
  const double al = m.alpha, gd = m.gdet, igd = face_rcp(gd);
  auto dens = [&](double u) { return quotient(al * u, gd, igd); };
#pragma unroll
  for (int i = 0; i < 3; i++) {   // rounded: a field that does not change must not drift
    P[B1 + i] = quotient(U[B1 + i], gd, igd);
    f.Bn[i] = al * P[B1 + i];
  }
  f.D = dens(U[RHO]);
  const double Q0 = dens(U[UU] - U[RHO]), Q1 = dens(U[U1]), Q2 = dens(U[U2]), Q3 = dens(U[U3]);
  const double ctt = m.gcon[sidx(0, 0)], ct1 = m.gcon[sidx(0, 1)], c13 = m.gcon[sidx(1, 3)];
  const double n1 = -al * ct1, c11Q = m.gcon[sidx(1, 1)] * Q1 + c13 * Q3;
  f.Qn = fma(Q0, -al * ctt, Q1 * n1);
  f.Qt[0] = fma(n1 * n1, Q1, c11Q);
  f.Qt[1] = m.gcon[sidx(2, 2)] * Q2;
  f.Qt[2] = fma(c13, Q1, m.gcon[sidx(3, 3)] * Q3);
  const double QQ = Q0 * (ctt * Q0 + ct1 * Q1) + Q1 * (ct1 * Q0 + c11Q) + Q2 * f.Qt[1] + Q3 * f.Qt[2];
  f.Qt2 = fmax(QQ + f.Qn * f.Qn, 0.0);
  f.QB = fma(Q1, f.Bn[0], fma(Q2, f.Bn[1], Q3 * f.Bn[2]));
  f.Bsq = fma(m.gcov[sidx(1, 1)] * f.Bn[0], f.Bn[0],
              fma(m.gcov[sidx(2, 2)] * f.Bn[1], f.Bn[1],
                  fma(m.gcov[sidx(3, 3)] * f.Bn[2], f.Bn[2], 2.0 * (m.gcov[sidx(1, 3)] * f.Bn[0]) * f.Bn[2])));
  return f;
}

// 1D_W (Noble et al. 2006) Newton solve for W = w gamma^2.  Residual
//   Q.n + W - p(W) + Bn^2 (1 + v^2)/2 - (Q.Bn)^2/(2 W^2),
//   v^2 = [Qt^2 W^2 + (Q.Bn)^2 (Bn^2 + 2W)] / [(Bn^2 + W)^2 W^2],
//   p = (gam-1)/gam [W (1 - v^2) - D sqrt(1 - v^2)].
// Start from the guess's W (doubled while v^2 >= 1); steps leaving W > 0,
// v^2 < 1 are halved (at most 20 times); stop at |dW| < tol W or maxit, then
// one more step.  Returns 1 (and the guess's hydro prims) on failure.
// The iteration carries 1/W, 1/(W + Bn^2) and v^2 of its W, which the test of a
// step forms anyway: two reciprocals, one of the derivative and one square
// root per step, from the hardware estimates, where the written form has eight
// correctly rounded quotients.
__device__ int invert_1dw(const Dev& g, const PointMetric<double>& m, const double U[NVAR],
                          const double guess[NVAR], double P[NVAR]) {
#pragma clang fp contract(off)
  const double gam = g.gam, igam = face_rcp(gam), gf = quotient(gam - 1.0, gam, igam);
  const NormalFrame q = normal_frame(m, U, P);
  const double D = q.D, Bsq = q.Bsq, QB2 = q.QB * q.QB;

  struct Point {
    double W, iW, iWB, v2;
  };
  auto at = [&](double W) {
    Point x;
    x.W = W;
    x.iW = face_rcp(W);
    x.iWB = face_rcp(W + Bsq);
    const double r = x.iWB * x.iWB;
    x.v2 = r * fma(QB2 * fma(2.0, W, Bsq), x.iW * x.iW, q.Qt2);
    return x;
  };
  auto step = [&](const Point& x) {
    const double W = x.W, g2 = 1.0 - x.v2;
    double h;   // 1 / (2 sqrt(1 - v^2))
    const double sq = face_sqrt(g2, h);
    const double iW2 = x.iW * x.iW, qw = QB2 * iW2, qw3 = qw * x.iW;
    const double pr = gf * fma(W, g2, -(D * sq));
    const double f = fma(-0.5, qw, fma(0.5 * Bsq, 1.0 + x.v2, (q.Qn + W) - pr));
    const double poly = fma(3.0 * W, W + Bsq, Bsq * Bsq);
    const double dv2 = -2.0 * ((x.iWB * x.iWB) * x.iWB) * fma(qw3, poly, q.Qt2);
    const double dpdv2 = gf * fma(D, h, -W);
    const double df = fma(dv2, fma(0.5, Bsq, -dpdv2), fma(-gf, g2, 1.0) + qw3);
    return -f * face_rcp(df);
  };
  auto fail = [&]() {
#pragma unroll
    for (int v = 0; v < 5; v++) P[v] = guess[v];
    return 1;
  };

  const double g1 = guess[U1], g2 = guess[U2], g3 = guess[U3];
  const double qsq = fma(m.gcov[sidx(1, 1)] * g1, g1,
                         fma(m.gcov[sidx(2, 2)] * g2, g2,
                             fma(m.gcov[sidx(3, 3)] * g3, g3, 2.0 * (m.gcov[sidx(1, 3)] * g1) * g3)));
  Point x = at(fma(gam, guess[UU], guess[RHO]) * (1.0 + qsq));
  for (int b = 0; b < 60 && !(x.v2 < 1.0); b++) x = at(2.0 * x.W);
  bool conv = false;
  for (int it = 0; it < g.maxit; it++) {
    double dW = step(x);
    Point y = at(x.W + dW);
    for (int b = 0; b < 20 && !(y.W > 0.0 && y.v2 < 1.0); b++) {
      dW *= 0.5;
      y = at(x.W + dW);
    }
    if (!isfinite(y.W) || y.W <= 0.0) return fail();
    x = y;
    if (fabs(dW) < g.tol * fabs(x.W)) {
      conv = true;
      break;
    }
  }
  if (!conv) return fail();
  x = at(x.W + step(x));
  if (!isfinite(x.W) || x.W <= 0.0) return fail();
  if (!(x.v2 >= 0.0 && x.v2 < 1.0)) return fail();
  double h;
  const double w2 = 1.0 - x.v2, sq = face_sqrt(w2, h);   // 1/gamma
  const double rho = D * sq;
  const double u = quotient(fma(x.W, w2, -rho), gam, igam);
  if (!(rho > 0.0) || !(u > 0.0)) return fail();
  const double gi = h + h, gamma = fma(fma(-sq, gi, 1.0), gi, gi);
  const double pre = gamma * x.iWB, qbw = q.QB * x.iW;
  double ut[3];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    ut[i] = pre * fma(qbw, q.Bn[i], q.Qt[i]);
    if (!isfinite(ut[i])) return fail();
  }
  P[RHO] = rho;
  P[UU] = u;
  P[U1] = ut[0];
  P[U2] = ut[1];
  P[U3] = ut[2];
  return 0;
}

// Kastaun et al. (2021) recovery, the bracketed alternative to 1D_W (the
// Algorithm section names it among the robust inversions).  With D, the
// spatial projection S of Q and Bn as in 1D_W, scaled by D:
//   r^2 = S.S/D^2, b^2 = Bn.Bn/D, rb = S.Bn/D^(3/2), q = -Q.n/D - 1,
// all fluid quantities are functions of mu = 1/(h W):
//   x = 1/(1 + mu b^2), rbar^2 = x^2 r^2 + mu x (1 + x) rb^2,
//   qbar = q - b^2/2 - mu^2 x^2 (b^2 r^2 - rb^2)/2,
//   v^2 = min(mu^2 rbar^2, vmax^2), W = (1 - v^2)^(-1/2), rho = D/W,
//   eps = max(W (qbar - mu rbar^2) + v^2 W^2/(1 + W), 0),
//   a = (gam - 1) eps/(1 + eps),
//   nu = max((1 + a)(1 + eps)/W, (1 + a)(1 + qbar - mu rbar^2)),
// and mu solves mu = 1/(nu + mu rbar^2).  h >= 1 bounds mu by mu+, the root
// of mu sqrt(1 + rbar^2(mu)) = 1 (found first, to 1e-12, then widened by
// 1e-10); the root in [0, mu+] is bracketed and taken by the Illinois
// (modified regula falsi) iteration to |d mu| <= tol mu, at most 4 maxit
// iterations each.  No guess is used except as the failure value (the
// guess's hydro prims, as in 1D_W).  1 - v^2 loses W^2 to cancellation, so
// the frame and v^2 are rounded in the order of the CPU reference of the
// method (quotients by corrected reciprocals, nothing fused): the two then
// differ far less than either does from the exact root.
__device__ int invert_kastaun(const Dev& g, const PointMetric<double>& m, const double U[NVAR],
                              const double guess[NVAR], double P[NVAR]) {
#pragma clang fp contract(off)
  const double gam = g.gam;
  const double gd = m.gdet, igd = face_rcp(gd);
#pragma unroll
  for (int i = 0; i < 3; i++) P[B1 + i] = quotient(U[B1 + i], gd, igd);
  auto fail = [&]() {
#pragma unroll
    for (int v = 0; v < 5; v++) P[v] = guess[v];
    return 1;
  };
  const double al = m.alpha;
  const double D = quotient(al * U[RHO], gd, igd);
  if (!(D > 0.0) || !isfinite(D)) return fail();
  const double Q0 = al * (quotient(U[UU], gd, igd) - quotient(U[RHO], gd, igd)), Q1 = quotient(al * U[U1], gd, igd),
               Q2 = quotient(al * U[U2], gd, igd), Q3 = quotient(al * U[U3], gd, igd);
  const double Bn[3] = {al * P[B1], al * P[B2], al * P[B3]};
  const double ctt = m.gcon[sidx(0, 0)], ct1 = m.gcon[sidx(0, 1)], c13 = m.gcon[sidx(1, 3)];
  const double n0 = ctt * -al, n1 = ct1 * -al;
  const double Qu0 = ctt * Q0 + ct1 * Q1, Qu1 = ct1 * Q0 + m.gcon[sidx(1, 1)] * Q1 + c13 * Q3,
               Qu2 = m.gcon[sidx(2, 2)] * Q2, Qu3 = c13 * Q1 + m.gcon[sidx(3, 3)] * Q3;
  const double Qn = Q0 * n0 + Q1 * n1;
  const double QQ = Q0 * Qu0 + Q1 * Qu1 + Q2 * Qu2 + Q3 * Qu3;
  const double QB = Q1 * Bn[0] + Q2 * Bn[1] + Q3 * Bn[2];
  const double g13 = m.gcov[sidx(1, 3)];
  const double Bsq = m.gcov[sidx(1, 1)] * Bn[0] * Bn[0] + g13 * Bn[0] * Bn[2] + m.gcov[sidx(2, 2)] * Bn[1] * Bn[1] +
                     g13 * Bn[2] * Bn[0] + m.gcov[sidx(3, 3)] * Bn[2] * Bn[2];
  const double Ssq = fmax(QQ + Qn * Qn, 0.0);
  // (D^2 scaled to order one: it leaves the reciprocal's range long before D does)
  const double iD = face_rcp(D), DD = fmin(D * D, 0x1.fffffffffffffp1023), s2 = unit_scale(0.5 * DD), D2 = s2 * DD;
  double hD;
  const double D32 = D * face_sqrt(D, hD);   // (past FP64's range from D = 3e205 on)
  const double r2 = quotient(s2 * Ssq, D2, face_rcp(D2)), b2 = quotient(Bsq, D, iD),
               rb = isfinite(D32) ? quotient(QB, D32, face_rcp(D32)) : 0.0, q = quotient(-Qn, D, iD) - 1.0;
  const double rb2 = rb * rb, br = b2 * r2 - rb2;
  const double vmax2 = g.vmax2;
  const int maxit = 4 * g.maxit;

  struct St {
    double x, rbar2, iW, W, eps, f;
  };
  auto state = [&](double mu) {
    St s;
    s.x = face_rcp(1.0 + mu * b2);
    s.rbar2 = s.x * s.x * r2 + mu * s.x * (1.0 + s.x) * rb2;
    const double qbar = q - 0.5 * b2 - 0.5 * (mu * mu) * (s.x * s.x) * br;
    const double v2 = fmin(mu * mu * s.rbar2, vmax2);
    double h;   // 1 / (2 sqrt(1 - v^2))
    s.iW = face_sqrt(1.0 - v2, h);
    s.W = fma(fma(-s.iW, h + h, 1.0), h + h, h + h);
    const double W1 = 1.0 + s.W;
    s.eps = fmax(s.W * (qbar - mu * s.rbar2) + quotient(v2 * s.W * s.W, W1, face_rcp(W1)), 0.0);
    const double e1 = 1.0 + s.eps;
    const double a1 = 1.0 + quotient((gam - 1.0) * s.eps, e1, face_rcp(e1));
    const double nu = fmax(a1 * e1 * s.iW, a1 * (1.0 + qbar - mu * s.rbar2));
    s.f = mu - face_rcp(nu + mu * s.rbar2);
    return s;
  };
  auto f = [&](double mu) { return state(mu).f; };
  auto fa = [&](double mu) {
    const double x = face_rcp(1.0 + mu * b2);
    const double rbar2 = x * x * r2 + mu * x * (1.0 + x) * rb2;
    double h;
    return mu * face_sqrt(1.0 + rbar2, h) - 1.0;
  };
  // root of h in [lo, hi] with h(lo) < 0 <= h(hi); false after maxit steps
  auto illinois = [&](auto h, double lo, double hi, double hlo, double hhi, double tol, double& root) {
    int side = 0;
    double prev = hi;
    for (int it = 0; it < maxit; it++) {
      const double dh = hhi - hlo;
      double mid = quotient(lo * hhi - hi * hlo, dh, face_rcp(dh));
      if (!(mid > lo && mid < hi)) mid = 0.5 * (lo + hi);
      double hm = h(mid);
      if (hm == 0.0 || fabs(mid - prev) <= tol * mid) {
        root = mid;
        return true;
      }
      prev = mid;
      if (hm < 0.0) {
        lo = mid;
        hlo = hm;
        if (side == -1) hhi = 0.5 * hhi;
        side = -1;
      } else {
        hi = mid;
        hhi = hm;
        if (side == 1) hlo = 0.5 * hlo;
        side = 1;
      }
    }
    return false;
  };
  double mup;
  if (!illinois(fa, 0.0, 1.0, -1.0, fa(1.0), 1e-12, mup)) return fail();
  mup = fmin(mup * (1.0 + 1e-10), 1.0);
  const double f0 = f(0.0), f1 = f(mup);
  if (!(f0 < 0.0) || !(f1 >= 0.0)) return fail();
  double mu = mup;
  if (f1 != 0.0 && !illinois(f, 0.0, mup, f0, f1, g.tol, mu)) return fail();
  const St s = state(mu);
  const double rho = D * s.iW;
  const double u = rho * s.eps;
  // eps clamped at 0 stands when floors are on: the energy floor raises u
  if (!(rho > 0.0) || !(u > 0.0 || (g.floors && u == 0.0)) || !isfinite(u)) return fail();
  const double pre = quotient(s.W * mu * s.x, D, iD), mqd = mu * QB;
  const double Qt[3] = {Qu1 + n1 * Qn, Qu2, Qu3};
  double ut[3];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    ut[i] = pre * (Qt[i] + quotient(mqd * Bn[i], D, iD));
    if (!isfinite(ut[i])) return fail();
  }
  P[RHO] = rho;
  P[UU] = u;
  P[U1] = ut[0];
  P[U2] = ut[1];
  P[U3] = ut[2];
  return 0;
}

// The implicit solver's per-zone Newton-Raphson used as the recovery
// (Implicit Solver section: with every fluid variable implicit and only
// ideal sources it solves U(P) = U* zone by zone).  Unknowns x = (rho, u,
// u~1, u~2, u~3), B from U*; residual R(x) = (U(x) - U*)_{0..4} / s, s the
// largest |U*_k|; Jacobian by forward differences (secant) with steps
// h_k = 1e-7 max(|x_k|, f_k), f = (0, 0, 1e-3, 1e-3, 1e-3); the step from a
// Householder QR of J with column pivoting (largest remaining column norm
// first, ties to the lower index); backtracking line search lambda = 1,
// 1/2, ... (at most 8 halvings) until rho, u > 0 and |R| decreases (the last
// try is taken otherwise, if rho, u > 0); converged when every |lambda dx_k|
// <= max(tol, 1e-12) max(|x_k|, f_k) (near the root the residual's roundoff
// makes ~1e-13 steps), failure after maxit iterations or on non-finite
// values keeps the guess.  Unrolled so that the 5 x 5 system stays in
// registers (no dynamic indexing); same operation order as the CPU
// reference of the method, without contraction.
__device__ __forceinline__ void implicit_residual(const Dev& g, const PointMetric<double>& m, const double x[5],
                                                  const double B[3], const double Us[NVAR], double scale,
                                                  double R[5]) {
#pragma clang fp contract(off)
  const double P[NVAR] = {x[0], x[1], x[2], x[3], x[4], B[0], B[1], B[2]};
  Fluid<double> f;
  fluid_state(P, m, f);
  double U[NVAR];
  prim_to_flux(P, f, m, g.gam, 0, U);
#pragma unroll
  for (int k = 0; k < 5; k++) R[k] = (U[k] - Us[k]) / scale;
}

// A 5 x 5 matrix of one thread held in LDS: element (i, j) at
// base[(5 i + j) BLOCK], base = the workgroup's array + threadIdx.x, so the
// lanes of a wavefront touch consecutive words.  The Newton system lives
// here rather than in registers, which keeps the solver's register budget
// far from the per-wave limit.
struct LdsMat {
  double* base;
  __device__ __forceinline__ double& operator()(int i, int j) const { return base[(i * 5 + j) * BLOCK]; }
};

// TINY: columns may be so small that the square of one's norm is no normal
// number.
template <bool TINY>
__device__ __forceinline__ bool qr_pivot(const LdsMat& A, double b[5], double y[5]) {
#pragma clang fp contract(off)
  int perm[5] = {0, 1, 2, 3, 4};
  double cn[5];
#pragma unroll
  for (int j = 0; j < 5; j++) {
    cn[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 5; i++) cn[j] += A(i, j) * A(i, j);
  }
#pragma unroll
  for (int k = 0; k < 5; k++) {
    int best = k;
    double cb = cn[k];
#pragma unroll
    for (int j = k + 1; j < 5; j++)
      if (cn[j] > cb) {
        cb = cn[j];
        best = j;
      }
#pragma unroll
    for (int j = k + 1; j < 5; j++)
      if (j == best) {
#pragma unroll
        for (int i = 0; i < 5; i++) {
          const double t = A(i, k);
          A(i, k) = A(i, j);
          A(i, j) = t;
        }
        const double t = cn[k];
        cn[k] = cn[j];
        cn[j] = t;
        const int tp = perm[k];
        perm[k] = perm[j];
        perm[j] = tp;
      }
    double nrm = 0.0;
#pragma unroll
    for (int i = k; i < 5; i++) nrm += A(i, k) * A(i, k);
    nrm = plain_sqrt(nrm);
    if (!(nrm > 0.0) || !isfinite(nrm)) return false;
    const double alpha = A(k, k) > 0.0 ? -nrm : nrm;
    double v[5];
#pragma unroll
    for (int i = 0; i < 5; i++) v[i] = i < k ? 0.0 : A(i, k);
    v[k] = v[k] - alpha;
    // (the reflection is the same for any multiple of v)
    if (TINY) {
#pragma unroll
      for (int i = k; i < 5; i++) v[i] = nrm < 0x1p-500 ? 0x1p500 * v[i] : v[i];
    }
    double vv = 0.0;
#pragma unroll
    for (int i = k; i < 5; i++) vv += v[i] * v[i];
    if (!(vv > 0.0)) return false;
    const double ivv = plain_rcp(vv);
#pragma unroll
    for (int j = k; j < 5; j++) {
      double d = 0.0;
#pragma unroll
      for (int i = k; i < 5; i++) d += v[i] * A(i, j);
      const double f = quotient(2.0 * d, vv, ivv);
#pragma unroll
      for (int i = k; i < 5; i++) A(i, j) = A(i, j) - f * v[i];
    }
    double d = 0.0;
#pragma unroll
    for (int i = k; i < 5; i++) d += v[i] * b[i];
    const double f = quotient(2.0 * d, vv, ivv);
#pragma unroll
    for (int i = k; i < 5; i++) b[i] = b[i] - f * v[i];
#pragma unroll
    for (int j = k + 1; j < 5; j++) {
      cn[j] = 0.0;
#pragma unroll
      for (int i = k + 1; i < 5; i++) cn[j] += A(i, j) * A(i, j);
    }
  }
  double z[5];
#pragma unroll
  for (int i = 4; i >= 0; i--) {
    double t = b[i];
#pragma unroll
    for (int j = i + 1; j < 5; j++) t = t - A(i, j) * z[j];
    if (!(fabs(A(i, i)) > 0.0)) return false;
    z[i] = plain_div(t, A(i, i));
  }
#pragma unroll
  for (int mm = 0; mm < 5; mm++) {
    double val = 0.0;
#pragma unroll
    for (int k = 0; k < 5; k++)
      if (perm[k] == mm) val = z[k];
    y[mm] = val;
  }
#pragma unroll
  for (int k = 0; k < 5; k++)
    if (!isfinite(y[k])) return false;
  return true;
}

// The Newton step from the iterate x: the Jacobian's columns of rho and u are of
// the order of 1 / rho and 1 / u.
__device__ __forceinline__ bool qr_pivot_solve(const LdsMat& A, const double x[5], double b[5], double y[5]) {
  if (x[0] > 0x1p480 || x[1] > 0x1p480) return qr_pivot<true>(A, b, y);
  return qr_pivot<false>(A, b, y);
}

// jac: this thread's 25 LDS words for the Jacobian (LdsMat base).
__device__ __forceinline__ int invert_implicit(const Dev& g, const PointMetric<double>& m, const double U[NVAR],
                                               const double guess[NVAR], double P[NVAR], double* jac) {
#pragma clang fp contract(off)
  const double gd = m.gdet;
  P[B1] = U[B1] / gd;
  P[B2] = U[B2] / gd;
  P[B3] = U[B3] / gd;
  auto fail = [&]() {
#pragma unroll
    for (int v = 0; v < 5; v++) P[v] = guess[v];
    return 1;
  };
  const double B[3] = {P[B1], P[B2], P[B3]};
  double scale = 0.0;
#pragma unroll
  for (int k = 0; k < 5; k++)
    if (fabs(U[k]) > scale) scale = fabs(U[k]);
  if (!(scale > 0.0) || !isfinite(scale)) return fail();
  const double fl[5] = {0.0, 0.0, 1e-3, 1e-3, 1e-3};
  double x[5];
#pragma unroll
  for (int k = 0; k < 5; k++) x[k] = guess[k];
  if (!(x[0] > 0.0) || !(x[1] > 0.0)) return fail();
  double R[5];
  implicit_residual(g, m, x, B, U, scale, R);
  double r2 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; k++) r2 += R[k] * R[k];
  bool conv = false;
  const double tol = g.tol > 1e-12 ? g.tol : 1e-12;
  const LdsMat J{jac};
  for (int it = 0; it < g.maxit && !conv; it++) {
    // secant Jacobian, one column per pass (components picked by compare,
    // so nothing in registers is indexed by the loop counter)
#pragma unroll 1
    for (int k = 0; k < 5; k++) {
      double xk = x[0], flk = fl[0];
#pragma unroll
      for (int mm = 1; mm < 5; mm++)
        if (mm == k) {
          xk = x[mm];
          flk = fl[mm];
        }
      const double ax = fabs(xk);
      const double h = 1e-7 * (ax > flk ? ax : flk);
      const double xkh = xk + h;
      double xp[5];
#pragma unroll
      for (int mm = 0; mm < 5; mm++) xp[mm] = mm == k ? xkh : x[mm];
      double Rp[5];
      implicit_residual(g, m, xp, B, U, scale, Rp);
      const double hh = xkh - xk;
#pragma unroll
      for (int mm = 0; mm < 5; mm++) J(mm, k) = (Rp[mm] - R[mm]) / hh;
    }
    double rhs[5], dx[5];
#pragma unroll
    for (int mm = 0; mm < 5; mm++) rhs[mm] = -R[mm];
    if (!qr_pivot_solve(J, x, rhs, dx)) return fail();
    double lam = 1.0, xn[5], Rn[5], rn2 = 0.0;
    bool ok = false;
    for (int ls = 0; ls <= 8; ls++) {
#pragma unroll
      for (int mm = 0; mm < 5; mm++) xn[mm] = x[mm] + lam * dx[mm];
      if (xn[0] > 0.0 && xn[1] > 0.0) {
        implicit_residual(g, m, xn, B, U, scale, Rn);
        rn2 = 0.0;
#pragma unroll
        for (int mm = 0; mm < 5; mm++) rn2 += Rn[mm] * Rn[mm];
        ok = isfinite(rn2);
        if (ok && rn2 < r2) break;
      } else {
        ok = false;
      }
      if (ls < 8) lam = 0.5 * lam;
    }
    if (!ok) return fail();
    conv = true;
#pragma unroll
    for (int mm = 0; mm < 5; mm++) {
      const double ax = fabs(xn[mm]);
      if (fabs(xn[mm] - x[mm]) > tol * (ax > fl[mm] ? ax : fl[mm])) conv = false;
      x[mm] = xn[mm];
      R[mm] = Rn[mm];
    }
    r2 = rn2;
  }
  if (!conv) return fail();
#pragma unroll
  for (int k = 0; k < 5; k++) {
    if (!isfinite(x[k])) return fail();
    P[k] = x[k];
  }
  return 0;
}

// The implicit solver's Newton iteration on the five hydro prims x from the
// guess x0 (rho, u > 0), with the steps, Jacobian, pivoted QR, line search
// and stopping rule of invert_implicit: res(x, R) fills the scaled residual
// R[5]; jac is this thread's 25 LDS words for the Jacobian (LdsMat base).
// Returns NEWTON_ROOT with the root in x, or, after `limit` iterations of
// fewer than g.maxit, NEWTON_OPEN with the iterate.  (invert_implicit keeps its own copy of
// the loop: compiled through this template, its kernel produced different
// and wrong states on torus steps, while this template gives parity here.)
enum { NEWTON_FAILED = 0, NEWTON_ROOT = 1, NEWTON_OPEN = 2 };
template <typename Res>
__device__ __forceinline__ int newton_hydro(const Dev& g, const double x0[5], Res res, double x[5],
                                            double* jac, int limit) {
#pragma clang fp contract(off)
  const double fl[5] = {0.0, 0.0, 1e-3, 1e-3, 1e-3};
#pragma unroll
  for (int k = 0; k < 5; k++) x[k] = x0[k];
  if (!(x[0] > 0.0) || !(x[1] > 0.0)) return NEWTON_FAILED;
  double R[5];
  res(x, R);
  double r2 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; k++) r2 += R[k] * R[k];
  bool conv = false;
  const double tol = g.tol > 1e-12 ? g.tol : 1e-12;
  const LdsMat J{jac};
  for (int it = 0; it < limit && !conv; it++) {
    // secant Jacobian, one column per pass (components picked by compare,
    // so nothing in registers is indexed by the loop counter)
#pragma unroll 1
    for (int k = 0; k < 5; k++) {
      double xk = x[0], flk = fl[0];
#pragma unroll
      for (int mm = 1; mm < 5; mm++)
        if (mm == k) {
          xk = x[mm];
          flk = fl[mm];
        }
      const double ax = fabs(xk);
      const double h = 1e-7 * (ax > flk ? ax : flk);
      const double xkh = xk + h;
      double xp[5];
#pragma unroll
      for (int mm = 0; mm < 5; mm++) xp[mm] = mm == k ? xkh : x[mm];
      double Rp[5];
      res(xp, Rp);
      const double hh = xkh - xk, ihh = plain_rcp(hh);
#pragma unroll
      for (int mm = 0; mm < 5; mm++) J(mm, k) = quotient(Rp[mm] - R[mm], hh, ihh);
    }
    double rhs[5], dx[5];
#pragma unroll
    for (int mm = 0; mm < 5; mm++) rhs[mm] = -R[mm];
    if (!qr_pivot_solve(J, x, rhs, dx)) return NEWTON_FAILED;
    double lam = 1.0, xn[5], Rn[5], rn2 = 0.0;
    bool ok = false;
    for (int ls = 0; ls <= 8; ls++) {
#pragma unroll
      for (int mm = 0; mm < 5; mm++) xn[mm] = x[mm] + lam * dx[mm];
      if (xn[0] > 0.0 && xn[1] > 0.0) {
        res(xn, Rn);
        rn2 = 0.0;
#pragma unroll
        for (int mm = 0; mm < 5; mm++) rn2 += Rn[mm] * Rn[mm];
        ok = isfinite(rn2);
        if (ok && rn2 < r2) break;
      } else {
        ok = false;
      }
      if (ls < 8) lam = 0.5 * lam;
    }
    if (!ok) return NEWTON_FAILED;
    conv = true;
#pragma unroll
    for (int mm = 0; mm < 5; mm++) {
      const double ax = fabs(xn[mm]);
      if (fabs(xn[mm] - x[mm]) > tol * (ax > fl[mm] ? ax : fl[mm])) conv = false;
      x[mm] = xn[mm];
      R[mm] = Rn[mm];
    }
    r2 = rn2;
  }
  if (!conv) return limit < g.maxit ? NEWTON_OPEN : NEWTON_FAILED;
#pragma unroll
  for (int k = 0; k < 5; k++)
    if (!isfinite(x[k])) return NEWTON_FAILED;
  return NEWTON_ROOT;
}

__device__ __forceinline__ int invert(const Dev& g, const PointMetric<double>& m, const double U[NVAR],
                                      const double guess[NVAR], double P[NVAR]) {
  if (g.inverter == GRMHD_INV_KASTAUN) return invert_kastaun(g, m, U, guess, P);
  return invert_1dw(g, m, U, guess, P);
}

