// The implicit solver's Newton iteration by eight lanes together.
//
// Included inside the anonymous namespace of grmhd.hip after inversion.hpp
// (and by a host test that runs the lanes in lockstep).

// newton_hydro's iteration continued from the iterate x (not converged after `from`
// iterations) by the eight lanes of a group together: lanes 0..4 take one
// column of the Jacobian each, and lane l the line search's step 2^-l; the
// first that reduces the residual is taken, as the steps one after the other
// would.  Per iteration the chain is three residuals instead of six to
// fourteen.  Every operation on a value is the one newton_hydro does, so the
// root is the same bit for bit.
template <typename Res>
__device__ __forceinline__ int newton_hydro_group(const Dev& g, Res res, double x[5], double* jac, int from) {
#pragma clang fp contract(off)
  const double fl[5] = {0.0, 0.0, 1e-3, 1e-3, 1e-3};
  const int lane = (int)(threadIdx.x & 63u), sub = lane & 7;
  double R[5];
  res(x, R);
  double r2 = 0.0;
#pragma unroll
  for (int k = 0; k < 5; k++) r2 += R[k] * R[k];
  bool conv = false;
  const double tol = g.tol > 1e-12 ? g.tol : 1e-12;
  const LdsMat J{jac};
  for (int it = from; it < g.maxit && !conv; it++) {
    double col[5];
    {
      const int k = sub < 5 ? sub : 0;
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
      for (int mm = 0; mm < 5; mm++) col[mm] = quotient(Rp[mm] - R[mm], hh, ihh);
    }
#pragma unroll
    for (int k = 0; k < 5; k++)
#pragma unroll
      for (int mm = 0; mm < 5; mm++) J(mm, k) = __shfl(col[mm], k, 8);
    double rhs[5], dx[5];
#pragma unroll
    for (int mm = 0; mm < 5; mm++) rhs[mm] = -R[mm];
    if (!qr_pivot_solve(J, x, rhs, dx)) return NEWTON_FAILED;
    double xn[5], Rn[5], rn2 = 0.0;
    bool ok = false;
    auto attempt = [&](double lam) {
#pragma unroll
      for (int mm = 0; mm < 5; mm++) {
        xn[mm] = x[mm] + lam * dx[mm];
        Rn[mm] = 0.0;
      }
      rn2 = 0.0;
      ok = xn[0] > 0.0 && xn[1] > 0.0;
      if (ok) {
        res(xn, Rn);
#pragma unroll
        for (int mm = 0; mm < 5; mm++) rn2 += Rn[mm] * Rn[mm];
        ok = isfinite(rn2);
      }
    };
    double lam = 1.0;
    for (int l = 0; l < sub; l++) lam = 0.5 * lam;
    attempt(lam);
    const unsigned good = (unsigned)(__ballot(ok && rn2 < r2) >> (lane & ~7)) & 255u;
    if (good) {
      const int from_lane = __ffs(good) - 1;
#pragma unroll
      for (int mm = 0; mm < 5; mm++) {
        xn[mm] = __shfl(xn[mm], from_lane, 8);
        Rn[mm] = __shfl(Rn[mm], from_lane, 8);
      }
      rn2 = __shfl(rn2, from_lane, 8);
    } else {
      attempt(0.00390625);   // the last step, 2^-8, taken if it is finite
      if (!ok) return NEWTON_FAILED;
    }
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
  if (!conv) return NEWTON_FAILED;
#pragma unroll
  for (int k = 0; k < 5; k++)
    if (!isfinite(x[k])) return NEWTON_FAILED;
  return NEWTON_ROOT;
}
