// Hand-written adjoint (vector-Jacobian product) of one SSPRK2 step.
//
// The reverse sweep is written out stage by stage: the inversion is
// differentiated by the implicit-function theorem (lambda_U = (dU/dP)^-T
// lambda_P at the recovered prims; a zone whose inversion failed passes its
// hydro adjoint to the guess), the RK combination and flux divergence are
// transposed explicitly, Flux-CT is transposed through its edge EMFs, every
// face flux is transposed through its stencil, and ghost fills are transposed
// by gathering each ghost's adjoint back onto the zone it was copied from
// (with the polar sign flips).  The local derivatives of the per-point
// physics: a face flux with respect to its two states' prims by a reverse
// sweep through each state (face_vjp.hpp), chained with the reconstruction's
// derivatives with respect to each stencil slot (the WENO5 and MC gradients
// in closed form); the source and the conserved variables with respect to
// one zone's prims by a reverse sweep through the zone; the inversion's
// Jacobian by columns on one zone state.  Every sum is a gather in a fixed
// order: the result is deterministic.
//
// The internal arrays hold variables in pairs like the state (vx).
//
// Included inside the anonymous namespace of grmhd.hip.

template <int RECON>
struct Stencil {
  static constexpr int W = RECON == GRMHD_RECON_MC ? 4 : 6;  // zones per face
  static constexpr int H = W / 2;                            // zones left of the face
  static constexpr int NSLOT = NVAR * W;                     // stencil inputs of one face
};

#include "face_vjp.hpp"

// Adjoint of the Flux-CT EMFs on every padded edge position (zero outside
// the edge box [0, n]^3 and on polar edges), from the stage adjoint lambda_L
// of the field components (zero in ghost zones).  With the rebuilt fluxes
// Ft1(B2) = (E3 + E3_{j+1})/2 etc., lambda_Ft(face f) = (LL(f) - LL(f - e_d))/dx_d.
__global__ void __launch_bounds__(BLOCK) k_adj_emf(Dev g, const double* __restrict__ LL,
                                                   double* __restrict__ LE1, double* __restrict__ LE2,
                                                   double* __restrict__ LE3) {
  long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= g.nz) return;
  int i = (int)(t % g.s1) - NG;
  long r = t / g.s1;
  int j = (int)(r % g.s2) - NG, k = (int)(r / g.s2) - NG;
  if (i < 0 || j < 0 || k < 0 || i > g.n1 || j > g.n2 || k > g.n3) {
    LE1[t] = LE2[t] = LE3[t] = 0.0;
    return;
  }
  const long nz = g.nz, si = 1, sj = g.s1, sk = g.plane;
  auto lf = [&](int v, long f, long sd, double dx) { return (LL[vx(v, nz, f)] - LL[vx(v, nz, f - sd)]) / dx; };
  bool pole = (g.pole_lo && j == 0) || (g.pole_hi && j == g.n2);
  // E3 enters Ft1(B2) at faces (i,j),(i,j-1) with +1/2 and Ft2(B1) at (i,j),(i-1,j) with -1/2
  double e3 = 0.5 * (lf(B2, t, si, g.dx1) + lf(B2, t - sj, si, g.dx1)) -
              0.5 * (lf(B1, t, sj, g.dx2) + lf(B1, t - si, sj, g.dx2));
  // E2 enters Ft3(B1) at (i,k),(i-1,k) with +1/2 and Ft1(B3) at (i,k),(i,k-1) with -1/2
  double e2 = 0.5 * (lf(B1, t, sk, g.dx3) + lf(B1, t - si, sk, g.dx3)) -
              0.5 * (lf(B3, t, si, g.dx1) + lf(B3, t - sk, si, g.dx1));
  // E1 enters Ft2(B3) at (j,k),(j,k-1) with +1/2 and Ft3(B2) at (j,k),(j-1,k) with -1/2
  double e1 = 0.5 * (lf(B3, t, sj, g.dx2) + lf(B3, t - sk, sj, g.dx2)) -
              0.5 * (lf(B2, t, sk, g.dx3) + lf(B2, t - sj, sk, g.dx3));
  LE1[t] = pole ? 0.0 : e1;
  LE2[t] = e2;
  LE3[t] = pole ? 0.0 : e3;
}

// Per face of the forward flux box: the adjoint of the LLF flux (hydro slots
// from the divergence, field slots through the EMF averages), pushed through
// the face's two states by one reverse sweep each.  Returns the gamma part.
//
// MC: stores the adjoints of the two reconstructed states, gL in G's first 8
// nz values and gR in the next (16 values a face; the gather applies the
// limiter's derivatives, which are selections among its stencil's
// differences).  WENO5: the derivatives of a state with respect to its five
// slots cost more than reading them back, so the face applies them and stores
// the adjoint of each of its 8 x 6 stencil inputs, pair a of the variables and
// slot s at Pair index (a * W + s) * nz + face.
template <int D, int RECON>
__device__ __forceinline__ double adj_face(const Dev& g, const Box& box, long t, const double* __restrict__ P,
                                           const double* __restrict__ tab, const double* __restrict__ LL,
                                           const double* __restrict__ LE1, const double* __restrict__ LE2,
                                           const double* __restrict__ LE3, double* __restrict__ G) {
  using St = Stencil<RECON>;
  int i, j, k;
  if (!box_index(box, t, i, j, k)) return 0.0;
  const long c = zid(g, i, j, k), nz = g.nz, si = 1, sj = g.s1, sk = g.plane;
  const long s = D == 1 ? si : (D == 2 ? sj : sk);
  const double idx = D == 1 ? g.idx1 : (D == 2 ? g.idx2 : g.idx3);
  double lam[NVAR];
  {
    const Pair<double>* l = (const Pair<double>*)LL;
#pragma unroll
    for (int a = 0; a < 2; a++) {
      const Pair<double> x = l[a * nz + c], y = l[a * nz + c - s];
      lam[2 * a] = (x.a - y.a) * idx;
      lam[2 * a + 1] = (x.b - y.b) * idx;
    }
    lam[U3] = (LL[vx(U3, nz, c)] - LL[vx(U3, nz, c - s)]) * idx;
  }
  const double q = 0.25;
  if (D == 1) {
    lam[B1] = 0.0;
    lam[B2] = q * (LE3[c] + LE3[c + sj]);
    lam[B3] = -q * (LE2[c] + LE2[c + sk]);
  } else if (D == 2) {
    lam[B1] = -q * (LE3[c] + LE3[c + si]);
    lam[B2] = 0.0;
    lam[B3] = q * (LE1[c] + LE1[c + sk]);
  } else {
    lam[B1] = q * (LE2[c] + LE2[c + si]);
    lam[B2] = -q * (LE1[c] + LE1[c + sj]);
    lam[B3] = 0.0;
  }
  bool zero = true;
#pragma unroll
  for (int v = 0; v < NVAR; v++) zero = zero && lam[v] == 0.0;
  if (zero || (D == 2 && ((g.pole_lo && j == 0) || (g.pole_hi && j == g.n2)))) {
    const double none[NVAR] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int sd = 0; sd < (RECON == GRMHD_RECON_MC ? 2 : St::W); sd++)
      if constexpr (RECON == GRMHD_RECON_MC) {
        store8(G + sd * NVAR * nz, nz, c, none);
      } else {
        for (int a = 0; a < NVAR / 2; a++) ((Pair<double>*)G)[(a * St::W + sd) * nz + c] = Pair<double>{0.0, 0.0};
      }
    return 0.0;
  }
  PointMetric<double> m;
  load_metric<double>(tab, g.plane, pid(g, i, j), m);
  const double gam = g.gam;
  double qL[NVAR], qR[NVAR];
  recon_pair<RECON, double>(P, nz, c, s, g.weno_eps, qL, qR);
  // the LLF flux F = (FL + FR)/2 - cmax (UR - UL)/2 gives the adjoints
  // lambda/2 of FL and FR, +-cmax lambda/2 of UL and UR, and
  // -lambda.(UR - UL)/2 of cmax, which goes to the speed that attains it (the
  // left state's and the larger root's on ties)
  double cmax, cb = 0.0;
  bool right;
  {
    double UL[NVAR], UR[NVAR], cl, cr;
    ZoneState z;
    auto side = [&](const double* p, double* U) {
      zone_state(p, m, gam, z);
      zone_cons(p, z, m.gdet, U);
      const SpeedQuadratic r = speed_quadratic<D>(p, m, gam, z);
      return (fabs(r.b) + r.s) * fabs(face_rcp(r.A));
    };
    cl = side(qL, UL);
    cr = side(qR, UR);
    right = cr > cl;
    cmax = right ? cr : cl;
#pragma unroll
    for (int v = 0; v < NVAR; v++) cb = fma(lam[v], UR[v] - UL[v], cb);
    cb *= -0.5;
  }
  double Fb[NVAR];
#pragma unroll
  for (int v = 0; v < NVAR; v++) Fb[v] = 0.5 * lam[v];
  double gL[NVAR], gR[NVAR], gsum = 0.0;
  // one side at a time (a single copy of the sweep: shorter live ranges)
#pragma unroll 1
  for (int side = 0; side < 2; side++) {
    double qs[NVAR], Ub[NVAR], qb[NVAR], gamb;
    const double h = side == 0 ? cmax : -cmax;
#pragma unroll
    for (int v = 0; v < NVAR; v++) {
      qs[v] = side == 0 ? qL[v] : qR[v];
      Ub[v] = h * Fb[v];
    }
    face_state_vjp<D>(qs, m, gam, Fb, Ub, right == (side == 1) ? cb : 0.0, qb, gamb);
    gsum += gamb;
    if constexpr (RECON == GRMHD_RECON_MC) {
      store8(G + side * NVAR * nz, nz, c, qb);
    } else {
#pragma unroll
      for (int v = 0; v < NVAR; v++) {
        gL[v] = side == 0 ? qb[v] : gL[v];
        gR[v] = side == 1 ? qb[v] : gR[v];
      }
    }
  }
  if constexpr (RECON == GRMHD_RECON_WENO5) {
#pragma unroll 1
    for (int a = 0; a < NVAR / 2; a++) {
      Pair<double> qs[St::W], gl = {gL[0], gL[1]}, gr = {gR[0], gR[1]}, o[St::W];
#pragma unroll
      for (int z = 0; z < St::W; z++) qs[z] = ((const Pair<double>*)P)[a * nz + c + (z - St::H) * s];
#pragma unroll
      for (int u = 1; u < NVAR / 2; u++)   // compare and select: no register array indexed by a
        if (u == a) {
          gl = Pair<double>{gL[2 * u], gL[2 * u + 1]};
          gr = Pair<double>{gR[2 * u], gR[2 * u + 1]};
        }
      // the left state is weno5(q0, .., q4), the right one weno5(q5, .., q1)
      auto slots = [&](double x0, double x1, double x2, double x3, double x4, double x5, double l, double r,
                       double d[St::W]) {
        double e[5];
        weno5_grad(x0, x1, x2, x3, x4, g.weno_eps, d[0], d[1], d[2], d[3], d[4]);
        weno5_grad(x5, x4, x3, x2, x1, g.weno_eps, e[0], e[1], e[2], e[3], e[4]);
        d[5] = 0.0;
#pragma unroll
        for (int z = 0; z < St::W; z++) d[z] = fma(l, d[z], z == 0 ? 0.0 : r * e[5 - z]);
      };
      double da[St::W], db[St::W];
      slots(qs[0].a, qs[1].a, qs[2].a, qs[3].a, qs[4].a, qs[5].a, gl.a, gr.a, da);
      slots(qs[0].b, qs[1].b, qs[2].b, qs[3].b, qs[4].b, qs[5].b, gl.b, gr.b, db);
#pragma unroll
      for (int z = 0; z < St::W; z++) ((Pair<double>*)G)[(a * St::W + z) * nz + c] = Pair<double>{da[z], db[z]};
    }
  }
  return gsum;
}

// Sum of v over the workgroup, written to part[blockIdx.x].
__device__ __forceinline__ void store_block_sum(double v, double* __restrict__ part) {
  double mx = 0.0;
  block_reduce(mx, v);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

// The three directions' faces in one launch (one tail instead of three), nb1
// and nb2 workgroups of the first two; each XCD takes a contiguous range.  Two
// waves per SIMD (218 VGPRs with MC, 250 with WENO5, no scratch).  64^3 MC: 60
// us a stage, where three launches on dense sums, with divisions and 32 stored
// values a face, took 174; 111 MB written and some 90 MB read, about half the
// memory rate, the rest the arithmetic and latency of the two sweeps.
#ifndef ADJ_FACE_WAVES
#define ADJ_FACE_WAVES 2
#endif
template <int RECON>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(ADJ_FACE_WAVES, 8)))
k_adj_face(Dev g, Box b1, Box b2, Box b3, unsigned nb1, unsigned nb2, const double* __restrict__ P,
           const double* __restrict__ tabF1, const double* __restrict__ tabF2, const double* __restrict__ tabC,
           const double* __restrict__ LL, const double* __restrict__ LE1, const double* __restrict__ LE2,
           const double* __restrict__ LE3, double* __restrict__ G1, double* __restrict__ G2, double* __restrict__ G3,
           double* __restrict__ part) {
  const unsigned b = xcd_order(blockIdx.x, gridDim.x);
  double gs;
  if (b < nb1)
    gs = adj_face<1, RECON>(g, b1, b * (long)BLOCK + threadIdx.x, P, tabF1, LL, LE1, LE2, LE3, G1);
  else if (b < nb1 + nb2)
    gs = adj_face<2, RECON>(g, b2, (b - nb1) * (long)BLOCK + threadIdx.x, P, tabF2, LL, LE1, LE2, LE3, G2);
  else
    gs = adj_face<3, RECON>(g, b3, (b - nb1 - nb2) * (long)BLOCK + threadIdx.x, P, tabC, LL, LE1, LE2, LE3, G3);
  store_block_sum(gs, part);
}

// Faces along one axis that a padded zone's stencil adjoints come from.
struct AdjAxis {
  const double* G;
  long s;        // stride of the axis
  int x, n;      // the zone's coordinate along it, interior zones
  int lo, hi;    // faces of the box along it
  bool on;       // the zone's line of faces is in the box
};

// Pair a of the gathered adjoints along one axis: MC, from the adjoints of
// the two states per face (gL of zone c's stencil at its upper face, gR at
// its lower one).  With g+ = gL + gR and g- = gL - gR of zone c and the slope
// mc(c) = mc(q_{c-1}, q_c, q_{c+1}), the states c +- mc/2 give q_c the adjoint
// g+ and the slope's inputs g-/2 times its derivatives.
__device__ __forceinline__ void gather_mc(const AdjAxis& f, int a, long nz, long t, const Pair<double>* __restrict__ P,
                                          double& acc0, double& acc1) {
  const Pair<double>*GL = (const Pair<double>*)f.G + a * nz + t, *GR = GL + NVAR / 2 * nz;
  auto face = [&](const Pair<double>* G, int o) {
    const int x = f.x + o;
    return x >= f.lo && x <= f.hi ? G[o * f.s] : Pair<double>{0.0, 0.0};
  };
  Pair<double> q[5], gl[3], gr[3];
#pragma unroll
  for (int o = -2; o <= 2; o++) {
    int x = f.x + o;
    x = x < -NG ? -NG : (x > f.n + NG - 1 ? f.n + NG - 1 : x);
    q[o + 2] = P[a * nz + t + (x - f.x) * f.s];
  }
#pragma unroll
  for (int o = -1; o <= 1; o++) {
    gl[o + 1] = face(GL, o + 1);
    gr[o + 1] = face(GR, o);
  }
  auto sum = [&](double q0, double q1, double q2, double q3, double q4, double l0, double l1, double l2, double r0,
                 double r1, double r2) {
    double x, y, sr, sc, sl;
    mc_slope_grad(q0, q1, q2, x, y, sr);
    mc_slope_grad(q1, q2, q3, x, sc, y);
    mc_slope_grad(q2, q3, q4, sl, x, y);
    return (l1 + r1) + 0.5 * fma(sr, l0 - r0, fma(sc, l1 - r1, sl * (l2 - r2)));
  };
  acc0 += sum(q[0].a, q[1].a, q[2].a, q[3].a, q[4].a, gl[0].a, gl[1].a, gl[2].a, gr[0].a, gr[1].a, gr[2].a);
  acc1 += sum(q[0].b, q[1].b, q[2].b, q[3].b, q[4].b, gl[0].b, gl[1].b, gl[2].b, gr[0].b, gr[1].b, gr[2].b);
}
// WENO5: the zone is slot s of the face (H - s) zones further on.
__device__ __forceinline__ void gather_weno(const AdjAxis& f, int a, long nz, long t, double& acc0, double& acc1) {
  using St = Stencil<GRMHD_RECON_WENO5>;
#pragma unroll
  for (int s = 0; s < St::W; s++) {
    const int o = St::H - s, x = f.x + o;
    if (x < f.lo || x > f.hi) continue;
    const Pair<double> g = ((const Pair<double>*)f.G)[(a * St::W + s) * nz + t + o * f.s];
    acc0 += g.a;
    acc1 += g.b;
  }
}

// Gather of the stencil adjoints onto every padded zone.  Bound by memory (64^3
// MC: 45 us for 111 MB of state adjoints and the prims).  zero_ghosts, where
// given: an array in the caller's layout whose ghost zones are set to zero.
template <int RECON>
__global__ void __launch_bounds__(BLOCK) k_adj_gather(Dev g, const double* __restrict__ P,
                                                      const double* __restrict__ G1, const double* __restrict__ G2,
                                                      const double* __restrict__ G3, double* __restrict__ LPh,
                                                      double* __restrict__ zero_ghosts) {
  const long t = xcd_order(blockIdx.x, gridDim.x) * (long)BLOCK + threadIdx.x;
  if (t >= g.nz) return;
  const int i = (int)(t % g.s1) - NG;
  const long r = t / g.s1;
  const int j = (int)(r % g.s2) - NG, k = (int)(r / g.s2) - NG;
  auto in = [](int x, int n) { return x >= 0 && x < n; };
  auto near = [](int x, int n) { return x >= -1 && x <= n; };
  const AdjAxis f1 = {G1, 1, i, g.n1, 0, g.n1, near(j, g.n2) && near(k, g.n3)};
  const AdjAxis f2 = {G2, g.s1, j, g.n2, 0, g.n2, near(i, g.n1) && near(k, g.n3)};
  const AdjAxis f3 = {G3, g.plane, k, g.n3, 0, g.n3, near(i, g.n1) && near(j, g.n2)};
#pragma unroll 1
  for (int a = 0; a < NVAR / 2; a++) {
    double x = 0.0, y = 0.0;
    auto axis = [&](const AdjAxis& f) {
      if (!f.on) return;
      if constexpr (RECON == GRMHD_RECON_MC)
        gather_mc(f, a, g.nz, t, (const Pair<double>*)P, x, y);
      else
        gather_weno(f, a, g.nz, t, x, y);
    };
    axis(f1);
    axis(f2);
    axis(f3);
    ((Pair<double>*)LPh)[a * g.nz + t] = Pair<double>{x, y};
  }
  if (zero_ghosts && !(in(i, g.n1) && in(j, g.n2) && in(k, g.n3)))
    for (int v = 0; v < NVAR; v++) zero_ghosts[v * g.nz + t] = 0.0;
}

// Implicit-function adjoint of the inversion at the recovered prims p, state
// z: lambda_U = (dU/dP)^-T lambda_P, and -lambda_U . dU/dgamma (returned).
// The field rows of the Jacobian are sqrt(-g) on the diagonal (U_B = sqrt(-g)
// B, independent of the rest): J^T x = lp with J = sqrt(-g) [[Jh, Jb], [0, I]]
// is Jh^T y = lp_h, y = sqrt(-g) x_h (Gaussian elimination with partial
// pivoting, every index fixed at compile time so the system stays in
// registers), then x_B = (lp_B - Jb^T y) / sqrt(-g).
__device__ __forceinline__ double inversion_vjp(const double p[NVAR], const PointMetric<double>& m, double gam,
                                                const ZoneState& z, const double lp[NVAR], double x[NVAR]) {
  double A[5][5], y[5], J[5];
  const double ru = z.ut, ulu[4] = {z.ut * z.l0, z.ut * z.l1, z.ut * z.l2, z.ut * z.l3};
  // rows of Jh^T: along rho (dw = 1), u (dw = gam, dptot = gam - 1), u~
#pragma unroll
  for (int n = 0; n < 4; n++) {
    A[RHO][UU + n] = n == 0 ? ulu[0] + ru : ulu[n];
    A[UU][UU + n] = n == 0 ? fma(gam, ulu[0], gam - 1.0) : gam * ulu[n];
  }
  A[RHO][RHO] = ru;
  A[UU][RHO] = 0.0;
#pragma unroll
  for (int c = 1; c < 4; c++) cons_column_velocity(c, p, m, z, A[UU + c]);
#pragma unroll
  for (int a = 0; a < 5; a++) y[a] = lp[a];
#pragma unroll
  for (int col = 0; col < 5; col++) {
    int piv = col;
    double best = fabs(A[col][col]);
#pragma unroll
    for (int rr = col + 1; rr < 5; rr++)
      if (fabs(A[rr][col]) > best) {
        best = fabs(A[rr][col]);
        piv = rr;
      }
#pragma unroll
    for (int rr = col + 1; rr < 5; rr++)
      if (rr == piv) {
#pragma unroll
        for (int b = col; b < 5; b++) {
          const double tmp = A[col][b];
          A[col][b] = A[rr][b];
          A[rr][b] = tmp;
        }
        const double tmp = y[col];
        y[col] = y[rr];
        y[rr] = tmp;
      }
    const double ip = plain_rcp(A[col][col]);
#pragma unroll
    for (int rr = col + 1; rr < 5; rr++) {
      const double fct = quotient(A[rr][col], A[col][col], ip);
#pragma unroll
      for (int b = col + 1; b < 5; b++) A[rr][b] = fma(-fct, A[col][b], A[rr][b]);
      y[rr] = fma(-fct, y[col], y[rr]);
    }
    A[col][col] = ip;   // only its reciprocal is needed from here on
  }
#pragma unroll
  for (int rr = 4; rr >= 0; rr--) {
    double sum = y[rr];
#pragma unroll
    for (int b = rr + 1; b < 5; b++) sum = fma(-A[rr][b], y[b], sum);
    y[rr] = sum * A[rr][rr];
  }
  const double ig = plain_rcp(m.gdet);
#pragma unroll
  for (int c = 0; c < 3; c++) {
    cons_column_field(c + 1, p, m, z, J);
    double sum = lp[B1 + c];
#pragma unroll
    for (int a = 0; a < 5; a++) sum = fma(-J[a], y[a], sum);
    x[B1 + c] = sum * ig;
  }
  // along gamma: dw = dptot = u
  double gz = p[UU] * y[UU];
#pragma unroll
  for (int n = 0; n < 4; n++) gz = fma(p[UU] * ulu[n], y[UU + n], gz);
#pragma unroll
  for (int a = 0; a < 5; a++) x[a] = y[a] * ig;
  return -gz;
}

// The same of a zone: a zone whose inversion failed kept its guess's hydro
// prims, so lambda goes to the guess and only B^i = U_B^i / sqrt(-g) carries
// lambda to U.
__device__ __forceinline__ double zone_inversion_vjp(bool failed, const double p[NVAR], const PointMetric<double>& m,
                                                     double gam, const double lp[NVAR], double x[NVAR]) {
  if (failed) {
#pragma unroll
    for (int v = 0; v < NVAR; v++) x[v] = v < 5 ? 0.0 : lp[v] / m.gdet;
    return 0.0;
  }
  ZoneState z;
  zone_state(p, m, gam, z);
  return inversion_vjp(p, m, gam, z, lp, x);
}

// First kernel of the reverse sweep: the inversion adjoint at the step's
// result P (lambda_P = the caller's LP), through the transposed stage 2,
// U^{n+1} = V + (dt/2) L(P1): lambda_V = lambda_U, lambda_L = (dt/2) lambda_U.
// LL's ghost zones are set to zero (they stay so).
__global__ void __launch_bounds__(BLOCK) k_adj_ift(Dev g, const double* __restrict__ P,
                                                   const unsigned char* __restrict__ flags,
                                                   const double* __restrict__ tabC, const double* __restrict__ LP,
                                                   double dt, double* __restrict__ LV, double* __restrict__ LL,
                                                   double* __restrict__ part) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x, nz = g.nz;
  double gz = 0.0;
  if (t < nz) {
    const int i = (int)(t % g.s1) - NG;
    const long r = t / g.s1;
    const int j = (int)(r % g.s2) - NG, k = (int)(r / g.s2) - NG;
    double x[NVAR];
#pragma unroll
    for (int v = 0; v < NVAR; v++) x[v] = 0.0;
    if (i >= 0 && j >= 0 && k >= 0 && i < g.n1 && j < g.n2 && k < g.n3) {
      double lp[NVAR], p[NVAR];
#pragma unroll
      for (int v = 0; v < NVAR; v++) lp[v] = LP[v * nz + t];
      PointMetric<double> m;
      load_metric<double>(tabC, g.plane, pid(g, i, j), m);
      load8(P, nz, t, p);
      gz = zone_inversion_vjp(flags[t], p, m, g.gam, lp, x);
      store8(LV, nz, t, x);
#pragma unroll
      for (int v = 0; v < NVAR; v++) x[v] *= 0.5 * dt;
    }
    store8(LL, nz, t, x);
  }
  store_block_sum(gz, part);
}

// Zones along one axis whose ghost fill (or own value) comes from zone x:
// bit 0 the zone itself, bit 1 + l ghost l (0..2 below, 3..5 above); flip: the
// ones filled with the polar sign.
__device__ __forceinline__ unsigned adj_preimages(int x, int n, int lo, int hi, unsigned& flip) {
  flip = 0;
  unsigned m = 1;
  if (x >= NG && x < n - NG) return m;
#pragma unroll 1
  for (int l = 0; l < 2 * NG; l++) {
    bool f = false;
    if ((l < NG ? lo : hi) == GRMHD_BC_FROZEN) continue;
    if (bc_map(l < NG ? l - NG : n + l - NG, n, lo, hi, f) != x) continue;
    m |= 2u << l;
    if (f) flip |= 2u << l;
  }
  return m;
}
__device__ __forceinline__ int adj_preimage(int x, int n, int bit) {
  return bit == 0 ? x : (bit <= NG ? bit - 1 - NG : n + bit - 1 - NG);
}

// Per interior zone: the ghost-fill transpose of the gathered stencil
// adjoint, plus the local terms: source^T lambda_L, (stage 1) U^T lambda_U0,
// and the guess adjoint of a failed inversion (flags and LPout of the stage's
// result).  Stage 1 stores the adjoint of the step's input prims; stage 2
// passes its adjoint of P1 on through the inversion of stage 1 and the
// transposed combination U1 = U^n + dt L(P^n), V = (U^n + U1)/2: lambda_U1 =
// lambda_U + lambda_V/2, lambda_Un = lambda_V/2 + lambda_U1 (into LV),
// lambda_L = dt lambda_U1.  It stores its adjoint only where that inversion
// (failed1) failed: stage 1 reads it there.  64^3: 26 us, and 35 with the
// inversion (50 and 50 us before, as two kernels with the connection's 40
// coefficients, nine dual-number passes and preimage lists in scratch).
template <bool STAGE1>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_adj_zone(Dev g, Box box, const double* __restrict__ Pin, const unsigned char* __restrict__ flags,
           const unsigned char* __restrict__ failed1, const double* __restrict__ tabC,
           const double* __restrict__ dgs, double dt, const double* __restrict__ LPh,
           const double* __restrict__ LPout, double* __restrict__ LL, double* __restrict__ LV,
           double* __restrict__ LPin, double* __restrict__ part) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x, nz = g.nz;
  int i, j, k;
  double gz = 0.0;
  if (box_index(box, t, i, j, k)) {
    const long c = zid(g, i, j, k), q2 = pid(g, i, j);
    double acc[NVAR];
#pragma unroll
    for (int v = 0; v < NVAR; v++) acc[v] = 0.0;
    unsigned f1, f2, f3;
    const unsigned m1 = adj_preimages(i, g.n1, g.bc[0], g.bc[1], f1);
    const unsigned m2 = adj_preimages(j, g.n2, g.bc[2], g.bc[3], f2);
    const unsigned m3 = adj_preimages(k, g.n3, g.bc[4], g.bc[5], f3);
    for (unsigned a = m1; a; a &= a - 1)
      for (unsigned b = m2; b; b &= b - 1)
        for (unsigned e = m3; e; e &= e - 1) {
          const int x = __ffs(a) - 1, y = __ffs(b) - 1, w = __ffs(e) - 1;
          const bool flip = (((f1 >> x) ^ (f2 >> y) ^ (f3 >> w)) & 1u) != 0;
          double l[NVAR];
          load8(LPh, nz, zid(g, adj_preimage(i, g.n1, x), adj_preimage(j, g.n2, y), adj_preimage(k, g.n3, w)), l);
#pragma unroll
          for (int v = 0; v < NVAR; v++) acc[v] += (flip && (v == U2 || v == B2)) ? -l[v] : l[v];
        }
    PointMetric<double> m;
    load_metric<double>(tabC, g.plane, q2, m);
    double p[NVAR], lU[NVAR], qb[NVAR];
    load8(Pin, nz, c, p);
    if (STAGE1) load8(LV, nz, c, lU);
    zone_terms_vjp(p, m, g.gam, [&](int n) { return ((const Pair<double>*)dgs)[n * g.plane + q2]; },
                   LL[vx(U1, nz, c)], LL[vx(U2, nz, c)], STAGE1 ? lU : nullptr, qb, gz);
#pragma unroll
    for (int v = 0; v < NVAR; v++) acc[v] += qb[v];
    if (flags[c]) {
#pragma unroll
      for (int v = 0; v < 5; v++) acc[v] += LPout[v * nz + c];
    }
    if (STAGE1) {
#pragma unroll
      for (int v = 0; v < NVAR; v++) LPin[v * nz + c] = acc[v];
    } else {
      const bool failed = failed1[c];
      if (failed) {
#pragma unroll
        for (int v = 0; v < 5; v++) LPin[v * nz + c] = acc[v];
      }
      double x[NVAR];
      gz += zone_inversion_vjp(failed, p, m, g.gam, acc, x);
      load8(LV, nz, c, lU);
#pragma unroll
      for (int v = 0; v < NVAR; v++) {
        x[v] = fma(0.5, lU[v], x[v]);
        lU[v] = fma(0.5, lU[v], x[v]);
        x[v] *= dt;
      }
      store8(LV, nz, c, lU);
      store8(LL, nz, c, x);
    }
  }
  store_block_sum(gz, part);
}

// Per-block partial sums of n gamma parts.
__global__ void __launch_bounds__(BLOCK) k_adj_gsum(long n, const double* __restrict__ part, double* pmax,
                                                    double* psum) {
  double s = 0.0;
  const long stride = (long)gridDim.x * blockDim.x;
  for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < n; t += stride) s += part[t];
  double mx = 0.0;
  block_reduce(mx, s);
  if (threadIdx.x == 0) {
    pmax[blockIdx.x] = 0.0;
    psum[blockIdx.x] = s;
  }
}
