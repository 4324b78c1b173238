// Per-point HARM physics for gfx950 in two arithmetics: double for the FP64
// path, float for the reduced-precision flux path.  Overloads on the
// argument type select between them.
//
//   * fluid four-vectors from the normal-observer velocity u~ (McKinney &
//     Gammie form the Algorithm section cites);
//   * rows of the ideal stress-energy tensor (EGRMHD section, ideal part);
//   * conserved variables / fluxes with the rest-mass energy removed;
//   * fast-magnetosonic characteristic speeds;
//   * linear-MC and WENO5 (Jiang-Shu weights) reconstruction.
#pragma once

#include <hip/hip_runtime.h>

#include "dual.hpp"

namespace grmhd {

enum { RHO = 0, UU = 1, U1 = 2, U2 = 3, U3 = 4, B1 = 5, B2 = 6, B3 = 7, NVAR = 8 };

// Symmetric 4x4 stored as 10 values: tt t1 t2 t3 11 12 13 22 23 33.
__host__ __device__ constexpr int sidx(int m, int n) {
  return (m < n ? m : n) == 0   ? (m < n ? n : m)
         : (m < n ? m : n) == 1 ? 3 + (m < n ? n : m)
         : (m < n ? m : n) == 2 ? 5 + (m < n ? n : m)
                                : 9;
}

// Geometry at one point, in the arithmetic type of the caller.
template <typename R>
struct PointMetric {
  R gcov[10];
  R gcon[10];
  R gdet;
  R alpha;
};

// Two neighbouring values, loaded and stored as one.  A vector memory
// instruction takes a CU 16 cycles for its 64 lanes whether they move 4, 8 or
// 16 bytes each (measured: 31 B per cycle with 8 bytes a lane, 63 with 16),
// and the flux kernel issued 60 of them per face row, more cycles than its
// arithmetic; so everything the kernels read together is stored in pairs.
template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

// State arrays (prims, stage registers, targets): variables 2q and 2q+1 of a
// zone next to each other, the pairs of one q over all nz padded zones.
__host__ __device__ constexpr long vx(int v, long nz, long c) { return ((long)(v >> 1) * nz + c) * 2 + (v & 1); }

template <typename R>
__device__ __forceinline__ void load8(const double* __restrict__ P, long nz, long c, R p[NVAR]) {
  const Pair<double>* q = (const Pair<double>*)P;
#pragma unroll
  for (int a = 0; a < NVAR / 2; a++) {
    const Pair<double> x = q[a * nz + c];
    p[2 * a] = (R)x.a;
    p[2 * a + 1] = (R)x.b;
  }
}
__device__ __forceinline__ void store8(double* __restrict__ P, long nz, long c, const double p[NVAR]) {
  Pair<double>* q = (Pair<double>*)P;
#pragma unroll
  for (int a = 0; a < NVAR / 2; a++) q[a * nz + c] = Pair<double>{p[2 * a], p[2 * a + 1]};
}

// Flux arrays of direction d = 1..3: the pairs (rho, u) and (u1, u2), then the
// two transverse field components, then u3 alone (the normal field has no
// flux).
__host__ __device__ constexpr int fslot(int d, int v) { return v - B1 < d - 1 ? v - B1 : v - B1 - 1; }
__host__ __device__ constexpr long fx(int d, int v, long nz, long c) {
  return v < U3 ? vx(v, nz, c) : (v == U3 ? 6 * nz + c : 4 * nz + 2 * c + fslot(d, v));
}
// stream: the launch's fluxes exceed the last-level cache (256 MB), so nothing
// of them is still there when the update reads them; stored past the L2 they
// leave it to the prims (128^3 WENO5, 10 steps: 10.17 -> 9.77 ms, 256^3 MC, 3
// steps: 22.6 -> 21.4; below that size they would be missed: 64^3
// production, 5 steps: 1.43 -> 1.45).
template <int D, typename FT>
__device__ __forceinline__ void store_flux(FT* __restrict__ F, long nz, long c, const FT f[NVAR], bool stream) {
  const FT ba = f[D == 1 ? B2 : B1], bb = f[D == 3 ? B2 : B3];
#ifdef __AMDGCN__
  if (stream) {
    typedef FT Vec2 __attribute__((ext_vector_type(2)));
    Vec2* q = (Vec2*)F;
    __builtin_nontemporal_store((Vec2){f[RHO], f[UU]}, q + c);
    __builtin_nontemporal_store((Vec2){f[U1], f[U2]}, q + nz + c);
    __builtin_nontemporal_store((Vec2){ba, bb}, q + 2 * nz + c);
    __builtin_nontemporal_store(f[U3], F + 6 * nz + c);
    return;
  }
#endif
  Pair<FT>* q = (Pair<FT>*)F;
  q[c] = Pair<FT>{f[RHO], f[UU]};
  q[nz + c] = Pair<FT>{f[U1], f[U2]};
  q[2 * nz + c] = Pair<FT>{ba, bb};
  F[6 * nz + c] = f[U3];
}
// The five hydro components; the field pair.
template <typename FT>
__device__ __forceinline__ void load_flux5(const FT* __restrict__ F, long nz, long c, double f[5]) {
  const Pair<FT>* q = (const Pair<FT>*)F;
  const Pair<FT> x = q[c], y = q[nz + c];
  f[RHO] = (double)x.a;
  f[UU] = (double)x.b;
  f[U1] = (double)y.a;
  f[U2] = (double)y.b;
  f[U3] = (double)F[6 * nz + c];
}
template <typename FT>
__device__ __forceinline__ Pair<FT> flux_field(const FT* __restrict__ F, long nz, long c) {
  return ((const Pair<FT>*)F)[2 * nz + c];
}

// Fields of a per-location geometry table: the entries that are not zero in
// the library's two spacetimes (below), ordered so that what is read together
// is paired; pairs over the padded (x1, x2) plane, so consecutive x1 columns
// are consecutive addresses.
enum {
  G_GTT, G_GT1, G_GT3, G_G33, G_G11, G_G13, G_G22, G_C22, G_CTT, G_CT1, G_DET, G_ALPHA, G_C11, G_C33, G_C13, G_SPARE,
  G_NF
};
__host__ __device__ constexpr long gx(int f, long plane, long q) { return vx(f, plane, q); }
enum { NCONN = 40 };  // Gamma^l_{mn}, m <= n
// Metric-derivative table of the geometric source: for nu = 1, 2 (row nu - 1)
// and each symmetric index s = (k, l), d_nu g_kl / 2 if k = l and d_nu g_kl if
// k < l (the pair (l, k) folded in), so that sum_s T^s D[s] = T^{kl} d_nu g_kl / 2.
// In the table the two derivatives of each of the seven entries that are not
// identically zero are a pair (dgs_entry gives its index).
enum { NDG = 20, NDGT = 14 };

// Both spacetimes of the library (flat space, and Kerr in modified
// Kerr-Schild coordinates) have g_{2 mu} = g^{2 mu} = 0 for mu != 2 -- x2 is
// orthogonal to the other coordinates -- and g^{t3} = 0.  Those seven entries
// are the constant zero rather than table fields, which gives the same values
// (and the same rounding of every expression that reads them) while keeping
// them out of registers.
__host__ __device__ constexpr bool x2_offdiag(int f) {
  return f == sidx(0, 2) || f == sidx(1, 2) || f == sidx(2, 3);
}

__host__ __device__ constexpr int dgs_entry(int s) {
  return s == sidx(0, 0) ? 0 : s == sidx(0, 1) ? 1 : s == sidx(0, 3) ? 2 : s == sidx(1, 1) ? 3
         : s == sidx(1, 3) ? 4 : s == sidx(2, 2) ? 5 : 6;
}

template <typename R>
__device__ __forceinline__ void load_metric(const double* __restrict__ tab, long plane, long q,
                                   PointMetric<R>& m) {
  const Pair<double>* t = (const Pair<double>*)tab;
  auto at = [&](int f) { return t[(f >> 1) * plane + q]; };
#pragma unroll
  for (int f = 0; f < 10; f++) m.gcov[f] = m.gcon[f] = (R)0;
  Pair<double> x = at(G_GTT);
  m.gcov[sidx(0, 0)] = (R)x.a;
  m.gcov[sidx(0, 1)] = (R)x.b;
  x = at(G_GT3);
  m.gcov[sidx(0, 3)] = (R)x.a;
  m.gcov[sidx(3, 3)] = (R)x.b;
  x = at(G_G11);
  m.gcov[sidx(1, 1)] = (R)x.a;
  m.gcov[sidx(1, 3)] = (R)x.b;
  x = at(G_G22);
  m.gcov[sidx(2, 2)] = (R)x.a;
  m.gcon[sidx(2, 2)] = (R)x.b;
  x = at(G_CTT);
  m.gcon[sidx(0, 0)] = (R)x.a;
  m.gcon[sidx(0, 1)] = (R)x.b;
  x = at(G_DET);
  m.gdet = (R)x.a;
  m.alpha = (R)x.b;
  x = at(G_C11);
  m.gcon[sidx(1, 1)] = (R)x.a;
  m.gcon[sidx(3, 3)] = (R)x.b;
  m.gcon[sidx(1, 3)] = (R)tab[gx(G_C13, plane, q)];
}

template <typename R>
struct Fluid {
  R ucon[4], ucov[4], bcon[4], bcov[4], bsq;
};

// FP64: every operation is rounded on its own, in the order written, so the
// face fluxes reproduce a plain evaluation of the same formulas; in flat
// space (exact metric constants) they agree with it bit for bit.
namespace f64 {
using R = double;
#pragma clang fp contract(off)
__device__ __forceinline__ R fdiv(R a, R b) { return a / b; }
#include "physics_body.inc"
}  // namespace f64

// FP32: contraction into fused multiply-adds allowed, fast divisions.
namespace f32 {
using R = float;
#pragma clang fp contract(fast)
__device__ __forceinline__ R fdiv(R a, R b) { return a * __builtin_amdgcn_rcpf(b); }
#include "physics_body.inc"
}  // namespace f32

// a / b from r = 1/b: correctly rounded but for rare ties.
__device__ __forceinline__ double quotient(double a, double b, double r) {
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// 1 / x to about an ulp.
__device__ __forceinline__ double face_rcp(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

__device__ __forceinline__ double hw_rsqrt(double x) {
#ifdef __AMDGCN__
  return __builtin_amdgcn_rsq(x);
#else
  return 1.0 / sqrt(x);
#endif
}

// FP64 quotient and square root without the scaling and the special cases of
// the correctly rounded ones: Newton's iteration for the reciprocal and
// Goldschmidt's for the root, from the hardware estimates, each closed by
// Markstein's correction with the residual in a fused multiply-add.  The same
// bits as the correctly rounded ones wherever no operand or intermediate is
// subnormal, infinite or NaN (a quotient by zero or infinity is NaN here).  A
// reciprocal shared by several quotients is formed once.
__device__ __forceinline__ double plain_rcp(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}
__device__ __forceinline__ double plain_div(double n, double d) { return quotient(n, d, plain_rcp(d)); }
__device__ __forceinline__ double plain_sqrt(double x) {
  const double y = hw_rsqrt(x), k = 0.5 * y;
  double g = x * y;
  const double r = fma(-k, g, 0.5);
  const double h = fma(k, r, k);
  g = fma(g, r, g);
  g = fma(fma(-g, g, x), h, g);
  g = fma(fma(-g, g, x), h, g);
  return x == 0.0 ? x : g;
}
// The per-point physics on them (Extended GRMHD).
namespace fplain {
using R = double;
#pragma clang fp contract(off)
__device__ __forceinline__ R fdiv(R a, R b) { return plain_div(a, b); }
__device__ __forceinline__ R sqrt(R x) { return plain_sqrt(x); }
#include "physics_body.inc"
}  // namespace fplain

// Dual numbers: the derivatives that the adjoint's reverse sweeps are tested
// against.
namespace fdual {
using R = Dual;
__device__ __forceinline__ R fdiv(R a, R b) { return a / b; }
__device__ __forceinline__ R fdiv(R a, double b) { return a / b; }
#include "physics_body.inc"
}  // namespace fdual

using f64::lower4;
using f32::lower4;
using fdual::lower4;
using f64::fluid_state;
using f32::fluid_state;
using fdual::fluid_state;
using f64::tmunu_row;
using f32::tmunu_row;
using fdual::tmunu_row;
using f64::metric_source;
using fdual::metric_source;
using f64::prim_to_flux;
using f32::prim_to_flux;
using fdual::prim_to_flux;
using f64::char_speeds;
using f32::char_speeds;
using fdual::char_speeds;
using f64::mc_slope;
using f32::mc_slope;
using fdual::mc_slope;
using f64::mc_left;
using f32::mc_left;
using fdual::mc_left;
using f64::mc_right;
using f32::mc_right;
using fdual::mc_right;
using f64::vl_left;
using f32::vl_left;
using f64::vl_right;
using f32::vl_right;
using f64::mp5;
using f32::mp5;
using f64::ppm_edges;
using f32::ppm_edges;
using f64::ppmx_edges;
using f32::ppmx_edges;

// WENO5 (Jiang-Shu weights d_k / (eps + beta_k)^2, d = (1, 6, 3)/10) from
// point values a..e of zones c-2..c+2: the value at the right edge of zone c.
// The FP64 form works on the four differences of the stencil: the second
// differences t_k and one-sided slopes u_k of the smoothness indicators and
// the candidates' offsets from c are short sums of them, and the edge value
// is c plus the weighted offset, so only that offset goes through the
// normalising quotient.  Reversing the stencil negates and swaps the
// differences exactly, so a zone's left-edge value, weno5(e, d, c, b, a),
// reuses its right edge's indicators and weight products bit for bit
// (weno5_pair).  Arranged for few operations: every indicator is scaled by 4
// (4 beta_k = (13/3) t_k^2 + u_k^2, with 4 eps), which leaves the weights
// unchanged; the factors 1/10 of d and 1/6 of the candidate polynomials
// cancel or move into the final fused multiply-add.  58 FP64 operations and
// two hardware reciprocals per edge pair, against 75 for the form on the
// zone values.
//
// FP64: only the fused multiply-adds written out (contraction off), so an
// evaluation rounds the same way in whatever code it is inlined; the
// normalising quotient comes from the hardware reciprocal (relative error
// below 2^-23) with the two leading terms of its error series (within about
// an ulp of the offset; the weights' denominator is a sum of positive normal
// numbers for weno_eps >= 1e-36).
#pragma clang fp contract(off)
namespace wd {
typedef double R;
// n / d: with e = 1 - d r of the hardware estimate r, 1/d = r (1 + e + e^2 + ..)
__device__ __forceinline__ R qdiv(R n, R d) {
  const R r = __builtin_amdgcn_rcp(d);
  const R e = fma(-d, r, (R)1);
  const R q = n * r;
  return fma(q, fma(e, e, e), q);
}
// Differences of the stencil and 4 (eps + beta) of (a, b, c), (b, c, d),
// (c, d, e).
struct Stencil5 {
  R d1, d2, d3, d4, s0, s1, s2;
};
__device__ __forceinline__ Stencil5 stencil5(R a, R b, R c, R d, R e, R eps) {
  Stencil5 z;
  const R eps4 = (R)4 * eps, k = (R)(13.0 / 3.0);
  z.d1 = b - a;
  z.d2 = c - b;
  z.d3 = d - c;
  z.d4 = e - d;
  const R t0 = z.d2 - z.d1, u0 = fma((R)3, z.d2, -z.d1);
  const R t1 = z.d3 - z.d2, u1 = z.d2 + z.d3;
  const R t2 = z.d4 - z.d3, u2 = fma((R)3, z.d3, -z.d4);
  z.s0 = fma(k * t0, t0, fma(u0, u0, eps4));
  z.s1 = fma(k * t1, t1, fma(u1, u1, eps4));
  z.s2 = fma(k * t2, t2, fma(u2, u2, eps4));
  return z;
}
// c + offset / 6 of the candidates' offsets (5 d2 - 2 d1, d2 + 2 d3,
// 4 d3 - d4) with weights w0, c6, 3 w2 over their sum (c6 = 6 times the middle
// product)
__device__ __forceinline__ R combine(R c, R d1, R d2, R d3, R d4, R w0, R c6, R w2) {
  const R p0 = fma((R)5, d2, (R)-2 * d1);
  const R p1 = fma((R)2, d3, d2);
  const R p2 = fma((R)4, d3, -d4);
  const R v2 = (R)3 * w2;
  return fma((R)(1.0 / 6.0), qdiv(fma(w0, p0, fma(c6, p1, v2 * p2)), (w0 + c6) + v2), c);
}
// Right and left edge from the weight products w0 = s1 s2, w1 = s0 s2,
// w2 = s0 s1 (of squared indicators).
__device__ __forceinline__ R right_edge(const Stencil5& z, R c, R w0, R w1, R w2) {
  return combine(c, z.d1, z.d2, z.d3, z.d4, w0, (R)6 * w1, w2);
}
__device__ __forceinline__ R left_edge(const Stencil5& z, R c, R w0, R w1, R w2) {
  return combine(c, -z.d4, -z.d3, -z.d2, -z.d1, w2, (R)6 * w1, w0);
}
}  // namespace wd

__device__ __forceinline__ double weno5(double a, double b, double c, double d, double e, double eps) {
  const wd::Stencil5 z = wd::stencil5(a, b, c, d, e, eps);
  const double q0 = z.s0 * z.s0, q1 = z.s1 * z.s1, q2 = z.s2 * z.s2;
  return wd::right_edge(z, c, q1 * q2, q0 * q2, q0 * q1);
}

// Both edges of zone c: left = weno5(e, d, c, b, a), right = weno5(a, b, c,
// d, e), from one set of indicators (reversing the stencil swaps s0 and s2).
__device__ __forceinline__ void weno5_pair(double a, double b, double c, double d, double e, double eps,
                                           double& left, double& right) {
  const wd::Stencil5 z = wd::stencil5(a, b, c, d, e, eps);
  const double q0 = z.s0 * z.s0, q1 = z.s1 * z.s1, q2 = z.s2 * z.s2;
  const double w0 = q1 * q2, w1 = q0 * q2, w2 = q0 * q1;
  right = wd::right_edge(z, c, w0, w1, w2);
  left = wd::left_edge(z, c, w0, w1, w2);
}

// WENO-Z (Borges et al. 2008, power 2 as in Castro, Costa & Don 2011): the
// WENO5 candidates and indicators with weights d_k (1 + (tau5 / (eps +
// beta_k))^2), tau5 = |beta_0 - beta_2|.  Over the common denominator of the
// squared indicators s_k = (4 (eps + beta_k))^2 (tau5 scaled by 4 alike,
// T = (4 tau5)^2) the weight products are d_k (s_k + T) prod_{j != k} s_j,
// formed like WENO5's; with weno_eps >= 1e-36 they stay normal while
// 4 (eps + beta) < 1e100, i.e. for differences of primitives below ~1e49.
__device__ __forceinline__ double wenoz(double a, double b, double c, double d, double e, double eps) {
  const wd::Stencil5 z = wd::stencil5(a, b, c, d, e, eps);
  const double tau = fabs(z.s0 - z.s2), T = tau * tau;
  const double q0 = z.s0 * z.s0, q1 = z.s1 * z.s1, q2 = z.s2 * z.s2;
  return wd::right_edge(z, c, (q0 + T) * (q1 * q2), (q1 + T) * (q0 * q2), (q2 + T) * (q0 * q1));
}

// FP32 forms: contraction into fused multiply-adds allowed.
#pragma clang fp contract(fast)

// FP32 form.  The indicators are scaled by 12 as in the FP64 form and then
// normalised by the smallest one, r_k = s_k / min s in [1, 1e6] (clamped:
// a stencil 1e6 times rougher than the smoothest keeps a relative weight
// below 1e-12 either way, under FP32 resolution); the weights d_k / r_k^2 are
// formed over the common denominator as in the FP64 form, so the products
// stay below 1e25 (no overflow, no 0/0), and the two divisions are hardware
// reciprocals (v_rcp_f32).
namespace wf {
typedef float R;
__device__ __forceinline__ R weno5(R a, R b, R c, R d, R e, R eps) {
  const R eps12 = 12.0f * eps;
  R t0 = (a + c) - 2.0f * b, u0 = fmaf(-4.0f, b, fmaf(3.0f, c, a));
  R t1 = (b + d) - 2.0f * c, u1 = b - d;
  R t2 = (c + e) - 2.0f * d, u2 = fmaf(-4.0f, d, fmaf(3.0f, c, e));
  R s0 = fmaf(13.0f * t0, t0, fmaf(3.0f * u0, u0, eps12));
  R s1 = fmaf(13.0f * t1, t1, fmaf(3.0f * u1, u1, eps12));
  R s2 = fmaf(13.0f * t2, t2, fmaf(3.0f * u2, u2, eps12));
  const R im = __builtin_amdgcn_rcpf(fminf(fminf(s0, s1), s2));
  R r0 = fminf(s0 * im, 1e6f), r1 = fminf(s1 * im, 1e6f), r2 = fminf(s2 * im, 1e6f);
  r0 *= r0;
  r1 *= r1;
  r2 *= r2;
  R p0 = fmaf(11.0f, c, fmaf(-7.0f, b, 2.0f * a));
  R p1 = fmaf(2.0f, d, fmaf(5.0f, c, -b));
  R p2 = fmaf(5.0f, d, fmaf(2.0f, c, -e));
  R w0 = r1 * r2, w1 = 6.0f * (r0 * r2), w2 = 3.0f * (r0 * r1);
  return fmaf(w0, p0, fmaf(w1, p1, w2 * p2)) * __builtin_amdgcn_rcpf(6.0f * ((w0 + w1) + w2));
}
}  // namespace wf

__device__ __forceinline__ float weno5(float a, float b, float c, float d, float e, float eps) {
  return wf::weno5(a, b, c, d, e, eps);
}

// FP32 form of weno5_pair (the normalised indicators are symmetric too).
namespace wf {
__device__ __forceinline__ R wcomb(R a, R b, R c, R d, R e, R w0, R w1, R w2) {
  R p0 = fmaf(11.0f, c, fmaf(-7.0f, b, 2.0f * a));
  R p1 = fmaf(2.0f, d, fmaf(5.0f, c, -b));
  R p2 = fmaf(5.0f, d, fmaf(2.0f, c, -e));
  return fmaf(w0, p0, fmaf(w1, p1, w2 * p2)) * __builtin_amdgcn_rcpf(6.0f * ((w0 + w1) + w2));
}
__device__ __forceinline__ void weno5_pair(R a, R b, R c, R d, R e, R eps, R& left, R& right) {
  const R eps12 = 12.0f * eps;
  R t0 = (a + c) - 2.0f * b, u0 = fmaf(-4.0f, b, fmaf(3.0f, c, a));
  R t1 = (b + d) - 2.0f * c, u1 = b - d;
  R t2 = (c + e) - 2.0f * d, u2 = fmaf(-4.0f, d, fmaf(3.0f, c, e));
  R s0 = fmaf(13.0f * t0, t0, fmaf(3.0f * u0, u0, eps12));
  R s1 = fmaf(13.0f * t1, t1, fmaf(3.0f * u1, u1, eps12));
  R s2 = fmaf(13.0f * t2, t2, fmaf(3.0f * u2, u2, eps12));
  const R im = __builtin_amdgcn_rcpf(fminf(fminf(s0, s1), s2));
  R r0 = fminf(s0 * im, 1e6f), r1 = fminf(s1 * im, 1e6f), r2 = fminf(s2 * im, 1e6f);
  r0 *= r0;
  r1 *= r1;
  r2 *= r2;
  const R r12 = r1 * r2, r02 = r0 * r2, r01 = r0 * r1;
  right = wcomb(a, b, c, d, e, r12, 6.0f * r02, 3.0f * r01);
  left = wcomb(e, d, c, b, a, r01, 6.0f * r02, 3.0f * r12);
}
}  // namespace wf

__device__ __forceinline__ void weno5_pair(float a, float b, float c, float d, float e, float eps,
                                           float& left, float& right) {
  wf::weno5_pair(a, b, c, d, e, eps, left, right);
}

// FP32 WENO-Z.  With b_k = 12 (eps + beta_k), rho_k = b_k / min b >= 1 and
// theta = 12 tau5 / min b (clamped at 1e18; beyond it the weights agree
// with the clamped ones to FP32 resolution), the weights divided by the
// common factor 1 + theta^2 are d_k (e + q / rho_k^2), e = 1 / (1 + theta^2),
// q = theta^2 e: each in (0, d_k], the smoothest stencil's equal to d_k, so
// nothing overflows and the sum never vanishes.  Hardware reciprocals.
namespace wf {
__device__ __forceinline__ R wenoz(R a, R b, R c, R d, R e, R eps) {
  const R eps12 = 12.0f * eps;
  R t0 = (a + c) - 2.0f * b, u0 = fmaf(-4.0f, b, fmaf(3.0f, c, a));
  R t1 = (b + d) - 2.0f * c, u1 = b - d;
  R t2 = (c + e) - 2.0f * d, u2 = fmaf(-4.0f, d, fmaf(3.0f, c, e));
  R s0 = fmaf(13.0f * t0, t0, fmaf(3.0f * u0, u0, eps12));
  R s1 = fmaf(13.0f * t1, t1, fmaf(3.0f * u1, u1, eps12));
  R s2 = fmaf(13.0f * t2, t2, fmaf(3.0f * u2, u2, eps12));
  const R im = __builtin_amdgcn_rcpf(fminf(fminf(s0, s1), s2));
  const R th = fminf(fabsf(s0 - s2) * im, 1e18f);
  const R th2 = th * th;
  const R ee = __builtin_amdgcn_rcpf(1.0f + th2), q = th2 * ee;
  R r0 = s0 * im, r1 = s1 * im, r2 = s2 * im;
  R w0 = fmaf(q, __builtin_amdgcn_rcpf(r0 * r0), ee);
  R w1 = 6.0f * fmaf(q, __builtin_amdgcn_rcpf(r1 * r1), ee);
  R w2 = 3.0f * fmaf(q, __builtin_amdgcn_rcpf(r2 * r2), ee);
  R p0 = fmaf(11.0f, c, fmaf(-7.0f, b, 2.0f * a));
  R p1 = fmaf(2.0f, d, fmaf(5.0f, c, -b));
  R p2 = fmaf(5.0f, d, fmaf(2.0f, c, -e));
  return fmaf(w0, p0, fmaf(w1, p1, w2 * p2)) * __builtin_amdgcn_rcpf(6.0f * ((w0 + w1) + w2));
}
}  // namespace wf

__device__ __forceinline__ float wenoz(float a, float b, float c, float d, float e, float eps) {
  return wf::wenoz(a, b, c, d, e, eps);
}

// Dual-number WENO5: the same weights, in the plain single-division form;
// only its derivative part is used (local Jacobians of the adjoint).
__device__ __forceinline__ Dual weno5(Dual a, Dual b, Dual c, Dual d, Dual e, Dual eps) {
  const Dual k1312 = 13.0 / 12.0;
  Dual p0 = (2.0 * a - 7.0 * b + 11.0 * c) / 6.0;
  Dual p1 = (-b + 5.0 * c + 2.0 * d) / 6.0;
  Dual p2 = (2.0 * c + 5.0 * d - e) / 6.0;
  Dual t0 = a - 2.0 * b + c, u0 = a - 4.0 * b + 3.0 * c;
  Dual t1 = b - 2.0 * c + d, u1 = b - d;
  Dual t2 = c - 2.0 * d + e, u2 = 3.0 * c - 4.0 * d + e;
  Dual s0 = eps + (k1312 * t0 * t0 + 0.25 * u0 * u0);
  Dual s1 = eps + (k1312 * t1 * t1 + 0.25 * u1 * u1);
  Dual s2 = eps + (k1312 * t2 * t2 + 0.25 * u2 * u2);
  s0 *= s0;
  s1 *= s1;
  s2 *= s2;
  Dual w0 = 0.1 * (s1 * s2), w1 = 0.6 * (s0 * s2), w2 = 0.3 * (s0 * s1);
  return (w0 * p0 + w1 * p1 + w2 * p2) / (w0 + w1 + w2);
}

// Partial derivatives g0..g4 of the WENO5 edge value weno5(a, .., e) with
// respect to the five stencil values, by the chain rule through the weights: with
// s_k = eps + beta_k, w_k = d_k / s_k^2, W = sum w_k, o_k = w_k / W and
// v = sum o_k p_k,
//   dv/dx = sum_k o_k dp_k/dx - 2 sum_k o_k ((p_k - v) / s_k) dbeta_k/dx,
// where beta_k = 13/12 t_k^2 + 1/4 u_k^2 (t_k, u_k linear in x).  The same
// function as the dual-number form above, differentiated in closed form.
__device__ __forceinline__ void weno5_grad(double a, double b, double c, double d, double e, double eps,
                                           double& g0, double& g1, double& g2, double& g3, double& g4) {
#pragma clang fp contract(off)
  const double t0 = (a - 2.0 * b) + c, u0 = (a - 4.0 * b) + 3.0 * c;
  const double t1 = (b - 2.0 * c) + d, u1 = b - d;
  const double t2 = (c - 2.0 * d) + e, u2 = (3.0 * c - 4.0 * d) + e;
  const double k = 13.0 / 12.0;
  const double s0 = eps + (k * t0 * t0 + 0.25 * u0 * u0);
  const double s1 = eps + (k * t1 * t1 + 0.25 * u1 * u1);
  const double s2 = eps + (k * t2 * t2 + 0.25 * u2 * u2);
  const double i0 = face_rcp(s0), i1 = face_rcp(s1), i2 = face_rcp(s2);
  const double w0 = 0.1 * (i0 * i0), w1 = 0.6 * (i1 * i1), w2 = 0.3 * (i2 * i2);
  const double iW = face_rcp((w0 + w1) + w2);
  const double o0 = w0 * iW, o1 = w1 * iW, o2 = w2 * iW;
  const double p0 = ((2.0 * a - 7.0 * b) + 11.0 * c) * (1.0 / 6.0);
  const double p1 = ((-b + 5.0 * c) + 2.0 * d) * (1.0 / 6.0);
  const double p2 = ((2.0 * c + 5.0 * d) - e) * (1.0 / 6.0);
  const double v = (o0 * p0 + o1 * p1) + o2 * p2;
  // -2 o_k (p_k - v) / s_k: the weight of dbeta_k/dx
  const double r0 = -2.0 * o0 * (p0 - v) * i0;
  const double r1 = -2.0 * o1 * (p1 - v) * i1;
  const double r2 = -2.0 * o2 * (p2 - v) * i2;
  const double h = 13.0 / 6.0;
  g0 = o0 * (2.0 / 6.0) + r0 * (h * t0 + 0.5 * u0);
  g1 = (o0 * (-7.0 / 6.0) + o1 * (-1.0 / 6.0)) + (r0 * (-2.0 * h * t0 - 2.0 * u0) + r1 * (h * t1 + 0.5 * u1));
  g2 = ((o0 * (11.0 / 6.0) + o1 * (5.0 / 6.0)) + o2 * (2.0 / 6.0)) +
         ((r0 * (h * t0 + 1.5 * u0) + r1 * (-2.0 * h * t1)) + r2 * (h * t2 + 1.5 * u2));
  g3 = (o1 * (2.0 / 6.0) + o2 * (5.0 / 6.0)) + (r1 * (h * t1 - 0.5 * u1) + r2 * (-2.0 * h * t2 - 2.0 * u2));
  g4 = o2 * (-1.0 / 6.0) + r2 * (h * t2 + 0.5 * u2);
}

// Partial derivatives of the MC edge values with respect to their three
// stencil values.  The MC slope minmod(2 dl, 2 dr, dc/2) (dl = c - l,
// dr = r - c, dc = r - l) is, away from its switching points, the selected
// candidate times a sign: the gradient is that candidate's, chosen by the
// same comparisons as the evaluation (fmin keeps the first operand on ties,
// |x| counts x = 0 as positive, a non-positive dl dr gives the zero slope).
__device__ __forceinline__ void mc_slope_grad(double l, double c, double r, double& gl, double& gc,
                                              double& gr) {
  const double dl = c - l, dr = r - c, dc = r - l;
  const double al = fabs(2.0 * dl), ar = fabs(2.0 * dr), ac = fabs(0.5 * dc);
  const bool pick_r = ar < al;
  const double m = pick_r ? ar : al;
  const bool pick_c = ac < m;
  const double sg = (dc > 0.0 ? 1.0 : -1.0) * (dl * dr > 0.0 ? 1.0 : 0.0);
  // d|k x|/dx = k sign(x), sign(0) = +1
  const double kl = sg * (dl < 0.0 ? -2.0 : 2.0), kr = sg * (dr < 0.0 ? -2.0 : 2.0);
  const double kc = sg * (dc < 0.0 ? -0.5 : 0.5);
  gl = pick_c ? -kc : (pick_r ? 0.0 : -kl);
  gc = pick_c ? 0.0 : (pick_r ? -kr : kl);
  gr = pick_c ? kc : (pick_r ? kr : 0.0);
}
// mc_left(l, c, r) = c + slope/2 and mc_right(l, c, r) = c - slope/2 (tests
// check mc_slope_grad through them).
__device__ __forceinline__ void mc_left_grad(double l, double c, double r, double& g0, double& g1, double& g2) {
  double sl, sc, sr;
  mc_slope_grad(l, c, r, sl, sc, sr);
  g0 = 0.5 * sl;
  g1 = 1.0 + 0.5 * sc;
  g2 = 0.5 * sr;
}
__device__ __forceinline__ void mc_right_grad(double l, double c, double r, double& g0, double& g1, double& g2) {
  double sl, sc, sr;
  mc_slope_grad(l, c, r, sl, sc, sr);
  g0 = -0.5 * sl;
  g1 = 1.0 - 0.5 * sc;
  g2 = -0.5 * sr;
}

// ---------------------------------------------------------- face physics --
//
// The state on one side of a face as the flux kernels need it: conserved
// variables U, the flux F^d along the face normal (both without the factor
// sqrt(-g), which is common to the two sides and applied once to their
// Lax-Friedrichs combination) and the larger of the two fast signal speeds'
// magnitudes (all the combination reads of them), from the
// reconstructed prims and the face metric.  The same
// formulas as fluid_state / prim_to_flux / char_speeds, arranged for the
// face, where these evaluations dominate the step's arithmetic:
//   * the face metric holds only the entries that are not identically zero
//     in the library's two spacetimes: flat space and Kerr in modified
//     Kerr-Schild coordinates both have g_{2 mu} = g^{2 mu} = 0 for mu != 2
//     and g^{t3} = 0, so those products are never formed;
//   * FP64: the speeds' quadratic times w (b^2 + w), which leaves its roots
//     unchanged, needs neither the sound nor the Alfven speed: with
//     n = gam p + b^2 and m = (b^2 + w) - n = rho + gam (2 - gam) u (w = rho +
//     gam u), c^2 = n / (n + m) exactly and A = m u^t u^t - n g^tt, likewise B
//     and C.  That leaves one reciprocal (of A) and two square roots per side,
//     of which the Lorentz factor's gives its reciprocal too;
//   * the two roots (b +- s)/A (b = -B/2, s >= 0) have the larger magnitude
//     (|b| + s)/|A|;
//   * fused multiply-adds, written out (contraction off), so that a face
//     rounds the same way in every kernel that evaluates it.
// In FP64 the reciprocals and square roots are the hardware estimates
// refined by Newton steps to about an ulp; the results differ from the
// written form by rounding only.
#pragma clang fp contract(off)

__device__ __forceinline__ float face_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// sqrt(x) for normal x > 0 (Goldschmidt from the hardware estimate; about an
// ulp), and with it h close to 1 / (2 sqrt(x)) (2^-46 relative).
__device__ __forceinline__ double face_sqrt(double x, double& h) {
  const double y = hw_rsqrt(x);
  const double g = x * y;
  const double k = 0.5 * y;
  const double r = fma(-k, g, 0.5);
  const double g1 = fma(g, r, g);
  h = fma(k, r, k);
  return fma(fma(-g1, g1, x), h, g1);
}
// sqrt(x) of a discriminant, zero if it is not positive: cold gas at rest has
// no signal speed at all, and a CFL step of it is refused.
__device__ __forceinline__ double speed_root(double x) {
  double h;
  const double s = face_sqrt(x, h);
  return x > 0.0 ? s : 0.0;
}
// 2^-e with 2^e <= |x| < 2^(e+1): scales a homogeneous expression without
// rounding (x normal, below 2^1023; 2^1023 for a subnormal x, -inf for an
// infinite one).
__device__ __forceinline__ double unit_scale(double x) {
  const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32);
  return __builtin_bit_cast(double, (unsigned long long)(0x7fe00000u - (hi & 0x7ff00000u)) << 32);
}

template <typename R>
struct FaceMetric {
  R gtt, gt1, gt3, g11, g13, g22, g33;   // covariant
  R ctt, ct1, c11, c22, c33;             // contravariant
  R gdet, alpha, ialpha;
};

// 1 / alpha = -g^tt alpha in FP64 (alpha = (-g^tt)^-1/2).
__device__ __forceinline__ double inverse_lapse(double alpha, double ctt) { return -ctt * alpha; }
__device__ __forceinline__ float inverse_lapse(float alpha, float) { return __builtin_amdgcn_rcpf(alpha); }

template <typename R>
__device__ __forceinline__ void load_face_metric(const double* __restrict__ tab, long plane, long q,
                                                 FaceMetric<R>& m) {
  const Pair<double>* t = (const Pair<double>*)tab;
  auto at = [&](int f) { return t[(f >> 1) * plane + q]; };
  const Pair<double> x0 = at(G_GTT), x1 = at(G_GT3), x2 = at(G_G11), x3 = at(G_G22), x4 = at(G_CTT), x5 = at(G_DET),
                     x6 = at(G_C11);
  m.gtt = (R)x0.a;
  m.gt1 = (R)x0.b;
  m.gt3 = (R)x1.a;
  m.g33 = (R)x1.b;
  m.g11 = (R)x2.a;
  m.g13 = (R)x2.b;
  m.g22 = (R)x3.a;
  m.c22 = (R)x3.b;
  m.ctt = (R)x4.a;
  m.ct1 = (R)x4.b;
  m.gdet = (R)x5.a;
  m.alpha = (R)x5.b;
  m.c11 = (R)x6.a;
  m.c33 = (R)x6.b;
  m.ialpha = inverse_lapse(m.alpha, m.ctt);
}

// Lorentz factor g = sqrt(x) of x = gamma^2 and alpha / g (FP64, FP32).
__device__ __forceinline__ double lorentz(double x, double alpha, double& iut) {
  double h;
  const double g = face_sqrt(x, h);
  const double i = h + h;                     // 1/g to 2^-46, then one step
  iut = alpha * fma(fma(-g, i, 1.0), i, i);
  return g;
}
__device__ __forceinline__ float lorentz(float x, float alpha, float& iut) {
  const float g = sqrt(x);
  iut = alpha * __builtin_amdgcn_rcpf(g);
  return g;
}

// Larger magnitude of the two fast speeds along D, from the gas pressure pg,
// b^2, the four-velocity components ut, ud and the metric's g^tt, g^tD, g^DD:
// roots v of (u^D - v u^t)^2 (1 - c^2) = c^2 (v^2 g^tt - 2 v g^tD + g^DD),
// c^2 = cs^2 + vA^2 - cs^2 vA^2, cs^2 = gam p / w, vA^2 = b^2 / (b^2 + w),
// w = rho + gam u.
__device__ __forceinline__ double fast_speed(double rho, double uu, double pg, double bsq, double gam, double ut,
                                             double ud, double ctt, double ctd, double cdd) {
  const double n0 = fma(gam, pg, bsq);
  const double m0 = fma(gam * (2.0 - gam), uu, rho);
  const double sc = unit_scale(n0 + m0);
  const double n = n0 * sc, m = m0 * sc;
  const double mut = m * ut, mud = m * ud;
  const double A = fma(mut, ut, -n * ctt);
  const double b = fma(mut, ud, -n * ctd);
  const double C = fma(mud, ud, -n * cdd);
  // a discriminant that is not positive counts as zero
  const double s = speed_root(fma(b, b, -(A * C)));
  return (fabs(b) + s) * fabs(face_rcp(A));
}
__device__ __forceinline__ float fast_speed(float rho, float uu, float pg, float bsq, float gam, float ut, float ud,
                                            float ctt, float ctd, float cdd) {
  const float we = fmaf(gam, uu, rho);
  const float sw = bsq + we;
  const float rr = face_rcp(we * sw);
  const float cs2 = ((gam * pg) * sw) * rr;
  const float va2 = (bsq * we) * rr;
  const float c2 = fmaf(-cs2, va2, cs2 + va2);
  const float ut2 = ut * ut, udt = ud * ut, ud2 = ud * ud;
  const float A = fmaf(-c2, ctt + ut2, ut2);
  const float B = -2.0f * fmaf(-c2, ctd + udt, udt);
  const float C = fmaf(-c2, cdd + ud2, ud2);
  float disc = fmaf(B, B, -4.0f * A * C);
  disc = disc > 0.0f ? disc : 0.0f;
  return (fabsf(B) + sqrt(disc)) * fabsf(0.5f * face_rcp(A));
}

// U / sqrt(-g), F^D / sqrt(-g) (D = 1..3) and the larger signal speed
// magnitude of the prims p.
template <int D, typename R>
__device__ __forceinline__ R face_side(const R p[NVAR], const FaceMetric<R>& m, R gam, R F[NVAR], R U[NVAR]) {
  const R rho = p[RHO], uu = p[UU], v1 = p[U1], v2 = p[U2], v3 = p[U3];
  const R Bc1 = p[B1], Bc2 = p[B2], Bc3 = p[B3];
  // four-velocity: gamma^2 = 1 + g_ij u~i u~j, u^t = gamma / alpha,
  // u^i = u~i - gamma alpha g^{ti}, lowered with the face metric
  const R qsq = fma(m.g11 * v1, v1, fma(m.g22 * v2, v2, fma(m.g33 * v3, v3, (R)2 * (m.g13 * v1) * v3)));
  R iut;
  const R gamma = lorentz((R)1 + qsq, m.alpha, iut);
  const R ga = gamma * m.alpha;
  const R ut = gamma * m.ialpha;
  const R u1 = fma(-ga, m.ct1, v1), u2 = v2, u3 = v3;
  const R l0 = fma(m.gtt, ut, fma(m.gt1, u1, m.gt3 * u3));
  const R l1 = fma(m.gt1, ut, fma(m.g11, u1, m.g13 * u3));
  const R l2 = m.g22 * u2;
  const R l3 = fma(m.gt3, ut, fma(m.g13, u1, m.g33 * u3));
  // magnetic four-vector: b^t = B^i u_i, b^i = (B^i + b^t u^i) / u^t
  const R bt = fma(Bc1, l1, fma(Bc2, l2, Bc3 * l3));
  const R b1 = fma(bt, u1, Bc1) * iut, b2 = fma(bt, u2, Bc2) * iut, b3 = fma(bt, u3, Bc3) * iut;
  const R k0 = fma(m.gtt, bt, fma(m.gt1, b1, m.gt3 * b3));
  const R k1 = fma(m.gt1, bt, fma(m.g11, b1, m.g13 * b3));
  const R k2 = m.g22 * b2;
  const R k3 = fma(m.gt3, bt, fma(m.g13, b1, m.g33 * b3));
  const R bsq = fma(bt, k0, fma(b1, k1, fma(b2, k2, b3 * k3)));
  // rows t (conserved variables) and D (flux) of
  // T^mu_nu = (rho + u + p + b^2) u^mu u_nu + (p + b^2/2) delta^mu_nu - b^mu b_nu
  const R pg = (gam - (R)1) * uu;
  const R w = ((rho + uu) + pg) + bsq;
  const R ptot = fma((R)0.5, bsq, pg);
  const R ud = D == 1 ? u1 : (D == 2 ? u2 : u3);
  const R bd = D == 1 ? b1 : (D == 2 ? b2 : b3);
  {
    const R wu = w * ut;
    const R ru = rho * ut;
    U[RHO] = ru;
    U[UU] = fma(wu, l0, fma(-bt, k0, ptot)) + ru;
    U[U1] = fma(wu, l1, -bt * k1);
    U[U2] = fma(wu, l2, -bt * k2);
    U[U3] = fma(wu, l3, -bt * k3);
    U[B1] = Bc1;
    U[B2] = Bc2;
    U[B3] = Bc3;
  }
  {
    const R wu = w * ud;
    const R ru = rho * ud;
    F[RHO] = ru;
    F[UU] = fma(wu, l0, -bd * k0) + ru;
    F[U1] = fma(wu, l1, fma(-bd, k1, D == 1 ? ptot : (R)0));
    F[U2] = fma(wu, l2, fma(-bd, k2, D == 2 ? ptot : (R)0));
    F[U3] = fma(wu, l3, fma(-bd, k3, D == 3 ? ptot : (R)0));
    F[B1] = fma(b1, ud, -bd * u1);
    F[B2] = fma(b2, ud, -bd * u2);
    F[B3] = fma(b3, ud, -bd * u3);
  }
  const R cdd = D == 1 ? m.c11 : (D == 2 ? m.c22 : m.c33);
  const R ctd = D == 1 ? m.ct1 : (R)0;
  return fast_speed(rho, uu, pg, bsq, gam, ut, ud, m.ctt, ctd, cdd);
}

// ---------------------------------------------------------- zone physics --
//
// The state at a zone centre as the update and the CFL rate need it, arranged
// as the face states are: only the metric entries that are not identically
// zero, reciprocals and square roots from the hardware estimates, fused
// multiply-adds written out.
struct ZoneState {
  double ut, u1, u2, u3;      // four-velocity
  double l0, l1, l2, l3;      // lowered
  double bt, b1, b2, b3;      // magnetic four-vector
  double k0, k1, k2, k3;      // lowered
  double bsq, w, ptot, pg;    // w = rho + u + p + b^2
  double iut;                 // 1 / u^t
};
__device__ __forceinline__ void zone_state(const double p[NVAR], const PointMetric<double>& m, double gam,
                                           ZoneState& z) {
  const double gtt = m.gcov[sidx(0, 0)], gt1 = m.gcov[sidx(0, 1)], gt3 = m.gcov[sidx(0, 3)], g11 = m.gcov[sidx(1, 1)],
               g13 = m.gcov[sidx(1, 3)], g22 = m.gcov[sidx(2, 2)], g33 = m.gcov[sidx(3, 3)];
  const double ctt = m.gcon[sidx(0, 0)], ct1 = m.gcon[sidx(0, 1)];
  const double v1 = p[U1], v2 = p[U2], v3 = p[U3], Bc1 = p[B1], Bc2 = p[B2], Bc3 = p[B3];
  const double qsq = fma(g11 * v1, v1, fma(g22 * v2, v2, fma(g33 * v3, v3, 2.0 * (g13 * v1) * v3)));
  const double gamma = lorentz(1.0 + qsq, m.alpha, z.iut);
  z.ut = quotient(gamma, m.alpha, inverse_lapse(m.alpha, ctt));
  z.u1 = fma(-(gamma * m.alpha), ct1, v1);
  z.u2 = v2;
  z.u3 = v3;
  z.l0 = fma(gtt, z.ut, fma(gt1, z.u1, gt3 * z.u3));
  z.l1 = fma(gt1, z.ut, fma(g11, z.u1, g13 * z.u3));
  z.l2 = g22 * z.u2;
  z.l3 = fma(gt3, z.ut, fma(g13, z.u1, g33 * z.u3));
  z.bt = fma(Bc1, z.l1, fma(Bc2, z.l2, Bc3 * z.l3));
  z.b1 = fma(z.bt, z.u1, Bc1) * z.iut;
  z.b2 = fma(z.bt, z.u2, Bc2) * z.iut;
  z.b3 = fma(z.bt, z.u3, Bc3) * z.iut;
  z.k0 = fma(gtt, z.bt, fma(gt1, z.b1, gt3 * z.b3));
  z.k1 = fma(gt1, z.bt, fma(g11, z.b1, g13 * z.b3));
  z.k2 = g22 * z.b2;
  z.k3 = fma(gt3, z.bt, fma(g13, z.b1, g33 * z.b3));
  z.bsq = fma(z.bt, z.k0, fma(z.b1, z.k1, fma(z.b2, z.k2, z.b3 * z.k3)));
  z.pg = (gam - 1.0) * p[UU];
  z.w = ((p[RHO] + p[UU]) + z.pg) + z.bsq;
  z.ptot = fma(0.5, z.bsq, z.pg);
}

// Conserved variables sqrt(-g) (rho u^t, T^t_t + rho u^t, T^t_i, B^i).
__device__ __forceinline__ void zone_cons(const double p[NVAR], const ZoneState& z, double gdet, double U[NVAR]) {
  const double wu = z.w * z.ut, ru = p[RHO] * z.ut;
  U[RHO] = gdet * ru;
  U[UU] = gdet * (fma(wu, z.l0, fma(-z.bt, z.k0, z.ptot)) + ru);
  U[U1] = gdet * fma(wu, z.l1, -z.bt * z.k1);
  U[U2] = gdet * fma(wu, z.l2, -z.bt * z.k2);
  U[U3] = gdet * fma(wu, z.l3, -z.bt * z.k3);
  U[B1] = gdet * p[B1];
  U[B2] = gdet * p[B2];
  U[B3] = gdet * p[B3];
}

// Geometric source of the x1 and x2 momentum equations (metric_source in
// physics_body.inc has the derivation): sqrt(-g) sum_kl T^{kl} d_nu g_kl / 2
// over the seven entries that vary, d(n) the derivative pair of entry n
// (dgs_entry), T^{kl} = w u^k u^l + ptot g^{kl} - b^k b^l.
template <typename Deriv>
__device__ __forceinline__ void zone_source(const ZoneState& z, const PointMetric<double>& m, Deriv d, double S[2]) {
  const double u[4] = {z.ut, z.u1, z.u2, z.u3}, b[4] = {z.bt, z.b1, z.b2, z.b3};
  double s1 = 0.0, s2 = 0.0;
#pragma unroll
  for (int x = 0; x < 4; x++) {
    const double wu = z.w * u[x];
#pragma unroll
    for (int y = x; y < 4; y++) {
      if (x2_offdiag(sidx(x, y))) continue;
      const double t = fma(-b[x], b[y], wu * u[y]);
      const double T = x == 0 && y == 3 ? t : fma(z.ptot, m.gcon[sidx(x, y)], t);
      const Pair<double> q = d(dgs_entry(sidx(x, y)));
      s1 = fma(T, q.a, s1);
      s2 = fma(T, q.b, s2);
    }
  }
  S[0] = m.gdet * s1;
  S[1] = m.gdet * s2;
}

// Larger magnitudes of the fast speeds along x1, x2 and x3 (fast_speed above;
// the quadratics' A, scale and enthalpy terms are common to the three).  An
// infinite density counts as a large one: the speeds are the flow's.
__device__ __forceinline__ void zone_speeds(double rho, double uu, const ZoneState& z, const PointMetric<double>& m,
                                            double gam, double c[3]) {
  const double n0 = fma(gam, z.pg, z.bsq);
  const double m0 = fma(gam * (2.0 - gam), uu, rho == (double)INFINITY ? 0x1p1020 : rho);
  const double sc = unit_scale(n0 + m0);
  const double n = n0 * sc, mm = m0 * sc;
  const double mut = mm * z.ut;
  const double A = fma(mut, z.ut, -n * m.gcon[sidx(0, 0)]);
  const double iA = fabs(face_rcp(A));
  const double ud[3] = {z.u1, z.u2, z.u3};
#pragma unroll
  for (int d = 0; d < 3; d++) {
    const double b = d == 0 ? fma(mut, ud[d], -n * m.gcon[sidx(0, 1)]) : mut * ud[d];
    const double C = fma(mm * ud[d], ud[d], -n * m.gcon[sidx(d + 1, d + 1)]);
    const double s = speed_root(fma(b, b, -(A * C)));
    c[d] = (fabs(b) + s) * iA;
  }
}

}  // namespace grmhd
