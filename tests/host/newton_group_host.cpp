// The implicit solver's Newton iteration by eight lanes (newton_hydro_group,
// continuing what one lane left open after a few iterations) against the one
// lane's to the end (newton_hydro), compiled for the host from the library's
// source with the lanes in lockstep.
//
//   newton_group_host <in> <out>
// in:  int32 ncases, int32 kerr, int32 maxit, int32 head, float64 gam, tol, a,
//      hslope, then per case float64 x1, x2, U[8], guess[8]
// out: per case float64 x[5], outcome of the one lane, then of the two-part
//      solve, then 1 if that one was left open
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <vector>

#include "hip/hip_runtime.h"
#include "lanes/lockstep.hpp"
#include "../../include/grmhd.h"
#include "../../paper_2408_01361_amd/csrc/geometry.hpp"
#include "../../paper_2408_01361_amd/csrc/physics.hpp"

using namespace grmhd;

namespace {

constexpr int BLOCK = 256;  // the Jacobian's LDS stride, as on the GPU

// The fields of the kernels' grid description that the recoveries read.
struct Dev {
  double gam, tol;
  int maxit;
  int inverter;
  double vmax2;
  int floors;
};

#include "../../paper_2408_01361_amd/csrc/inversion.hpp"
#include "../../paper_2408_01361_amd/csrc/newton_group.hpp"

}  // namespace

static void need(bool ok, const char* what) {
  if (!ok) {
    fprintf(stderr, "newton_group_host: %s\n", what);
    exit(2);
  }
}

int main(int argc, char** argv) {
  need(argc == 3, "usage: newton_group_host <in> <out>");
  FILE* f = fopen(argv[1], "rb");
  need(f != nullptr, "cannot open input");
  int hdr[4];
  double par[4];
  need(fread(hdr, sizeof(int), 4, f) == 4 && fread(par, sizeof(double), 4, f) == 4, "short header");
  const int n = hdr[0], head = hdr[3];
  need(n >= 0 && n < (1 << 20) && head > 0 && head < hdr[2], "bad header");
  const Dev g{par[0], par[1], hdr[2], 2, 0.0, 0};
  const SpaceTime st{hdr[1], par[2], par[3]};
  std::vector<double> in((size_t)n * 18), out((size_t)n * 13, 0.0);
  need(fread(in.data(), sizeof(double), in.size(), f) == in.size(), "short input");
  fclose(f);
  std::vector<double> jac(25 * BLOCK);
  for (int q = 0; q < n; q++) {
    const double* c = &in[(size_t)q * 18];
    const double* U = c + 2;
    PointMetric<double> m;
    metric_point(st, c[0], c[1], m.gcov, m.gcon, m.gdet, m.alpha);
    const double B[3] = {U[B1] / m.gdet, U[B2] / m.gdet, U[B3] / m.gdet};
    double scale = 0.0;
    for (int k = 0; k < 5; k++) scale = fabs(U[k]) > scale ? fabs(U[k]) : scale;
    auto res = [&](const double x[5], double R[5]) { implicit_residual(g, m, x, B, U, scale, R); };
    double* o = &out[(size_t)q * 13];
    o[5] = newton_hydro(g, c + 10, res, o, jac.data(), g.maxit);
    double x[5];
    const int how = newton_hydro(g, c + 10, res, x, jac.data(), head);
    if (how != NEWTON_OPEN) {
      memcpy(o + 6, x, sizeof(x));
      o[11] = how;
      continue;
    }
    o[12] = 1.0;
    double each[8][5];
    int outcome[8];
    lanes::run([&](int lane) {
      memcpy(each[lane], x, sizeof(x));
      outcome[lane] = newton_hydro_group(g, res, each[lane], jac.data() + lane, head);
    });
    for (int l = 1; l < 8; l++)
      need(outcome[l] == outcome[0] && memcmp(each[l], each[0], sizeof(x)) == 0, "the lanes of a zone disagree");
    memcpy(o + 6, each[0], sizeof(x));
    o[11] = outcome[0];
  }
  FILE* o = fopen(argv[2], "wb");
  need(o != nullptr, "cannot open output");
  need(fwrite(out.data(), sizeof(double), out.size(), o) == out.size(), "short write");
  fclose(o);
  return 0;
}
