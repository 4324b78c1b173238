// The geometric source as the update kernels form it (zone_state and
// zone_source on the paired metric-derivative entries), compiled for the host
// from the library's source.
//
//   zone_source_host <in> <out>
// in:  int32 npoints, int32 kerr, float64 gam, a, hslope,
//      then per point float64 x1, x2, P[8]
// out: per point float64 S1, S2 (the x1 and x2 momentum sources)
#include <stdio.h>
#include <stdlib.h>
#include <vector>

#include "hip/hip_runtime.h"
#include "../../include/grmhd.h"
#include "../../paper_2408_01361_amd/csrc/geometry.hpp"
#include "../../paper_2408_01361_amd/csrc/physics.hpp"

using namespace grmhd;

static void need(bool ok, const char* what) {
  if (!ok) {
    fprintf(stderr, "zone_source_host: %s\n", what);
    exit(2);
  }
}

int main(int argc, char** argv) {
  need(argc == 3, "usage: zone_source_host <in> <out>");
  FILE* f = fopen(argv[1], "rb");
  need(f != nullptr, "cannot open input");
  int hdr[2];
  double par[3];
  need(fread(hdr, sizeof(int), 2, f) == 2 && fread(par, sizeof(double), 3, f) == 3, "short header");
  const int n = hdr[0];
  need(n >= 0 && n < (1 << 24), "bad point count");
  const SpaceTime st{hdr[1], par[1], par[2]};
  std::vector<double> in((size_t)n * 10), out((size_t)n * 2);
  need(fread(in.data(), sizeof(double), in.size(), f) == in.size(), "short input");
  fclose(f);
  for (int q = 0; q < n; q++) {
    const double* c = &in[(size_t)q * 10];
    PointMetric<double> m;
    metric_point(st, c[0], c[1], m.gcov, m.gcon, m.gdet, m.alpha);
    double D[NDG];
    source_metric_point(st, c[0], c[1], D);
    Pair<double> table[NDGT / 2];   // as the kernels' table holds them
    for (int s = 0; s < 10; s++)
      if (!x2_offdiag(s)) table[dgs_entry(s)] = Pair<double>{D[s], D[10 + s]};
    ZoneState z;
    zone_state(c + 2, m, par[0], z);
    zone_source(z, m, [&](int e) { return table[e]; }, &out[(size_t)q * 2]);
  }
  FILE* o = fopen(argv[2], "wb");
  need(o != nullptr, "cannot open output");
  need(fwrite(out.data(), sizeof(double), out.size(), o) == out.size(), "short write");
  fclose(o);
  return 0;
}
