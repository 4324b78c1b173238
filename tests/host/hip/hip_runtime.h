// Host stand-in for <hip/hip_runtime.h>: with it the per-point device code of
// the library (geometry, physics, the primitive-variable recoveries and the
// adjoint's sweeps) compiles as plain C++ on the host.  The function
// qualifiers become nothing and the hardware reciprocals become divisions,
// better estimates than the hardware's: the refinement steps that follow them
// run as on the GPU, but from a start that is already rounded, so what they
// correct there is not tested here.
#pragma once
#include <math.h>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline

static inline float host_rcpf(float x) { return 1.0f / x; }
static inline double host_rcp(double x) { return 1.0 / x; }
#define __builtin_amdgcn_rcpf(x) host_rcpf(x)
#define __builtin_amdgcn_rcp(x) host_rcp(x)
