// Device helpers shared by the Krylov kernels: wave sums in FP64 and the
// Givens rotation of the Hessenberg least squares.
#pragma once
#include "ddamg_internal.h"

namespace ddamg {
namespace dev {

__device__ inline double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ inline double cabs2(cx<double> a) { return a.r * a.r + a.i * a.i; }

// rotation [c s; -conj(s) c] (c real) with c a + s b = r, -conj(s) a + c b = 0
__device__ inline void givens(cx<double> a, cx<double> b, double& c, cx<double>& s, cx<double>& r) {
  const double na = sqrt(cabs2(a)), nb = sqrt(cabs2(b));
  if (nb == 0.0) {
    c = 1.0;
    s = mk(0.0, 0.0);
    r = a;
    return;
  }
  if (na == 0.0) {
    c = 0.0;
    s = (1.0 / nb) * conj(b);
    r = mk(nb, 0.0);
    return;
  }
  const double nrm = sqrt(na * na + nb * nb);
  const cx<double> ph = (1.0 / na) * a;
  c = na / nrm;
  s = (1.0 / nrm) * (ph * conj(b));
  r = nrm * ph;
}

}  // namespace dev
}  // namespace ddamg
