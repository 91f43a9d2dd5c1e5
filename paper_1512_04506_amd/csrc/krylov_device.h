// Device helpers shared by the Krylov kernels: wave sums in FP64, the sums of
// one workgroup of AT lanes (coarse GMRES) and the Givens rotation of the
// Hessenberg least squares.
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

// one coarse vector, one workgroup
constexpr int AT = 1024;
constexpr int AW = AT / 64;
constexpr int AJ = 4;  // inner products per reduction (8 real sums)

// v[0..7] summed over the 64 lanes: three halving steps leave one value per
// lane (value 4 (lane / 32) + 2 (lane / 16 % 2) + lane / 8 % 2), three more
// sum it over its eight lanes: 10 exchanges instead of 48
__device__ inline double sum8(double v[8], int lane) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool up = (lane & 32) != 0;
    const double send = up ? v[j] : v[j + 4], keep = up ? v[j + 4] : v[j];
    v[j] = keep + __shfl_xor(send, 32, 64);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const bool up = (lane & 16) != 0;
    const double send = up ? v[j] : v[j + 2], keep = up ? v[j + 2] : v[j];
    v[j] = keep + __shfl_xor(send, 16, 64);
  }
  {
    const bool up = (lane & 8) != 0;
    const double send = up ? v[0] : v[1], keep = up ? v[1] : v[0];
    v[0] = keep + __shfl_xor(send, 8, 64);
  }
  v[0] += __shfl_xor(v[0], 4, 64);
  v[0] += __shfl_xor(v[0], 2, 64);
  v[0] += __shfl_xor(v[0], 1, 64);
  return v[0];
}

// out[0 .. cnt) (LDS) = the workgroup's sums of acc[0 .. AJ), cnt <= AJ; red [8][AW]
__device__ inline void block_sum(cx<double>* out, const cx<double> acc[AJ], int cnt, double (*red)[AW]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double v[8];
#pragma unroll
  for (int q = 0; q < AJ; ++q) {
    v[2 * q] = acc[q].r;
    v[2 * q + 1] = acc[q].i;
  }
  const double s = sum8(v, lane);
  if ((lane & 7) == 0) red[lane >> 3][w] = s;
  __syncthreads();
  if (threadIdx.x < 2 * cnt) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < AW; ++k) t += red[threadIdx.x][k];
    reinterpret_cast<double*>(out)[threadIdx.x] = t;
  }
  __syncthreads();
}

}  // namespace dev
}  // namespace ddamg
