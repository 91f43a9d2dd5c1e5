// Inversion of the even self blocks of D_c (Alg. 2's D_ee^{-1}): in-place
// Gauss-Jordan with partial (row) pivoting in FP64, one workgroup per even
// coarse site; the inverse is stored column-major in T.
#include "sap_device.h"

namespace ddamg {

namespace {

using namespace dev;

__device__ inline double lane_value(double v, int lane) {  // lane uniform
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// the largest value of the wave, at least zero
__device__ inline double wave_max(double v) {
  v = fmax(v, dpp_move<0xB1, 0xF>(v));   // quad_perm [1,0,3,2]
  v = fmax(v, dpp_move<0x4E, 0xF>(v));   // quad_perm [2,3,0,1]
  v = fmax(v, dpp_move<0x114, 0xF>(v));  // row_shr:4
  v = fmax(v, dpp_move<0x118, 0xF>(v));  // row_shr:8
  v = fmax(v, dpp_move<0x142, 0xA>(v));  // row_bcast:15 into rows 1 and 3
  v = fmax(v, dpp_move<0x143, 0xC>(v));  // row_bcast:31 into rows 2 and 3
  return lane_value(v, 63);
}

// nc <= 32: every entry in the register of one lane, lane % W the row, the
// columns dealt to the 256 / W groups of W lanes.  A step hands column k to
// all waves through LDS, one barrier; each finds the pivot by itself and
// takes the pivot row from its own lanes.  The pivot rows stay where they
// are, the interchanges are undone by the addresses of the result.  Bound:
// the chain of a step (pivot search, reciprocal, barrier).  16 sites, nc 32,
// FP64: 31 us, 66 with the matrix in LDS, where a step has eight barriers.
template <typename T, typename S>
__global__ __launch_bounds__(256) void invert_even_kernel(cx<T>* Dinv, CoarseView<S> cv, int nc, int* status) {
  constexpr int W = 32, RS = 256 / W, NQ = W / RS;  // columns j0 + RS q of row i
  __shared__ cx<double> col[2][W];
  __shared__ int perm[W];
  const int ci = blockIdx.x;  // even sites are internal indices [0, neven)
  const int t = threadIdx.x, i = t % W, j0 = t / W, half = t & 32;
  const size_t nn = (size_t)nc * nc;
  double sc = 1.0;
  if constexpr (is_half<S>()) sc = (double)cv.Dsc[ci * 9];
  cx<double> a[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int j = j0 + RS * q;
    a[q] = i < nc && j < nc ? sc * ldc<double>(cv.D, (size_t)ci * 9 * nn + (size_t)j * nc + i) : mk(0.0, 0.0);
  }
  bool used = i >= nc;  // rows that no later step may choose
  int mine = 0;         // the step that chose this row
  for (int k = 0; k < nc; ++k) {
    cx<double>* ck = col[k & 1];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (j0 + RS * q == k) ck[i] = a[q];
    __syncthreads();
    const cx<double> f = ck[i];
    const double n2 = f.r * f.r + f.i * f.i, v = !used && n2 > 0.0 ? n2 : -1.0;
    const double m = wave_max(v);
    if (!(m > 0.0)) {  // uniform over the workgroup: all waves hold the column
      if (t == 0) atomicExch(status, 1);
      return;
    }
    const int p = __builtin_ctzll(__ballot(v == m)) % W;
    const cx<double> pv = ck[p];
    const double pn = pv.r * pv.r + pv.i * pv.i;
    const cx<double> ipv = mk(pv.r / pn, -pv.i / pn);
    const bool pivot = i == p;
    if (pivot) {
      used = true;
      mine = k;
    }
    if (t == 0) perm[k] = p;
    // the pivot row scaled (its pivot becomes 1 / pv), column k eliminated from the others
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (RS * q >= nc) break;
      cx<double> r = mk(__shfl(a[q].r, half + p, 64), __shfl(a[q].i, half + p, 64));
      if (j0 + RS * q == k) {
        r = mk(1.0, 0.0);
        a[q] = mk(0.0, 0.0);
      }
      const cx<double> rk = r * ipv;
      a[q] = pivot ? rk : a[q] - f * rk;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int j = j0 + RS * q;
    if (i < nc && j < nc) Dinv[(size_t)ci * nn + (size_t)perm[j] * nc + mine] = cvt<T>(a[q]);
  }
}

// nc > 32: the matrix in LDS (its entries no longer leave a SIMD's registers
// the waves to hide a step: nc 48, 1296 sites, 319 us, 332 in registers)
template <typename T, typename S>
__global__ __launch_bounds__(256) void invert_even_lds_kernel(cx<T>* Dinv, CoarseView<S> cv, int nc, int* status) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  cx<double>* M = reinterpret_cast<cx<double>*>(smem_raw);  // row-major nc x nc
  cx<double>* colk = M + (size_t)nc * nc;                    // column k before elimination
  int* perm = reinterpret_cast<int*>(colk + nc);
  __shared__ int piv_row;
  __shared__ int singular;
  const int ci = blockIdx.x;  // even sites are internal indices [0, neven)
  const size_t nn = (size_t)nc * nc;
  double sc = 1.0;
  if constexpr (is_half<S>()) sc = (double)cv.Dsc[ci * 9];
  for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
    const int col = e / nc, row = e % nc;
    M[row * nc + col] = sc * ldc<double>(cv.D, (size_t)ci * 9 * nn + e);
  }
  if (threadIdx.x == 0) singular = 0;
  __syncthreads();
  for (int k = 0; k < nc; ++k) {
    if (threadIdx.x < 64) {
      double best = -1.0;
      int bi = k;
      for (int i = k + threadIdx.x; i < nc; i += 64) {
        cx<double> v = M[i * nc + k];
        double a = v.r * v.r + v.i * v.i;
        if (a > best) { best = a; bi = i; }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        double ob = __shfl_xor(best, o, 64);
        int oi = __shfl_xor(bi, o, 64);
        if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
      }
      if (threadIdx.x == 0) {
        piv_row = bi;
        perm[k] = bi;
        if (!(best > 0.0)) singular = 1;
      }
    }
    __syncthreads();
    if (singular) break;
    const int p = piv_row;
    if (p != k)
      for (int j = threadIdx.x; j < nc; j += blockDim.x) {
        cx<double> t = M[k * nc + j];
        M[k * nc + j] = M[p * nc + j];
        M[p * nc + j] = t;
      }
    __syncthreads();
    const cx<double> pv = M[k * nc + k];
    const double pn = pv.r * pv.r + pv.i * pv.i;
    const cx<double> ipv = mk(pv.r / pn, -pv.i / pn);
    __syncthreads();
    // scale the pivot row (the pivot entry becomes 1/pv)
    for (int j = threadIdx.x; j < nc; j += blockDim.x) M[k * nc + j] = (j == k ? mk(1.0, 0.0) : M[k * nc + j]) * ipv;
    __syncthreads();
    for (int i = threadIdx.x; i < nc; i += blockDim.x) colk[i] = M[i * nc + k];
    __syncthreads();
    // eliminate column k from the other rows
    for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
      const int i = e / nc, j = e % nc;
      if (i == k) continue;
      const cx<double> f = colk[i];
      const cx<double> rk = M[k * nc + j];
      M[i * nc + j] = (j == k ? mk(0.0, 0.0) : M[i * nc + j]) - f * rk;
    }
    __syncthreads();
  }
  if (singular) {
    if (threadIdx.x == 0) atomicExch(status, 1);
    return;
  }
  // undo the row interchanges as column interchanges, last first
  for (int k = nc - 1; k >= 0; --k) {
    const int p = perm[k];
    if (p != k)
      for (int i = threadIdx.x; i < nc; i += blockDim.x) {
        cx<double> t = M[i * nc + k];
        M[i * nc + k] = M[i * nc + p];
        M[i * nc + p] = t;
      }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
    const int col = e / nc, row = e % nc;
    Dinv[(size_t)ci * nn + e] = cvt<T>(M[row * nc + col]);
  }
}

}  // namespace

template <typename T, typename S>
void launch_invert_even_blocks(cx<T>* Dinv, const CoarseView<S>& cv, const Geom& g, int* status, hipStream_t st) {
  if (g.nc <= 32) {
    invert_even_kernel<T, S><<<g.neven, 256, 0, st>>>(Dinv, cv, g.nc, status);
  } else {
    const size_t lds = (size_t)(g.nc * g.nc + g.nc) * sizeof(cx<double>) + (size_t)g.nc * sizeof(int);
    invert_even_lds_kernel<T, S><<<g.neven, 256, lds, st>>>(Dinv, cv, g.nc, status);
  }
}
#define INST(T, S) \
  template void launch_invert_even_blocks<T, S>(cx<T>*, const CoarseView<S>&, const Geom&, int*, hipStream_t);
INST(double, double)
INST(float, float)
INST(float, __half)
#undef INST

}  // namespace ddamg
