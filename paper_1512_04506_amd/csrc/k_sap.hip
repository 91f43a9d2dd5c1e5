// Fused SAP colour phase (Alg. 3, multiplicative Schwarz reading).
//
// One workgroup per (block of the given colour, rhs); one thread per site of
// the block.  The workgroup
//   1. forms the residual r = y - D x on its sites (the block's x staged in
//      LDS; neighbour values from the other colour come from global memory
//      and are not written in this phase, so there is no race),
//   2. runs n_mr minimal-residual steps on B e = r, where B is D restricted
//      to the block (hops leaving the block dropped): the current residual
//      rho lives in registers and is exchanged between sites through LDS,
//      the two inner products of each step are workgroup reductions,
//   3. adds the correction e to x on its own sites.
// Blocks of one colour never touch each other, so one launch per colour is
// one Schwarz half-sweep.  Blocks of 4^4 sites take the kernels of k_sap4.hip;
// this one serves every other shape.
#include "dirac_device.h"
#include "sap_device.h"

namespace ddamg {

namespace {

using namespace dev;

// At least two waves per SIMD: the FP64 instance would otherwise take 262
// registers and run one wave per SIMD (the FP32 ones are below 256 anyway).
template <typename T, typename S, int NR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void sap_phase_kernel(
    cx<T>* __restrict__ x, const cx<T>* __restrict__ y, GaugeView<S> gv, Geom g, int colour, int n_mr, size_t rs,
    int nrhs) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int vb = g.vblock;
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);          // [NR][12][vb]
  T* red = reinterpret_cast<T*>(lds + NR * 12 * vb);          // [nwaves][3 NR]
  const int nwaves = (blockDim.x + 63) / 64;
  // Workgroup = (block of the colour, group of NR rhs), rhs group fastest so
  // that the workgroups sharing a block's links and clover run side by side.
  // Blocks of one colour are contiguous; the swizzle gives each XCD one
  // contiguous run of them (a compact lattice region and its halo, and the
  // links read by all rhs groups of those blocks stay in that XCD's L2).
  const int ngroup = (nrhs + NR - 1) / NR;
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = colour * g.neven + wl / ngroup;
  const int r0 = (wl % ngroup) * NR;
  const int nr = min(NR, nrhs - r0);  // rhs handled by this workgroup
  const int l = threadIdx.x;
  const bool act = l < vb;
  const size_t V = g.V;
  x += (size_t)r0 * rs;
  y += (size_t)r0 * rs;
  GaugeLd<S, false> gl(gv, V);

  const int s = ci * vb + (act ? l : 0);
  const SitePos pos = site_pos(g, s);
  cx<T> rho[NR][4][3], e[NR][4][3];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        rho[r][sp][k] = mk((T)0, (T)0);
        e[r][sp][k] = mk((T)0, (T)0);
      }
  // residual r = y - D x with the current x: the block's x is staged in LDS
  // (the buffer the MR steps use later) for the in-block hops, the halo from
  // the other colour comes from global memory; a missing second rhs repeats
  // the first and is never stored
  if (act) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 12; ++k)
        lds[(r * 12 + k) * vb + l] = elem(x + (size_t)min(r, nr - 1) * rs + (size_t)k * V, (unsigned)s);
  }
  __syncthreads();
  if (act) {
    cx<T> acc[NR][4][3], p[NR][4][3];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          acc[r][sp][k] = mk((T)0, (T)0);
          p[r][sp][k] = lds[(r * 12 + 3 * sp + k) * vb + l];
        }
    sap_clover<NR, T, S>(acc, p, gl, s);
    staged_hops<0, NR, 0, T, S>(acc, lds, x, rs, nr, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<1, NR, 0, T, S>(acc, lds, x, rs, nr, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<2, NR, 0, T, S>(acc, lds, x, rs, nr, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<3, NR, 0, T, S>(acc, lds, x, rs, nr, pos, g, gl, V);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k)
          rho[r][sp][k] = elem(y + (size_t)min(r, nr - 1) * rs + (size_t)(3 * sp + k) * V, (unsigned)s) - acc[r][sp][k];
  }

  __syncthreads();  // every lane is done reading the staged x
  for (int it = 0; it < n_mr; ++it) {
    // Launder the gauge loader: the loads of B below are the same in every
    // MR step, and hoisting them out of the loop would pin them in registers
    // for the whole kernel.
    auto gli = gl;
    gli.launder();
    if (act) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int k = 0; k < 3; ++k) lds[(r * 12 + 3 * sp + k) * vb + l] = rho[r][sp][k];
    }
    __syncthreads();
    cx<T> q[NR][4][3];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k) q[r][sp][k] = mk((T)0, (T)0);
    T dots[NR][3];
#pragma unroll
    for (int r = 0; r < NR; ++r) dots[r][0] = dots[r][1] = dots[r][2] = (T)0;
    if (act) {
      sap_clover<NR, T, S>(q, rho, gli, s);
      block_hops<0, NR, 0, T, S>(q, lds, pos, g, gli);
      block_hops<1, NR, 0, T, S>(q, lds, pos, g, gli);
      block_hops<2, NR, 0, T, S>(q, lds, pos, g, gli);
      block_hops<3, NR, 0, T, S>(q, lds, pos, g, gli);
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const cx<T> t = cmulc(q[r][sp][k], rho[r][sp][k]);
            dots[r][0] += t.r;
            dots[r][1] += t.i;
            dots[r][2] += q[r][sp][k].r * q[r][sp][k].r + q[r][sp][k].i * q[r][sp][k].i;
          }
    }
    const int w = l >> 6;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const T v = wave_sum63(dots[r][c]);
        if ((l & 63) == 63) red[w * 3 * NR + 3 * r + c] = v;
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      T a_re = 0, a_im = 0, n2 = 0;
      for (int k = 0; k < nwaves; ++k) {
        a_re += red[k * 3 * NR + 3 * r + 0];
        a_im += red[k * 3 * NR + 3 * r + 1];
        n2 += red[k * 3 * NR + 3 * r + 2];
      }
      const T inv = n2 > (T)0 ? (T)1 / n2 : (T)0;
      const cx<T> alpha = mk(a_re * inv, a_im * inv);
      if (act) {
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            e[r][sp][k] = e[r][sp][k] + alpha * rho[r][sp][k];
            rho[r][sp][k] = rho[r][sp][k] - alpha * q[r][sp][k];
          }
      }
    }
  }
  if (act) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r >= nr) break;
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const size_t i = (size_t)r * rs + (size_t)(3 * sp + k) * V + s;
          x[i] = x[i] + e[r][sp][k];
        }
    }
  }
}

}  // namespace

template <typename T, typename S, int NR>
static void launch_sap_nr(cx<T>* x, const cx<T>* y, const GaugeView<S>& gv, const Geom& g, int colour, int n_mr,
                          int nrhs, hipStream_t st) {
  const int threads = ((g.vblock + 63) / 64) * 64;
  const int nwaves = threads / 64;
  const size_t rs = (size_t)12 * g.V;
  const size_t lds = (size_t)NR * 12 * g.vblock * sizeof(cx<T>) + (size_t)3 * NR * nwaves * sizeof(T);
  const int grid = g.nblocks / 2 * ((nrhs + NR - 1) / NR);
  sap_phase_kernel<T, S, NR><<<grid, threads, lds, st>>>(x, y, gv, g, colour, n_mr, rs, nrhs);
}

template <typename T, typename S>
void launch_sap_phase(cx<T>* x, const cx<T>* y, const GaugeView<S>& gv, const Geom& g, int colour, int n_mr, int nrhs,
                      hipStream_t st) {
  if (nrhs <= 0) return;
  // FP32: two right-hand sides per thread share every link and clover load.
  // FP64 keeps one per thread to fit the register file.
  if constexpr (sizeof(T) == 4) {
    if (nrhs > 1) {
      launch_sap_nr<T, S, 2>(x, y, gv, g, colour, n_mr, nrhs, st);
      return;
    }
  }
  launch_sap_nr<T, S, 1>(x, y, gv, g, colour, n_mr, nrhs, st);
}

template void launch_sap_phase<double, double>(cx<double>*, const cx<double>*, const GaugeView<double>&, const Geom&,
                                               int, int, int, hipStream_t);
template void launch_sap_phase<float, float>(cx<float>*, const cx<float>*, const GaugeView<float>&, const Geom&,
                                             int, int, int, hipStream_t);
template void launch_sap_phase<float, __half>(cx<float>*, const cx<float>*, const GaugeView<__half>&, const Geom&,
                                              int, int, int, hipStream_t);

}  // namespace ddamg
