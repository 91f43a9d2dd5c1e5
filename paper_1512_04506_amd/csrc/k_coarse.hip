// Coarse-grid kernels: restriction y_c = R y (Eq. R), prolongation
// x = P x_c with P = R^dag (Alg. 2), the backward couplings from the forward
// ones (Eq. dagger), FP16 quantisation of D_c and the inversion of the even
// self-coupling blocks for the even/odd coarse solve.
//
// Coarse vectors are [rhs][coarse site][2 ntv] complex with coarse sites in
// the internal order (even parity first).  D_c is [site][slot][col][row]
// (column-major 2ntv x 2ntv blocks) so that the lanes of a wave, one per row,
// read consecutive addresses for every column.
#include <algorithm>
#include <type_traits>

#include "mfma_device.h"

namespace ddamg {

namespace {

using namespace dev;

// ----------------------------------------------------------- restriction
// y_c[r](block, h, a) = sum over the block's sites and the six components of
// chirality h of conj(W_a) y_r.  It is bound by reading the basis and the
// fields once; on lattices of a few dozen blocks by too few waves in flight,
// so the work of a block is cut over test vectors or sites as well.
//
// Few rhs, on the vector units: workgroup = (block, share of the test-vector
// tiles), one lane per site of the block (its sites are contiguous in the
// block-major layout, so every load is coalesced), RT right-hand sides
// (blockIdx.y) kept in registers and AT test vectors at a time; the 64 lanes
// of a wave are summed by a butterfly reduce-scatter (63 shuffle-adds for 32
// values) and the waves through LDS.  One rhs: 8^4 (N_tv 16, FP32) 22.3 -> 5.1 us, 16^3x32
// (N_tv 24, FP16) 49 -> 34.6 us = 5.0 TB/s; a lone rhs used to run as four.

// One halving step of the butterfly, unrolled at compile time so that every
// register index is static: lanes with bit HALF set keep the upper half of
// their values and receive the partner's upper half, the others the lower.
template <int HALF, int NV, typename T>
__device__ inline void rs_step(T v[NV], int lane) {
  const bool up = (lane & HALF) != 0;
#pragma unroll
  for (int j = 0; j < HALF; ++j) {
    const T send = up ? v[j] : v[j + HALF];
    const T keep = up ? v[j + HALF] : v[j];
    v[j] = keep + __shfl_xor(send, HALF, 64);
  }
  if constexpr (HALF > 1) rs_step<HALF / 2, NV, T>(v, lane);
}

// v[0..NV-1] (NV a power of two <= 32): after the call lane i holds the sum
// over the 64 lanes of v[i % NV] (full sums over the lane bits >= NV first,
// then a reduce-scatter over the lower bits)
template <int NV, typename T>
__device__ inline T reduce_scatter(T v[NV], int lane) {
#pragma unroll
  for (int o = 32; o >= NV; o >>= 1)
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] += __shfl_xor(v[j], o, 64);
  rs_step<NV / 2, NV, T>(v, lane);
  return v[0];
}

template <typename T, typename S, int RT, int AT>
__global__ __launch_bounds__(256) void restrict_kernel(cx<T>* __restrict__ out, size_t ostr_r, size_t ostr_b,
                                                       const cx<T>* __restrict__ y, size_t ystr, BasisView<S> bv,
                                                       Geom g, int nrhs, int na) {
  constexpr int NV = AT * 2 * RT * 2;  // real partial sums per lane
  constexpr int MAXAT = 32 / AT;       // ntv <= 32
  __shared__ T red[4][MAXAT][NV];
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = wl / na, share = wl - ci * na;  // the shares of a block read the same y side by side
  const int r0 = blockIdx.y * RT;                // rhs of this workgroup
  y += (size_t)r0 * ystr;
  out += (size_t)r0 * ostr_r;
  nrhs -= r0;
  const int l = threadIdx.x;
  const int lane = l & 63, w = l >> 6;
  const int nw = blockDim.x >> 6;
  const bool act = l < g.vblock;
  const size_t V = g.V;
  const unsigned site = (unsigned)(ci * g.vblock + (act ? l : 0));
  const int nat = (g.ntv + AT - 1) / AT;
  const int at0 = share * nat / na, at1 = (share + 1) * nat / na;
  // Every load below is unconditional (clamped to valid addresses and
  // masked by a factor instead): a load guarded by a value that is itself
  // loaded would serialise the memory accesses of the whole loop.
  cx<T> yv[RT][12];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    const bool m = act && j < nrhs;
    const cx<T>* yr = y + (size_t)min(j, nrhs - 1) * ystr;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const cx<T> v = elem(yr + (size_t)k * V, site);
      yv[j][k] = m ? v : mk((T)0, (T)0);
    }
  }
  // no barrier inside this loop: each wave parks its reduced values per
  // test-vector tile and runs ahead
  for (int at = at0; at < at1; ++at) {
    const int a0 = at * AT;
    T v[NV];
#pragma unroll
    for (int q = 0; q < AT; ++q) {
      const int a = min(a0 + q, g.ntv - 1);
      T sc = (act && a0 + q < g.ntv) ? (T)1 : (T)0;
      if constexpr (is_half<S>()) sc *= (T)elem(bv.Wsc + (size_t)a * V, site);
      cx<T> wv[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) wv[k] = sc * ldc<T>(bv.W + ((size_t)a * 12 + k) * V, site);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < RT; ++j) {
          cx<T> acc = mk((T)0, (T)0);
#pragma unroll
          for (int k = 0; k < 6; ++k) acc = acc + cmulc(wv[6 * h + k], yv[j][6 * h + k]);
          const int idx = ((q * 2 + h) * RT + j) * 2;
          v[idx] = acc.r;
          v[idx + 1] = acc.i;
        }
    }
    const T mine = reduce_scatter<NV, T>(v, lane);
    if (lane < NV) red[w][at - at0][lane] = mine;
  }
  __syncthreads();
  for (int e = l; e < (at1 - at0) * NV; e += blockDim.x) {
    const int at = e / NV, idx = e % NV;
    T t = (T)0;
    for (int k = 0; k < nw; ++k) t += red[k][at][idx];
    // idx = ((q * 2 + h) * RT + j) * 2 + part
    const int part = idx & 1, j = (idx >> 1) % RT, h = (idx / (2 * RT)) & 1, q = idx / (4 * RT);
    const int a = (at0 + at) * AT + q;
    if (a < g.ntv && j < nrhs) {
      T* o = reinterpret_cast<T*>(out + (size_t)j * ostr_r + (size_t)ci * ostr_b + h * g.ntv + a);
      o[part] = t;
    }
  }
}

// Many rhs, on the matrix cores: per block and chirality a GEMM of ntv x nrhs
// over the rows (site, component), 16x16x4 instructions, four real products
// per complex one.  Lane (li, lg) holds test vector (and rhs) li of a 16-wide
// tile and, of 16 consecutive sites, the sites 4 lg .. 4 lg + 3: one 16-byte
// load of an FP16 basis plane (32 in FP32), the four lanes of a test vector
// side by side, and the K order (site 4 lg + i in step i) is the same for
// both operands, so they go from memory to the matrix cores with no LDS and
// no barrier.  The waves of a workgroup take the 16-site runs of the block in
// turn and are added through LDS at the end.  Test vectors and rhs beyond the
// last are read as the last and their results dropped.  Against the basis
// staged through LDS in chunks of 8 (FP64: 4) sites behind two barriers each,
// and the vector units below 16 rhs, which read the basis once per four:
// 24^3x48, FP16, N_tv 24: 24 rhs 917 -> 687 us (3.5 TB/s), 12 rhs 663 -> 414
// us (3.9 TB/s); FP64: 16^4, N_tv 20, 4 rhs 194 -> 93 us, 8^3x16, N_tv 16,
// 16 rhs 150 -> 25 us (32 blocks: 64 workgroups of eight waves instead of 32
// of four).
template <typename T, typename S, int MT, int NT>
__global__ __launch_bounds__(512) void restrict_mm_kernel(cx<T>* __restrict__ out, size_t ostr_r, size_t ostr_b,
                                                          const cx<T>* __restrict__ y, size_t ystr, BasisView<S> bv,
                                                          Geom g, int nrhs) {
  using Acc = typename MmAcc<T>::type;
  using X = stc_t<S>;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  T* red = reinterpret_cast<T*>(smem_raw);  // [nw / 2][MT NT 8][64]
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = wl >> 1, h = wl & 1;
  const int r0 = blockIdx.y * (16 * NT);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = blockDim.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int ntv = g.ntv, vb = g.vblock;
  const size_t V = g.V;
  const X* Wp[MT];
  const float* Sp[MT];
  const cx<T>* Yp[NT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int a = min(li + 16 * m, ntv - 1);
    Wp[m] = bv.W + ((size_t)a * 12 + 6 * h) * V + (size_t)ci * vb;
    Sp[m] = is_half<S>() ? bv.Wsc + (size_t)a * V + (size_t)ci * vb : nullptr;
  }
#pragma unroll
  for (int n = 0; n < NT; ++n)
    Yp[n] = y + (size_t)min(r0 + li + 16 * n, nrhs - 1) * ystr + (size_t)(6 * h) * V + (size_t)ci * vb;
  Acc re[MT][NT], im[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) re[m][n][v] = im[m][n][v] = (T)0;
  for (int s0 = 16 * w; s0 < vb; s0 += 16 * nw) {
    const int s = s0 + 4 * lg;
    const bool full = s0 + 16 <= vb;
    float sc[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[m][i] = 1.f;
    if constexpr (is_half<S>()) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (full) {
          const Run<float, 4> q = load_run<float, 4>(Sp[m] + s);
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[m][i] = q.v[i];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[m][i] = Sp[m][min(s + i, vb - 1)];
        }
      }
    }
#pragma unroll 2
    for (int k = 0; k < 6; ++k) {
      Run<X, 4> wv[MT];
      Run<cx<T>, 4> yv[NT];
      if (full) {
#pragma unroll
        for (int m = 0; m < MT; ++m) wv[m] = load_run<X, 4>(Wp[m] + (size_t)k * V + s);
#pragma unroll
        for (int n = 0; n < NT; ++n) yv[n] = load_run<cx<T>, 4>(Yp[n] + (size_t)k * V + s);
      } else {  // the sites beyond the block contribute zero
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int si = min(s + i, vb - 1);
          const bool in = s + i < vb;
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            wv[m].v[i] = Wp[m][(size_t)k * V + si];
            if (!in) sc[m][i] = 0.f;
          }
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const cx<T> v = Yp[n][(size_t)k * V + si];
            yv[n].v[i] = in ? v : mk((T)0, (T)0);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          cx<T> a = ldc<T>(wv[m].v, (size_t)i);
          if (is_half<S>() || !full) a = (T)sc[m][i] * a;
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const cx<T> b = yv[n].v[i];
            re[m][n] = mm_mfma(a.r, b.r, re[m][n]);
            im[m][n] = mm_mfma(a.r, b.i, im[m][n]);
            re[m][n] = mm_mfma(a.i, b.i, re[m][n]);
            im[m][n] = mm_mfma(-a.i, b.r, im[m][n]);
          }
        }
    }
  }
  constexpr int NP = MT * NT * 8;
  for (int half = nw >> 1; half >= 1; half >>= 1) {
    if (w >= half && w < 2 * half) {
      T* p = red + (size_t)(w - half) * NP * 64 + lane;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            p[((m * NT + n) * 8 + v) * 64] = re[m][n][v];
            p[((m * NT + n) * 8 + 4 + v) * 64] = im[m][n][v];
          }
    }
    __syncthreads();
    if (w < half) {
      const T* p = red + (size_t)w * NP * 64 + lane;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            re[m][n][v] += p[((m * NT + n) * 8 + v) * 64];
            im[m][n][v] += p[((m * NT + n) * 8 + 4 + v) * 64];
          }
    }
    __syncthreads();
  }
  if (w != 0) return;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int a = 16 * m + mm_row<T>(lg, v), r = r0 + 16 * n + li;
        if (a < ntv && r < nrhs)
          out[(size_t)r * ostr_r + (size_t)ci * ostr_b + h * ntv + a] = mk(re[m][n][v], im[m][n][v]);
      }
}

// ---------------------------------------------------------- prolongation
// x[r](site, k) = sum_a W_a(site, k) x_c[r](block, h(k), a).  Workgroup =
// (block, group of KP spin-colour components of one chirality h), the group
// fastest so that the workgroups of a block (which share its scales) run
// side by side on one XCD; one lane per site.  Each basis entry is loaded
// once per pass of PT rhs and feeds them all; the block's coarse vectors of
// chirality h sit in LDS and each broadcast read feeds the KP components
// (three in FP32; one in FP64, for the register file).
// PT rhs per pass (12 hold the registers; 1, 4 and 8 compute no padded rhs),
// the coarse vectors padded with zeros to whole passes so that the loop over
// the test vectors has no branch and four of them (eight for one rhs) are in
// flight.  Bound: HBM for few rhs, VALU beside it for 12.  FP16, N_tv 24: 1 rhs
// on 16^3x32 43.6 -> 27.7 us, 12 rhs on 24^3x48 564 -> 447 us; FP32, 8 rhs on
// 16^4 36 -> 30 us; 1 rhs on 8^4 8.3 -> 5.2 us.
template <typename T>
constexpr int prolong_kp() { return sizeof(T) == 8 ? 1 : 3; }

template <typename T, typename S, int PT>
__global__ __launch_bounds__(256) void prolong_kernel(cx<T>* __restrict__ x, size_t xstr, const cx<T>* __restrict__ xc,
                                                      size_t cstr, BasisView<S> bv, Geom g, int nrhs) {
  constexpr int KP = prolong_kp<T>(), NG = 12 / KP;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  cx<T>* xl = reinterpret_cast<cx<T>*>(smem_raw);  // [ntv][rhs of the pass] of chirality h, pass after pass
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = wl / NG, k0 = (wl % NG) * KP, h = k0 / 6;
  const int l = threadIdx.x;
  const int ntv = g.ntv;
  const size_t V = g.V;
  const int npad = (nrhs + PT - 1) / PT * PT;  // zeros beyond nrhs: no test per rhs in the loop
  for (int e = l; e < npad * ntv; e += blockDim.x) {
    const int r = e / ntv, a = e % ntv;
    xl[((r / PT) * ntv + a) * PT + r % PT] =
        r < nrhs ? xc[(size_t)r * cstr + (size_t)ci * g.nc + h * ntv + a] : mk((T)0, (T)0);
  }
  __syncthreads();
  if (l >= g.vblock) return;
  const unsigned site = (unsigned)(ci * g.vblock + l);
  for (int r0 = 0; r0 < nrhs; r0 += PT) {
    const int nr = min(PT, nrhs - r0);
    cx<T> acc[PT][KP];
#pragma unroll
    for (int j = 0; j < PT; ++j)
#pragma unroll
      for (int q = 0; q < KP; ++q) acc[j][q] = mk((T)0, (T)0);
#pragma unroll (PT == 1 ? 8 : 4)
    for (int a = 0; a < ntv; ++a) {
      T sc = (T)1;
      if constexpr (is_half<S>()) sc = (T)elem(bv.Wsc + (size_t)a * V, site);
      cx<T> wv[KP];
#pragma unroll
      for (int q = 0; q < KP; ++q) wv[q] = sc * ldc<T>(bv.W + ((size_t)a * 12 + k0 + q) * V, site);
      const cx<T>* xa = xl + (size_t)r0 * ntv + a * PT;
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const cx<T> c = xa[j];
#pragma unroll
        for (int q = 0; q < KP; ++q) acc[j][q] = cfma(wv[q], c, acc[j][q]);
      }
    }
#pragma unroll
    for (int j = 0; j < PT; ++j)
      if (j < nr)
#pragma unroll
        for (int q = 0; q < KP; ++q) x[(size_t)(r0 + j) * xstr + (size_t)(k0 + q) * V + site] = acc[j][q];
  }
}

// ------------------------------------------------------ Eq. (dagger) fill
// backward block of the neighbour j = i + mu:
//   D[j][2+2mu](row, col) = s_row s_col conj(D[i][1+2mu](col, row)),
// s = -1 on left-handed (row < ntv), +1 on right-handed components.
template <typename T>
__global__ void dagger_fill_kernel(cx<T>* Dc, const int* nbr, int nc, int ntv) {
  const int ci = blockIdx.x;
  const int mu = blockIdx.y;
  const int j = nbr[ci * 9 + 1 + 2 * mu];
  const size_t nn = (size_t)nc * nc;
  const cx<T>* fwd = Dc + ((size_t)ci * 9 + 1 + 2 * mu) * nn;
  cx<T>* bwd = Dc + ((size_t)j * 9 + 2 + 2 * mu) * nn;
  for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
    const int col = e / nc, row = e % nc;
    const T sgn = ((row < ntv) == (col < ntv)) ? (T)1 : (T)-1;
    bwd[(size_t)col * nc + row] = sgn * conj(fwd[(size_t)row * nc + col]);
  }
}

// ------------------------------------------------------ D_c quantisation
template <typename T, typename S>
__global__ __launch_bounds__(256) void quantize_coarse_kernel(stc_t<S>* Dq, float* Dsc, const cx<T>* Dc, int nc) {
  const size_t nn = (size_t)nc * nc;
  const size_t base = (size_t)blockIdx.x * nn;
  if constexpr (is_half<S>()) {
    __shared__ float red[4];
    float m = 0.f;
    for (size_t e = threadIdx.x; e < nn; e += blockDim.x) {
      cx<T> v = Dc[base + e];
      m = fmaxf(m, fmaxf(fabsf((float)v.r), fabsf((float)v.i)));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    if (threadIdx.x == 0) Dsc[blockIdx.x] = m;
    const double inv = m > 0.f ? 1.0 / (double)m : 0.0;
    for (size_t e = threadIdx.x; e < nn; e += blockDim.x) {
      cx<T> v = Dc[base + e];
      Dq[base + e] = __floats2half2_rn((float)(v.r * inv), (float)(v.i * inv));
    }
  } else {
    for (size_t e = threadIdx.x; e < nn; e += blockDim.x) stc_store(Dq, base + e, cvt<double>(Dc[base + e]));
  }
}

// ------------------------------------------------------ layout conversion
template <typename S>
__global__ void export_coarse_kernel(cx<double>* out, CoarseView<S> cv, Geom g) {
  const int ci = blockIdx.x, slot = blockIdx.y;
  const int nc = g.nc;
  int bc[4];
  int_block_coords(g, ci, bc);
  const int b = lex_block(g, bc);
  const size_t nn = (size_t)nc * nc;
  double sc = 1.0;
  if constexpr (is_half<S>()) sc = (double)cv.Dsc[ci * 9 + slot];
  for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
    const int col = e / nc, row = e % nc;
    out[((size_t)b * 9 + slot) * nn + (size_t)row * nc + col] = sc * ldc<double>(cv.D, ((size_t)ci * 9 + slot) * nn + e);
  }
}

// D_c from the exported layout (block lexicographic, row-major blocks) into
// the internal one (internal block order, column-major blocks)
template <typename T>
__global__ void coarse_import_kernel(cx<T>* D, const cx<double>* in, Geom g) {
  const int ci = blockIdx.x, slot = blockIdx.y;
  const int nc = g.nc;
  int bc[4];
  int_block_coords(g, ci, bc);
  const int b = lex_block(g, bc);
  const size_t nn = (size_t)nc * nc;
  for (int e = threadIdx.x; e < nc * nc; e += blockDim.x) {
    const int col = e / nc, row = e % nc;
    D[((size_t)ci * 9 + slot) * nn + e] = cvt<T>(in[((size_t)b * 9 + slot) * nn + (size_t)row * nc + col]);
  }
}

__device__ inline int lex_to_int_block(const Geom& g, int b) {
  int bc[4];
  bc[0] = b % g.NB[0]; b /= g.NB[0];
  bc[1] = b % g.NB[1]; b /= g.NB[1];
  bc[2] = b % g.NB[2];
  bc[3] = b / g.NB[2];
  return block_to_int(g, bc);
}

template <typename T>
__global__ void coarse_to_internal_kernel(cx<T>* out, const cx<double>* canon, Geom g, int nrhs) {
  const int nb = g.nblocks, nc = g.nc;
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)nrhs * nb * nc) return;
  const int k = (int)(idx % nc);
  const size_t rb = idx / nc;
  const int b = (int)(rb % nb);
  const size_t r = rb / nb;
  out[(r * nb + lex_to_int_block(g, b)) * nc + k] = cvt<T>(canon[idx]);
}

template <typename T>
__global__ void coarse_to_canonical_kernel(cx<double>* canon, const cx<T>* in, Geom g, int nrhs) {
  const int nb = g.nblocks, nc = g.nc;
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)nrhs * nb * nc) return;
  const int k = (int)(idx % nc);
  const size_t rb = idx / nc;
  const int b = (int)(rb % nb);
  const size_t r = rb / nb;
  canon[idx] = cvt<double>(in[(r * nb + lex_to_int_block(g, b)) * nc + k]);
}

}  // namespace

namespace {
template <typename T, typename S, int RT, int AT>
void restrict_few(cx<T>* out, size_t ostr_r, size_t ostr_b, const cx<T>* y, size_t ystr, const BasisView<S>& bv,
                  const Geom& g, int nrhs, hipStream_t st) {
  // shares of the test vectors until there are about four workgroups per CU
  const int nat = (g.ntv + AT - 1) / AT;
  const int na = std::max(1, std::min(nat, 1024 / g.nblocks));
  const int threads = ((g.vblock + 63) / 64) * 64;
  restrict_kernel<T, S, RT, AT>
      <<<dim3(g.nblocks * na, (nrhs + RT - 1) / RT), threads, 0, st>>>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, na);
}
template <typename T, typename S, int MT, int NT>
void restrict_many(cx<T>* out, size_t ostr_r, size_t ostr_b, const cx<T>* y, size_t ystr, const BasisView<S>& bv,
                   const Geom& g, int nrhs, hipStream_t st) {
  const int ngr = (nrhs + 16 * NT - 1) / (16 * NT);
  // four waves, eight while the grid is under four workgroups per CU; no more than 16-site runs
  int nw = 2 * g.nblocks * ngr < 1024 ? 8 : 4;
  while (nw > 1 && 8 * nw >= g.vblock) nw /= 2;
  const size_t lds = (size_t)(nw / 2) * MT * NT * 8 * 64 * sizeof(T);
  restrict_mm_kernel<T, S, MT, NT><<<dim3(2 * g.nblocks, ngr), 64 * nw, lds, st>>>(out, ostr_r, ostr_b, y, ystr, bv,
                                                                                     g, nrhs);
}
}  // namespace

template <typename T, typename S>
void launch_restrict(cx<T>* out, size_t ostr_r, size_t ostr_b, const cx<T>* y, size_t ystr, const BasisView<S>& bv,
                     const Geom& g, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  constexpr bool f32 = sizeof(T) == 4;
  if (nrhs == 1)
    restrict_few<T, S, 1, f32 ? 4 : 2>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else if (nrhs == 2)
    restrict_few<T, S, 2, f32 ? 2 : 1>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else if (restrict_by_lanes(f32, g.ntv, g.vblock, nrhs))
    restrict_few<T, S, f32 ? 4 : 2, f32 ? 2 : 1>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else if (g.ntv <= 16 && nrhs <= 16)
    restrict_many<T, S, 1, 1>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else if (g.ntv <= 16)
    restrict_many<T, S, 1, 2>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else if (nrhs <= 16)
    restrict_many<T, S, 2, 1>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
  else
    restrict_many<T, S, 2, 2>(out, ostr_r, ostr_b, y, ystr, bv, g, nrhs, st);
}

template <typename T, typename S>
void launch_prolong(cx<T>* x, size_t xstr, const cx<T>* xc, size_t cstr, const BasisView<S>& bv, const Geom& g,
                    int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  const int threads = ((g.vblock + 63) / 64) * 64;
  const auto run = [&](auto pt) {
    constexpr int PT = decltype(pt)::value;
    const size_t lds = (size_t)((nrhs + PT - 1) / PT * PT) * g.ntv * sizeof(cx<T>);
    prolong_kernel<T, S, PT>
        <<<g.nblocks * (12 / prolong_kp<T>()), threads, lds, st>>>(x, xstr, xc, cstr, bv, g, nrhs);
  };
  if (nrhs == 1)
    run(std::integral_constant<int, 1>());
  else if (nrhs <= 4)
    run(std::integral_constant<int, 4>());
  else if (nrhs <= 8)
    run(std::integral_constant<int, 8>());
  else
    run(std::integral_constant<int, 12>());
}

template <typename T>
void launch_dagger_fill(cx<T>* Dc, const int* nbr, const Geom& g, hipStream_t st) {
  dagger_fill_kernel<T><<<dim3(g.nblocks, 4), 256, 0, st>>>(Dc, nbr, g.nc, g.ntv);
}

template <typename T, typename S>
void launch_quantize_coarse(stc_t<S>* Dq, float* Dsc, const cx<T>* Dc, const Geom& g, hipStream_t st) {
  quantize_coarse_kernel<T, S><<<g.nblocks * 9, 256, 0, st>>>(Dq, Dsc, Dc, g.nc);
}

template <typename T, typename S>
void launch_export_coarse(cx<double>* out, const CoarseView<S>& cv, const Geom& g, hipStream_t st) {
  export_coarse_kernel<S><<<dim3(g.nblocks, 9), 256, 0, st>>>(out, cv, g);
}

template <typename T>
void launch_coarse_import(cx<T>* D, const cx<double>* in, const Geom& g, hipStream_t st) {
  coarse_import_kernel<T><<<dim3(g.nblocks, 9), 256, 0, st>>>(D, in, g);
}

template <typename T>
void launch_coarse_to_internal(cx<T>* out, const cx<double>* canon, const Geom& g, int nrhs, hipStream_t st) {
  size_t n = (size_t)nrhs * g.nblocks * g.nc;
  if (n) coarse_to_internal_kernel<T><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(out, canon, g, nrhs);
}
template <typename T>
void launch_coarse_to_canonical(cx<double>* canon, const cx<T>* in, const Geom& g, int nrhs, hipStream_t st) {
  size_t n = (size_t)nrhs * g.nblocks * g.nc;
  if (n) coarse_to_canonical_kernel<T><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(canon, in, g, nrhs);
}

#define INST_TS(T, S)                                                                                               \
  template void launch_restrict<T, S>(cx<T>*, size_t, size_t, const cx<T>*, size_t, const BasisView<S>&,            \
                                      const Geom&, int, hipStream_t);                                                \
  template void launch_prolong<T, S>(cx<T>*, size_t, const cx<T>*, size_t, const BasisView<S>&, const Geom&, int,    \
                                     hipStream_t);                                                                   \
  template void launch_quantize_coarse<T, S>(stc_t<S>*, float*, const cx<T>*, const Geom&, hipStream_t);             \
  template void launch_export_coarse<T, S>(cx<double>*, const CoarseView<S>&, const Geom&, hipStream_t);
INST_TS(double, double)
INST_TS(float, float)
INST_TS(float, __half)
#undef INST_TS

#define INST_T(T)                                                                                                   \
  template void launch_dagger_fill<T>(cx<T>*, const int*, const Geom&, hipStream_t);                                 \
  template void launch_coarse_import<T>(cx<T>*, const cx<double>*, const Geom&, hipStream_t);                        \
  template void launch_coarse_to_internal<T>(cx<T>*, const cx<double>*, const Geom&, int, hipStream_t);              \
  template void launch_coarse_to_canonical<T>(cx<double>*, const cx<T>*, const Geom&, int, hipStream_t);
INST_T(double)
INST_T(float)
#undef INST_T

}  // namespace ddamg
