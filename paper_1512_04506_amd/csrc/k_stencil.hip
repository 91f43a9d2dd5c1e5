// The nine-slot coarse stencil D_c (Eq. cgo), alone or followed by the dense
// per-site product with D_ee^{-1}, and that product by itself (Alg. 2):
//   out(i) = [M_i] (add(i) + cs D_self(i) xs(i) + cn sum_{slot > 0} D_slot(i) xn(nbr(i)))
// for one coarse site i per workgroup.  D_c is [site][slot][col][row]
// (column-major 2ntv x 2ntv blocks), so the blocks of a site are one dense
// matrix of nc rows and nslot nc columns in memory, and a run of rows of one
// column is one contiguous load.
//
// What bounds it is D_c itself (read once: 83 KB per site in FP16 at N_tv
// 24) and, on lattices of a few hundred coarse sites, the latency of a
// workgroup's chain.  Both kernels therefore spread the columns of all slots
// over the waves of the workgroup, with no barrier between the slots, and
// add the waves' partial results through LDS once at the end.
#include <algorithm>
#include <type_traits>

#include "mfma_device.h"

namespace ddamg {

namespace {

using namespace dev;

// the operands of one call; D: the first column used at site 0 (slot s_beg),
// dsite entries from one site to the next; ncol = nslot nc columns
template <typename T, typename S>
struct StArgs {
  cx<T>* out;
  size_t ostr;
  const cx<T>* add;
  size_t astr;
  const cx<T>* xs;  // input of slot 0, first entry of the first output site
  size_t xsstr;
  const cx<T>* xn;  // input of slots 1 .. 8, entry 0 of site xn_first
  size_t xnstr;
  int xn_first;
  T cs, cn;
  const stc_t<S>* D;
  size_t dsite;
  const float* Dsc;  // scales [site][9] (half)
  const int* nbr;    // [site][9]
  const cx<T>* M;    // per-site matrices of the second product, or null
  int out_first, s_beg, nslot, nc, nrhs;
  const int* gate;
};

// input vector (rhs 0) of slot index q (0 .. nslot - 1) at site ci and its rhs stride
template <typename T, typename S>
__device__ inline const cx<T>* st_input(const StArgs<T, S>& a, int ci, int q, size_t& str) {
  const int slot = a.s_beg + q;
  if (slot == 0) {
    str = a.xsstr;
    return a.xs + (size_t)(ci - a.out_first) * a.nc;
  }
  str = a.xnstr;
  return a.xn + (size_t)(a.nbr[ci * 9 + slot] - a.xn_first) * a.nc;
}
template <typename T, typename S>
__device__ inline T st_coef(const StArgs<T, S>& a, int ci, int q) {
  const int slot = a.s_beg + q;
  T c = slot == 0 ? a.cs : a.cn;
  if constexpr (is_half<S>()) c *= (T)a.Dsc[ci * 9 + slot];
  return c;
}

// ------------------------------------------------------------- 1 .. 4 rhs
// RP consecutive rows per lane (16 bytes of D_c per load in FP16), GL lanes
// for the rows, 64 / GL columns per wave and SW waves: column c of all slots
// belongs to column group c mod (SW 64 / GL), so every load of a lane is
// independent of the others.  The inputs, times the slot's factor, sit in
// LDS.  RP and SW: stencil_gemv_shape (blas_sizes.h).  Against one workgroup
// walking the slots with two barriers each: 19.9 -> 7.6 us for one rhs on 256
// sites (16^3x32, FP16, N_tv 24).
constexpr int ST_T = 1024;

template <typename T, int RP, int RB>
__device__ inline void st_accumulate(cx<T> acc[RP][RB], const cx<T> d[RP], const cx<T>* x) {
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    const cx<T> xj = x[j];
#pragma unroll
    for (int q = 0; q < RP; ++q) acc[q][j] = cfma(d[q], xj, acc[q][j]);
  }
}

template <typename T, typename X, int RP>
struct alignas(RP * sizeof(X)) StRows {
  X v[RP];
};

// acc over the columns c0, c0 + step, ... < ncol of the nc-row matrix D (row
// offset included), inputs xl[c][RB]
template <typename T, typename X, int RP, int RB>
__device__ inline void st_columns(cx<T> acc[RP][RB], const X* D, int nc, int c0, int step, int ncol, const cx<T>* xl) {
#pragma unroll 4
  for (int c = c0; c < ncol; c += step) {
    const StRows<T, X, RP> w = *reinterpret_cast<const StRows<T, X, RP>*>(D + (size_t)c * nc);
    cx<T> d[RP];
#pragma unroll
    for (int q = 0; q < RP; ++q) d[q] = ldc<T>(w.v, (size_t)q);
    st_accumulate<T, RP, RB>(acc, d, xl + (size_t)c * RB);
  }
}

// sum over the column groups of a wave (lanes GL apart), then red[wave][row][RB]
template <typename T, int RP, int RB>
__device__ inline void st_wave_reduce(cx<T> acc[RP][RB], int GL, bool store, cx<T>* red, int row) {
  for (int o = 32; o >= GL; o >>= 1)
#pragma unroll
    for (int q = 0; q < RP; ++q)
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        acc[q][j].r += __shfl_xor(acc[q][j].r, o, 64);
        acc[q][j].i += __shfl_xor(acc[q][j].i, o, 64);
      }
  if (store)
#pragma unroll
    for (int q = 0; q < RP; ++q)
#pragma unroll
      for (int j = 0; j < RB; ++j) red[(row + q) * RB + j] = acc[q][j];
}

template <typename T, typename S, int RP, int RB>
__global__ __launch_bounds__(ST_T) void stencil_gemv_kernel(StArgs<T, S> a, int GL) {
  if (a.gate && *a.gate == 0) return;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int nc = a.nc, ncol = a.nslot * nc;
  cx<T>* xl = reinterpret_cast<cx<T>*>(smem_raw);  // [ncol][RB]
  cx<T>* red = xl + (size_t)ncol * RB;             // [waves][nc][RB]
  const int ls = blockIdx.x, ci = a.out_first + ls;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = blockDim.x >> 6;
  for (int e = t; e < ncol * RB; e += blockDim.x) {
    const int j = e / ncol, c = e - j * ncol, q = c / nc, k = c - q * nc;
    size_t str;
    const cx<T>* x = st_input(a, ci, q, str);
    xl[c * RB + j] = j < a.nrhs ? st_coef(a, ci, q) * x[(size_t)j * str + k] : mk((T)0, (T)0);
  }
  const int rg = lane & (GL - 1), sub = lane / GL, cpw = 64 / GL;
  const bool act = RP * rg < nc;
  const int row = act ? RP * rg : 0;
  cx<T> acc[RP][RB];
#pragma unroll
  for (int q = 0; q < RP; ++q)
#pragma unroll
    for (int j = 0; j < RB; ++j) acc[q][j] = mk((T)0, (T)0);
  __syncthreads();
  st_columns<T, stc_t<S>, RP, RB>(acc, a.D + (size_t)ci * a.dsite + row, nc, w * cpw + sub, nw * cpw, ncol, xl);
  st_wave_reduce<T, RP, RB>(acc, GL, act && sub == 0, red + (size_t)w * nc * RB, row);
  __syncthreads();
  // the result, element (row, rhs) per thread; with M it is the input of the second product
  for (int e = t; e < nc * RB; e += blockDim.x) {
    const int rw = e / RB, j = e - rw * RB;
    cx<T> s = a.add && j < a.nrhs ? a.add[(size_t)j * a.astr + (size_t)ls * nc + rw] : mk((T)0, (T)0);
    for (int k = 0; k < nw; ++k) s = s + red[(size_t)k * nc * RB + e];
    if (a.M)
      xl[e] = s;
    else if (j < a.nrhs)
      a.out[(size_t)j * a.ostr + (size_t)ls * nc + rw] = s;
  }
  if (!a.M) return;
#pragma unroll
  for (int q = 0; q < RP; ++q)
#pragma unroll
    for (int j = 0; j < RB; ++j) acc[q][j] = mk((T)0, (T)0);
  __syncthreads();
  st_columns<T, cx<T>, RP, RB>(acc, a.M + (size_t)ls * nc * nc + row, nc, w * cpw + sub, nw * cpw, nc, xl);
  st_wave_reduce<T, RP, RB>(acc, GL, act && sub == 0, red + (size_t)w * nc * RB, row);
  __syncthreads();
  for (int e = t; e < nc * RB; e += blockDim.x) {
    const int rw = e / RB, j = e - rw * RB;
    cx<T> s = mk((T)0, (T)0);
    for (int k = 0; k < nw; ++k) s = s + red[(size_t)k * nc * RB + e];
    if (j < a.nrhs) a.out[(size_t)j * a.ostr + (size_t)ls * nc + rw] = s;
  }
}

// --------------------------------------------------------------- 5+ rhs
// The matrix cores: D_c times up to 16 rhs per workgroup, in chunks of 16
// columns of one slot that the waves take in turn.  Lane (li, lg) loads, of
// the four columns 4 lg .. 4 lg + 3 of a chunk, the rows RPL li .. RPL li +
// RPL - 1 (RPL = ceil(nc / 16)): 16 lanes read a whole column of D_c, 4
// columns per instruction; row RPL li + t is row li of the t-th 16-row tile,
// so a wave holds all rows and every input element is loaded and converted
// once per workgroup.  FP32 and FP64 take the 16x16x4 instructions (four
// real products per complex one).
// D_c stored in FP16 goes to v_mfma_f32_16x16x16_f16 as it is stored: the
// FP32 input is split into two FP16 parts, x s = hi + 2^-11 lo with hi =
// f16(x s), lo = f16((x s - hi) 2^11) and s a power of two per rhs and chunk
// that brings the chunk's largest |x| into [1/2, 1), so the two products
// carry the input to 2^-22 of the chunk's largest element; the slot's scale
// and 1 / s are applied to the chunk's FP32 result.  With s taken over all
// slots of a site, the inputs were read twice and every wave converted all
// of them for its own 16 rows: 314 -> 193 us for 12 rhs on 8192 sites
// at N_tv 24 (D_c 679 MB: 3.9 TB/s), 28.6 -> 11.5 us for 8 rhs on 128 sites at
// N_tv 20 in FP32 (the eight-wave workgroups of a small grid).
typedef _Float16 st_h4 __attribute__((ext_vector_type(4)));
constexpr int MM_RHS = 16;

// one chunk as loaded: entries of D_c and of the input vector of this lane's rhs
template <typename T, typename X, int RPL>
struct MmChunk {
  Run<X, RPL> d[4];
  cx<T> x[4];
  T coef;
};

// columns k0 + 4 lg + i of the matrix D (row offset included; clamped, the
// input is zero beyond nc), the input vector x of the lane's rhs
template <typename T, typename X, int RPL>
__device__ inline void mm_load(MmChunk<T, X, RPL>& c, const X* D, const cx<T>* x, int nc, int k0, int lg) {
  const int k = k0 + 4 * lg;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int kc = min(k + i, nc - 1);
    c.d[i] = load_run<X, RPL>(D + (size_t)kc * nc);
    c.x[i] = x[kc];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (k + i >= nc) c.x[i] = mk((T)0, (T)0);
}

template <typename T, int RPL>
__device__ inline void mm_chunk(typename MmAcc<T>::type re[RPL], typename MmAcc<T>::type im[RPL],
                                const MmChunk<T, cx<T>, RPL>& c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const T xr = c.coef * c.x[i].r, xi = c.coef * c.x[i].i;
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      re[t] = mm_mfma(c.d[i].v[t].r, xr, re[t]);
      im[t] = mm_mfma(c.d[i].v[t].r, xi, im[t]);
      re[t] = mm_mfma(c.d[i].v[t].i, -xi, re[t]);
      im[t] = mm_mfma(c.d[i].v[t].i, xr, im[t]);
    }
  }
}

template <typename T, int RPL>
__device__ inline void mm_chunk(mm_f4 re[RPL], mm_f4 im[RPL], const MmChunk<float, __half2, RPL>& c) {
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) m = fmaxf(m, fmaxf(fabsf(c.x[i].r), fabsf(c.x[i].i)));
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  // m in [2^(e-1), 2^e), e clamped to where 2^-e and 2^e are normal numbers
  const int e = min(max((int)(__float_as_uint(m) >> 23) - 126, -125), 125);
  const float s = __uint_as_float((unsigned)(127 - e) << 23);
  const float inv = c.coef * __uint_as_float((unsigned)(127 + e) << 23);
  st_h4 xr_h, xi_h, xr_l, xi_l, xm_h, xm_l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float br = s * c.x[i].r, bi = s * c.x[i].i;
    xr_h[i] = (_Float16)br;
    xi_h[i] = (_Float16)bi;
    xr_l[i] = (_Float16)((br - (float)xr_h[i]) * 2048.f);
    xi_l[i] = (_Float16)((bi - (float)xi_h[i]) * 2048.f);
  }
  xm_h = -xi_h;
  xm_l = -xi_l;
  const mm_f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < RPL; ++t) {
    st_h4 ar, ai;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ar[i] = (_Float16)__low2half(c.d[i].v[t]);
      ai[i] = (_Float16)__high2half(c.d[i].v[t]);
    }
    mm_f4 hr = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, xr_h, zero, 0, 0, 0);
    mm_f4 hi = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, xi_h, zero, 0, 0, 0);
    mm_f4 lr = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, xr_l, zero, 0, 0, 0);
    mm_f4 li = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, xi_l, zero, 0, 0, 0);
    hr = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, xm_h, hr, 0, 0, 0);
    hi = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, xr_h, hi, 0, 0, 0);
    lr = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, xm_l, lr, 0, 0, 0);
    li = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, xr_l, li, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      re[t][v] = fmaf(inv, fmaf(lr[v], 1.f / 2048.f, hr[v]), re[t][v]);
      im[t][v] = fmaf(inv, fmaf(li[v], 1.f / 2048.f, hi[v]), im[t][v]);
    }
  }
}

// adds the waves' tiles through red ([slots][16 rhs][nc + 1]): halves of the
// waves fold until two are left, whose tiles stay in slots 0 and 1
template <typename T, int RPL>
__device__ inline void mm_store(cx<T>* slot, const typename MmAcc<T>::type re[RPL],
                                const typename MmAcc<T>::type im[RPL], int nc, int li, int lg) {
#pragma unroll
  for (int t = 0; t < RPL; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      slot[li * (nc + 1) + min(RPL * mm_row<T>(lg, v), nc - RPL) + t] = mk(re[t][v], im[t][v]);
}
template <typename T, int RPL>
__device__ inline void mm_fold(cx<T>* red, typename MmAcc<T>::type re[RPL], typename MmAcc<T>::type im[RPL], int nc,
                               int li, int lg, int w, int nw) {
  const size_t ss = (size_t)MM_RHS * (nc + 1);
  for (int half = nw / 2; half >= 2; half >>= 1) {
    if (w >= half && w < 2 * half) mm_store<T, RPL>(red + (w - half) * ss, re, im, nc, li, lg);
    __syncthreads();
    if (w < half) {
      const cx<T>* slot = red + w * ss;
#pragma unroll
      for (int t = 0; t < RPL; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const cx<T> o = slot[li * (nc + 1) + min(RPL * mm_row<T>(lg, v), nc - RPL) + t];
          re[t][v] += o.r;
          im[t][v] += o.i;
        }
    }
    __syncthreads();
  }
  if (w < 2) mm_store<T, RPL>(red + w * ss, re, im, nc, li, lg);
  __syncthreads();
}

template <typename T, typename S, int RPL>
__global__ __launch_bounds__(512) void stencil_mm_kernel(StArgs<T, S> a) {
  if (a.gate && *a.gate == 0) return;
  using Acc = typename MmAcc<T>::type;
  using X = stc_t<S>;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  cx<T>* red = reinterpret_cast<cx<T>*>(smem_raw);
  const int nc = a.nc, nkc = (nc + 15) / 16, nchunk = a.nslot * nkc;
  const int ls = blockIdx.x, ci = a.out_first + ls;
  const int r0 = blockIdx.y * MM_RHS, nr = min(MM_RHS, a.nrhs - r0);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, nw = blockDim.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int bj = r0 + min(li, nr - 1);           // this lane's rhs (clamped)
  const int row = min(RPL * li, nc - RPL);       // first row (clamped: rows computed twice agree)
  const X* Ds = a.D + (size_t)ci * a.dsite + row;
  Acc re[RPL], im[RPL];
#pragma unroll
  for (int q = 0; q < RPL; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) re[q][v] = im[q][v] = (T)0;
  auto load = [&](MmChunk<T, X, RPL>& c, int ch) {
    const int q = ch / nkc, k0 = 16 * (ch - q * nkc);
    size_t str;
    const cx<T>* x = st_input(a, ci, q, str);
    c.coef = st_coef(a, ci, q);
    mm_load<T, X, RPL>(c, Ds + (size_t)q * nc * nc, x + (size_t)bj * str, nc, k0, lg);
  };
  MmChunk<T, X, RPL> cur, nxt;
  if (w < nchunk) load(cur, w);
  for (int ch = w; ch < nchunk; ch += nw) {
    if (ch + nw < nchunk) load(nxt, ch + nw);
    mm_chunk<T, RPL>(re, im, cur);
    cur = nxt;
  }
  mm_fold<T, RPL>(red, re, im, nc, li, lg, w, nw);
  const size_t ss = (size_t)MM_RHS * (nc + 1);
  for (int e = t; e < nr * nc; e += blockDim.x) {
    const int j = e / nc, rw = e - j * nc;
    const size_t at = (size_t)j * (nc + 1) + rw;
    cx<T> s = red[at] + red[ss + at];
    if (a.add) s = s + a.add[(size_t)(r0 + j) * a.astr + (size_t)ls * nc + rw];
    if (a.M)
      red[at] = s;
    else
      a.out[(size_t)(r0 + j) * a.ostr + (size_t)ls * nc + rw] = s;
  }
  if (!a.M) return;
  // second product: the columns of M over the first two waves (each up to
  // two chunks), their tiles in slots 1 and 2
  __syncthreads();
  if (w < 2) {
#pragma unroll
    for (int q = 0; q < RPL; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) re[q][v] = im[q][v] = (T)0;
    for (int ch = w; ch < nkc; ch += 2) {
      MmChunk<T, cx<T>, RPL> c;
      c.coef = (T)1;
      mm_load<T, cx<T>, RPL>(c, a.M + (size_t)ls * nc * nc + row, red + (size_t)min(li, nr - 1) * (nc + 1), nc, 16 * ch,
                             lg);
      mm_chunk<T, RPL>(re, im, c);
    }
    mm_store<T, RPL>(red + (1 + w) * ss, re, im, nc, li, lg);
  }
  __syncthreads();
  for (int e = t; e < nr * nc; e += blockDim.x) {
    const int j = e / nc, rw = e - j * nc;
    const size_t at = (size_t)j * (nc + 1) + rw;
    a.out[(size_t)(r0 + j) * a.ostr + (size_t)ls * nc + rw] = red[ss + at] + red[2 * ss + at];
  }
}

// Few rows on many sites (FP32 arithmetic, no second product): a wave per 16
// rows and 16 rhs walks the slots four columns at a time, which wastes none of
// a short column, and leaves its tile straight from the registers
// (stencil_by_tiles, blas_sizes.h, with times).
template <typename S>
__global__ __launch_bounds__(128) void stencil_tile_kernel(StArgs<float, S> a) {
  if (a.gate && *a.gate == 0) return;
  const int nc = a.nc, ls = blockIdx.x, ci = a.out_first + ls;
  const int r0 = blockIdx.y * MM_RHS, nr = min(MM_RHS, a.nrhs - r0);
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int r16 = 16 * (threadIdx.x >> 6);       // the wave's first row
  const int bj = r0 + min(li, nr - 1);           // this lane's rhs (clamped)
  const stc_t<S>* D = a.D + (size_t)ci * a.dsite + min(r16 + li, nc - 1);
  mm_f4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
  for (int q = 0; q < a.nslot; ++q, D += (size_t)nc * nc) {
    size_t str;
    const cx<float>* x = st_input(a, ci, q, str);
    x += (size_t)bj * str;
    const float coef = st_coef(a, ci, q);
#pragma unroll 4
    for (int k0 = 0; k0 < nc; k0 += 4) {
      const int k = k0 + lg, kc = min(k, nc - 1);
      const cx<float> d = ldc<float>(D, (size_t)kc * nc), xk = x[kc];
      const float br = k < nc ? coef * xk.r : 0.f, bi = k < nc ? coef * xk.i : 0.f;
      re = mm_mfma(d.r, br, re);
      im = mm_mfma(d.r, bi, im);
      re = mm_mfma(d.i, -bi, re);
      im = mm_mfma(d.i, br, im);
    }
  }
  if (li >= nr) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int rw = r16 + mm_row<float>(lg, v);
    if (rw >= nc) continue;
    cx<float> s = mk(re[v], im[v]);
    if (a.add) s = s + a.add[(size_t)bj * a.astr + (size_t)ls * nc + rw];
    a.out[(size_t)bj * a.ostr + (size_t)ls * nc + rw] = s;
  }
}

template <typename T, typename S, int RP, int RB>
void gemv_launch(const StArgs<T, S>& a, int nout, int nw, hipStream_t st) {
  int GL = 1;
  while (GL * RP < a.nc) GL *= 2;  // <= 32: nc <= 64, RP >= 2
  const size_t lds = ((size_t)a.nslot + nw) * a.nc * RB * sizeof(cx<T>);
  stencil_gemv_kernel<T, S, RP, RB><<<nout, 64 * nw, lds, st>>>(a, GL);
}

template <typename T, typename S, int RPL>
void mm_launch(const StArgs<T, S>& a, int nout, hipStream_t st) {
  const int ngr = (a.nrhs + MM_RHS - 1) / MM_RHS;
  // four waves, eight on grids of at most one workgroup per CU or so (FP64
  // stays at four: the partial tiles of eight do not fit)
  const int nw = sizeof(T) == 4 && nout * ngr <= 512 ? 8 : 4;
  const size_t lds = (size_t)std::max(nw / 2, 3) * MM_RHS * (a.nc + 1) * sizeof(cx<T>);
  stencil_mm_kernel<T, S, RPL><<<dim3(nout, ngr), 64 * nw, lds, st>>>(a);
}

template <typename T, typename S>
void stencil_launch(const StArgs<T, S>& a, int nout, hipStream_t st) {
  if (a.nrhs <= 0 || nout <= 0) return;
  const GemvShape g = stencil_gemv_shape(sizeof(cx<T>), is_half<S>(), a.nc, a.nslot, a.nrhs, nout);
  if (g.waves) {
    const auto run = [&](auto rb) {
      constexpr int RB = decltype(rb)::value;
      if constexpr (sizeof(T) == 4) {
        if (g.rows == 4) {
          gemv_launch<T, S, 4, RB>(a, nout, g.waves, st);
          return;
        }
      }
      gemv_launch<T, S, 2, RB>(a, nout, g.waves, st);
    };
    switch (a.nrhs) {
      case 1: run(std::integral_constant<int, 1>()); break;
      case 2: run(std::integral_constant<int, 2>()); break;
      case 3: run(std::integral_constant<int, 3>()); break;
      default: run(std::integral_constant<int, 4>()); break;
    }
    return;
  }
  if constexpr (sizeof(T) == 4) {
    const int ngr = (a.nrhs + MM_RHS - 1) / MM_RHS;
    if (!a.M && stencil_by_tiles(is_half<S>(), a.nc, a.nrhs, nout * ngr)) {
      stencil_tile_kernel<S><<<dim3(nout, ngr), 64 * ((a.nc + 15) / 16), 0, st>>>(a);
      return;
    }
  }
  switch ((a.nc + 15) / 16) {  // nc = 2 ntv <= 64
    case 1: mm_launch<T, S, 1>(a, nout, st); break;
    case 2: mm_launch<T, S, 2>(a, nout, st); break;
    case 3: mm_launch<T, S, 3>(a, nout, st); break;
    default: mm_launch<T, S, 4>(a, nout, st); break;
  }
}

}  // namespace

template <typename T, typename S>
void launch_coarse_stencil(cx<T>* out, size_t ostr, int out_first, int nout, const cx<T>* add, size_t astr,
                           const cx<T>* xs, size_t xsstr, int xs_first, T cs, const cx<T>* xn, size_t xnstr,
                           int xn_first, T cn, const CoarseView<S>& cv, const Geom& g, int nrhs, hipStream_t st,
                           const int* gate, const cx<T>* M) {
  StArgs<T, S> a;
  const size_t nn = (size_t)g.nc * g.nc;
  a.out = out;
  a.ostr = ostr;
  a.add = add;
  a.astr = astr;
  a.xs = xs ? xs + (size_t)(out_first - xs_first) * g.nc : nullptr;
  a.xsstr = xsstr;
  a.xn = xn;
  a.xnstr = xnstr;
  a.xn_first = xn_first;
  a.cs = cs;
  a.cn = cn;
  a.s_beg = cs != (T)0 ? 0 : 1;
  a.nslot = (cn != (T)0 ? 9 : 1) - a.s_beg;
  a.D = cv.D + (size_t)a.s_beg * nn;
  a.dsite = 9 * nn;
  a.Dsc = cv.Dsc;
  a.nbr = cv.nbr;
  a.M = M;
  a.out_first = out_first;
  a.nc = g.nc;
  a.nrhs = nrhs;
  a.gate = gate;
  stencil_launch<T, S>(a, nout, st);
}

template <typename T>
void launch_block_matvec(cx<T>* out, size_t ostr, const cx<T>* M, const cx<T>* x, size_t xstr, int nsites, int nc,
                         int nrhs, hipStream_t st) {
  StArgs<T, T> a{};
  a.out = out;
  a.ostr = ostr;
  a.xs = x;
  a.xsstr = xstr;
  a.cs = (T)1;
  a.D = M;
  a.dsite = (size_t)nc * nc;
  a.nslot = 1;
  a.nc = nc;
  a.nrhs = nrhs;
  stencil_launch<T, T>(a, nsites, st);
}

#define INST(T, S)                                                                                                  \
  template void launch_coarse_stencil<T, S>(cx<T>*, size_t, int, int, const cx<T>*, size_t, const cx<T>*, size_t,    \
                                            int, T, const cx<T>*, size_t, int, T, const CoarseView<S>&, const Geom&, \
                                            int, hipStream_t, const int*, const cx<T>*);
INST(double, double)
INST(float, float)
INST(float, __half)
#undef INST
template void launch_block_matvec<double>(cx<double>*, size_t, const cx<double>*, const cx<double>*, size_t, int, int,
                                          int, hipStream_t);
template void launch_block_matvec<float>(cx<float>*, size_t, const cx<float>*, const cx<float>*, size_t, int, int, int,
                                         hipStream_t);

}  // namespace ddamg
