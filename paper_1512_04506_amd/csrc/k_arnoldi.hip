// The coarse GMRES around its operator (Alg. 2), one workgroup per rhs: the
// start of a cycle, an Arnoldi step (classical Gram-Schmidt twice, the norm,
// the Givens rotations and the convergence test) and the end of a cycle.  At
// the end, the scalar work of the outer Gram-Schmidt.
//
// A coarse vector of a lattice up to 16^3x32 is some 10^4 elements, 100 KB
// that lie in L2: what bounds the first steps of a cycle is the number of
// dependent launches and of reductions over workgroups, not the data.  One
// workgroup holds the new vector in registers through the whole step and
// reduces within itself, so a step is one launch instead of ten (mdot and its
// final sum, maxpy, twice, the norm, the column, the scaling) and a start one
// instead of five.  It reads the k + 1 basis vectors four times through one
// compute unit, so its time grows with k where theirs hardly does: 12288
// elements, FP32, one rhs, 22 us a step over the first two, 46 over eight, 72
// over fifteen, against 49, 76 and 108 of the separate launches with 8192
// elements to a workgroup.  arnoldi_one_group (blas_sizes.h) says up to which k
// a step is taken here.  A thread holds at most 24 elements in FP32, 16 in
// FP64 (the registers of a 1024-lane workgroup); longer vectors keep the
// many-workgroup kernels of k_blas.hip throughout.
#include "krylov_device.h"

namespace ddamg {

namespace {

using namespace dev;

// elements whose loads may be in flight together: the registers of a
// 1024-lane workgroup (128) hold no more beside the vector
template <int EPT>
constexpr int hold() { return EPT > 16 ? 4 : 8; }

// h[j] = V_j^H w, j < nv (element e = t + AT i of the workgroup's vector in w[i])
template <typename T, int EPT>
__device__ inline void sw_dots(cx<double>* h, const cx<T>* V, size_t vsj, int nv, const cx<T> w[EPT], int n,
                               double (*red)[AW]) {
  constexpr int HOLD = hold<EPT>();
  for (int j0 = 0; j0 < nv; j0 += AJ) {
    cx<T> acc[AJ];
#pragma unroll
    for (int q = 0; q < AJ; ++q) acc[q] = mk((T)0, (T)0);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      if ((int)threadIdx.x < n - AT * i) {
#pragma unroll
        for (int q = 0; q < AJ; ++q)
          if (j0 + q < nv) acc[q] = cfmac(elem(V + (size_t)(j0 + q) * vsj + AT * i, threadIdx.x), w[i], acc[q]);
      }
      if (i % HOLD == HOLD - 1) asm volatile("" ::: "memory");
    }
    cx<double> d[AJ];
#pragma unroll
    for (int q = 0; q < AJ; ++q) d[q] = cvt<double>(acc[q]);
    block_sum(h + j0, d, min(AJ, nv - j0), red);
  }
}
// |w|^2 into h[0].r
template <typename T, int EPT>
__device__ inline void sw_norm2(cx<double>* h, const cx<T> w[EPT], double (*red)[AW]) {
  cx<double> d[AJ];
#pragma unroll
  for (int q = 0; q < AJ; ++q) d[q] = mk(0.0, 0.0);
  T s = (T)0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) s += w[i].r * w[i].r + w[i].i * w[i].i;  // elements beyond n are zero
  d[0].r = (double)s;
  block_sum(h, d, 1, red);
}
// w -= sum_j h_j V_j
template <typename T, int EPT>
__device__ inline void sw_update(cx<T> w[EPT], const cx<double>* h, const cx<T>* V, size_t vsj, int nv, int n) {
  constexpr int HOLD = hold<EPT>();
  for (int j = 0; j < nv; ++j) {
    const cx<T> c = cvt<T>(-1.0 * h[j]);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      if ((int)threadIdx.x < n - AT * i) w[i] = cfma(c, elem(V + (size_t)j * vsj + AT * i, threadIdx.x), w[i]);
      if (i % HOLD == HOLD - 1) asm volatile("" ::: "memory");
    }
  }
}

// an rhs's active flag for the host, in its pinned memory: a copy of the
// flags behind the kernel was another 3 us on the stream for each step
__device__ inline void post_flag(int* host_active, int r, int act) {
  __hip_atomic_store(host_active + r, act, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Start of a cycle: V_0 = r / |r| with r = b_o - c_w (c_w null: b_o, the
// first cycle, whose x_o is set to zero and whose stop threshold tol |y_c|
// is computed, tol < 0: never test), the state of arnoldi_start_kernel.
// s.any counts the active rhs: every rhs adds the change of its own flag, and
// the first cycle takes down what an earlier call of more rhs, stopped by its
// iteration limit, left in the flags beyond this one's (of nflags).
template <typename T, int EPT>
__global__ __launch_bounds__(AT) void coarse_start_kernel(ArnoldiState s, cx<T>* V0, size_t vsr, const cx<T>* bo,
                                                          const cx<T>* cw, size_t bstr, int n, cx<T>* xo, size_t xstr,
                                                          const cx<T>* yc, size_t ystr, int nc_all, double tol,
                                                          int* host_active, int nflags) {
  __shared__ double red[8][AW];
  __shared__ cx<double> h[AJ];
  const int r = blockIdx.x, t = threadIdx.x, m = s.m;
  bo += (size_t)r * bstr;
  V0 += (size_t)r * vsr;
  cx<T> w[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) w[i] = t < n - AT * i ? elem(bo + AT * i, (unsigned)t) : mk((T)0, (T)0);
  // |r|^2 and, in the first cycle, |y_c|^2 in one reduction
  cx<double> d[AJ];
#pragma unroll
  for (int q = 0; q < AJ; ++q) d[q] = mk(0.0, 0.0);
  if (cw) {
    cw += (size_t)r * bstr;
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      if (t < n - AT * i) w[i] = w[i] - elem(cw + AT * i, (unsigned)t);
      if (i % hold<EPT>() == hold<EPT>() - 1) asm volatile("" ::: "memory");
    }
  } else {
    const cx<T>* y = yc + (size_t)r * ystr;
    for (int e0 = t; e0 < nc_all; e0 += 8 * AT) {  // at most eight in a chain of T
      T a = (T)0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (e0 + q * AT < nc_all) a += y[e0 + q * AT].r * y[e0 + q * AT].r + y[e0 + q * AT].i * y[e0 + q * AT].i;
      d[1].r += (double)a;
    }
    for (int e = t; e < n; e += AT) xo[(size_t)r * xstr + e] = mk((T)0, (T)0);
    if (r == 0)
      for (int q = gridDim.x + t; q < nflags; q += AT)
        if (s.active[q]) {
          s.active[q] = 0;
          atomicAdd(s.any, -1);
        }
  }
  T a = (T)0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) a += w[i].r * w[i].r + w[i].i * w[i].i;
  d[0].r = (double)a;
  block_sum(h, d, 2, red);
  const double abstol = cw ? s.abstol[r] : tol < 0.0 ? -1.0 : tol * sqrt(fmax(h[1].r, 0.0));
  const double beta = sqrt(fmax(h[0].r, 0.0));
  const bool act = abstol < 0.0 ? beta > 0.0 : beta > abstol;
  const double inv = act ? 1.0 / beta : 0.0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = t + AT * i;
    if (e < n) V0[e] = cvt<T>(inv * cvt<double>(w[i]));
  }
  if (t <= m) s.g[(size_t)r * (m + 1) + t] = mk(t == 0 ? beta : 0.0, 0.0);
  if (t == 0) {
    const int was = s.active[r], now = act ? 1 : 0;
    post_flag(host_active, r, now);
    s.abstol[r] = abstol;
    s.active[r] = now;
    s.inv_h[r] = inv;
    s.kdone[r] = 0;
    s.est[r] = beta;
    if (now != was) atomicAdd(s.any, now - was);
  }
}

// Column k of rhs r, H[0 .. k] in LDS, subdiagonal hn: the rotations cs, sn
// of the earlier columns, the new one, the rotated rhs (gk: its entry k), the
// estimate and the stop test of arnoldi_column_kernel.  One lane; H[0 .. k +
// 1] is left for the caller to store.
__device__ inline bool finish_column(const ArnoldiState& s, int r, int k, cx<double>* H, const double* cs,
                                     const cx<double>* sn, cx<double> gk, double tol, double hn) {
  const int m = s.m;
  H[k + 1] = mk(hn, 0.0);
  for (int j = 0; j < k; ++j) {
    const cx<double> u = cs[j] * H[j] + sn[j] * H[j + 1];
    H[j + 1] = cs[j] * H[j + 1] - conj(sn[j]) * H[j];
    H[j] = u;
  }
  double c;
  cx<double> sv, rr;
  givens(H[k], H[k + 1], c, sv, rr);
  H[k] = rr;
  H[k + 1] = mk(0.0, 0.0);
  const cx<double> gn = neg(conj(sv) * gk);
  const double est = sqrt(cabs2(gn));
  const bool stop = !(hn > 0.0) || (tol >= 0.0 && est <= tol) || k + 1 >= m;
  s.cs[(size_t)r * m + k] = mk(c, 0.0);
  s.sn[(size_t)r * m + k] = sv;
  s.g[(size_t)r * (m + 1) + k] = c * gk;
  s.g[(size_t)r * (m + 1) + k + 1] = gn;
  s.est[r] = est;
  s.kdone[r] = k + 1;
  s.inv_h[r] = stop ? 0.0 : 1.0 / hn;
  if (stop) {
    s.active[r] = 0;
    atomicAdd(s.any, -1);
  }
  return stop;
}

// Arnoldi step k: w = V_{k+1} (the operator applied to V_k) orthogonalised
// against V_0 .. V_k by classical Gram-Schmidt twice and normalised in
// place; the column of H, the rotations and the stop test of
// arnoldi_column_kernel, whose state of the earlier columns is read into LDS
// beside the vector (read one after the other by one lane it took as long as
// the inner products).  An rhs that stops keeps its vector unscaled.
template <typename T, int EPT>
__global__ __launch_bounds__(AT) void coarse_arnoldi_kernel(ArnoldiState s, int k, cx<T>* Vb, size_t vsj, size_t vsr,
                                                            int n, int* host_active) {
  __shared__ double red[8][AW];
  __shared__ cx<double> h1[64 + AJ], h2[64 + AJ], hn2[AJ], sn[64], H[66], gk;
  __shared__ double cs[64], tol, inv;
  const int r = blockIdx.x, t = threadIdx.x, m = s.m;
  if (!s.active[r]) {
    if (t == 0) {
      s.inv_h[r] = 0.0;
      post_flag(host_active, r, 0);
    }
    return;
  }
  const cx<T>* V = Vb + (size_t)r * vsr;
  cx<T>* wg = Vb + (size_t)(k + 1) * vsj + (size_t)r * vsr;
  cx<T> w[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    w[i] = t < n - AT * i ? elem(wg + AT * i, (unsigned)t) : mk((T)0, (T)0);
  }
  if (t < k) {  // k < 64
    cs[t] = s.cs[(size_t)r * m + t].r;
    sn[t] = s.sn[(size_t)r * m + t];
  }
  if (t == 64) gk = s.g[(size_t)r * (m + 1) + k];
  if (t == 128) tol = s.abstol[r];
  sw_dots<T, EPT>(h1, V, vsj, k + 1, w, n, red);
  sw_update<T, EPT>(w, h1, V, vsj, k + 1, n);
  sw_dots<T, EPT>(h2, V, vsj, k + 1, w, n, red);
  sw_update<T, EPT>(w, h2, V, vsj, k + 1, n);
  sw_norm2<T, EPT>(hn2, w, red);
  if (t == 0) {
    for (int j = 0; j <= k; ++j) H[j] = h1[j] + h2[j];
    const double hn = sqrt(fmax(hn2[0].r, 0.0));
    const bool stop = finish_column(s, r, k, H, cs, sn, gk, tol, hn);
    post_flag(host_active, r, stop ? 0 : 1);
    inv = stop ? 1.0 : 1.0 / hn;
  }
  __syncthreads();
  if (t <= k + 1) s.H[(size_t)r * (m + 1) * m + (size_t)k * (m + 1) + t] = H[t];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if (t < n - AT * i) wg[AT * i + t] = cvt<T>(inv * cvt<double>(w[i]));
  }
}

// End of a cycle: y = H^{-1} g over the kdone columns of the rhs (back
// substitution by columns, lane j of every wave holding g_j), x_o += V y for
// the workgroup's elements
constexpr int FT = 256;
constexpr int F_ELEMS = 2048;
template <typename T>
__global__ __launch_bounds__(FT) void coarse_finish_kernel(ArnoldiState s, const cx<T>* Vb, size_t vsj, size_t vsr,
                                                           cx<T>* xo, size_t xstr, size_t n) {
  __shared__ cx<T> y[64];
  const int r = blockIdx.y, lane = threadIdx.x & 63, m = s.m;
  const int kd = s.kdone[r];  // <= m <= 64
  if (kd == 0) return;
  if (threadIdx.x < 64) {
    const cx<double>* H = s.H + (size_t)r * (m + 1) * m;
    cx<double> g = lane < kd ? s.g[(size_t)r * (m + 1) + lane] : mk(0.0, 0.0);
    for (int i0 = kd - 1; i0 >= 0; i0 -= 4) {
      cx<double> hc[4];  // four columns in flight
#pragma unroll
      for (int q = 0; q < 4; ++q)
        hc[q] = lane <= i0 - q ? H[(size_t)(i0 - q) * (m + 1) + lane] : mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 - q;
        if (i < 0) break;
        const cx<double> d = mk(__shfl(hc[q].r, i, 64), __shfl(hc[q].i, i, 64));
        const cx<double> gi = mk(__shfl(g.r, i, 64), __shfl(g.i, i, 64));
        const double dn = cabs2(d);
        const cx<double> yi = dn > 0.0 ? (1.0 / dn) * (conj(d) * gi) : mk(0.0, 0.0);
        if (lane == i) g = yi;
        if (lane < i) g = g - hc[q] * yi;
      }
    }
    if (lane < kd) y[lane] = cvt<T>(g);
  }
  __syncthreads();
  const cx<T>* V = Vb + (size_t)r * vsr;
  cx<T>* x = xo + (size_t)r * xstr;
  const size_t e0 = (size_t)blockIdx.x * F_ELEMS;
  for (size_t e = e0 + threadIdx.x; e < min(n, e0 + F_ELEMS); e += FT) {
    cx<T> acc = x[e];
#pragma unroll 4
    for (int j = 0; j < kd; ++j) acc = acc + y[j] * V[(size_t)j * vsj + e];
    x[e] = acc;
  }
}

// ------------------------------------------------------ outer Gram-Schmidt
// The scalar work after each of the two passes over the outer basis, one
// workgroup per rhs: the partial sums of its inner products, a wave for each,
// and what follows from them.  Each was a chain of single-wave launches (sums
// 4, coefficients 5; sums 4, norm 5, column 5 us and a copy of the flags to
// the host) that no vector work hides when a lattice is small.  8^4, one rhs,
// seven steps: 5 and 4 us now, the solve 2225 -> 2142 us; 16^3x32 3770 -> 3670.
// out[j] (LDS), j < nvec: sum over the chunks of part[j][chunk]
__device__ inline void sum_parts(cx<double>* out, const cx<double>* part, int nvec, int nchunk) {
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x >> 6; j < nvec; j += AW) {
    double re = 0.0, im = 0.0;
#pragma unroll 4
    for (int c = lane; c < nchunk; c += 64) {
      const cx<double> v = part[(size_t)j * nchunk + c];
      re += v.r;
      im += v.i;
    }
    re = wave_sum_d(re);
    im = wave_sum_d(im);
    if (lane == 0) out[j] = mk(re, im);
  }
  __syncthreads();
}

// Before the deferred pass, with h[j] = V_j^H w (j <= k) and |w|^2: if
// correct, c[j] = h2[j] (j < k), the pending vector's corrections, kept apart
// from h2 (which the pass's sums overwrite), and h[k] = sigma (h[k] -
// sum_{j<k} conj(c_j) h[j]), the inner product of w with the corrected v_k
// from those with the stored vectors; then wsc = 1 / |w'| from |w'|^2 =
// |w|^2 - sum_{j<=k} |h_j|^2, floored at 1e-20 |w|^2 against cancellation
// (only a scale: the exact |w''| follows the pass).
__global__ __launch_bounds__(AT) void gs_coef_kernel(const cx<double>* part, int nchunk, cx<double>* h, cx<double>* c,
                                                     const cx<double>* h2, int ldh, const double* sigma, int k,
                                                     int correct, double* wsc, const int* active) {
  __shared__ cx<double> hs[GS_FUSED_MAXV + 1];
  const int r = blockIdx.x, t = threadIdx.x;
  if (!active[r]) return;
  sum_parts(hs, part + (size_t)r * (k + 2) * nchunk, k + 2, nchunk);
  if (t >= 64) return;
  cx<double> hj = t <= k ? hs[t] : mk(0.0, 0.0);
  if (correct) {
    cx<double> d = mk(0.0, 0.0);
    if (t < k) {
      const cx<double> cj = h2[(size_t)r * ldh + t];
      c[(size_t)r * ldh + t] = cj;
      d = conj(cj) * hj;
    }
    d = mk(wave_sum_d(d.r), wave_sum_d(d.i));
    if (t == k) hj = sigma[r] * (hj - d);
  }
  if (t <= k) h[(size_t)r * ldh + t] = hj;
  const double n = wave_sum_d(cabs2(hj));
  if (t == 0) {
    const double w2 = hs[k + 1].r, e = fmax(w2 - n, 1e-20 * w2);
    wsc[r] = (e > 0.0 && isfinite(e)) ? 1.0 / sqrt(e) : 0.0;
  }
}

// After it, with h2[j] = V_j^H w' (j <= k) and |w'|^2: |w''|^2 = |w'|^2 -
// sum_j |h2_j|^2 (w'' = w' - V h2 with V orthonormal), the factor that
// normalises w'' (zero for a vanishing or non-finite norm: the step then
// stops that rhs) and column k, H = h1 + h2.
__global__ __launch_bounds__(AT) void gs_column_kernel(ArnoldiState s, int k, const cx<double>* part, int nchunk,
                                                       const cx<double>* h1, cx<double>* h2, int ldh, double* inv,
                                                       int* host_active) {
  __shared__ cx<double> hs[GS_FUSED_MAXV + 1], H[GS_FUSED_MAXV + 2], sn[GS_FUSED_MAXV], gk;
  __shared__ double cs[GS_FUSED_MAXV], tol, n2;
  const int r = blockIdx.x, t = threadIdx.x, m = s.m;
  if (!s.active[r]) {
    if (t == 0) {
      s.inv_h[r] = 0.0;
      post_flag(host_active, r, 0);
    }
    return;
  }
  if (t < k) {
    cs[t] = s.cs[(size_t)r * m + t].r;
    sn[t] = s.sn[(size_t)r * m + t];
  }
  if (t <= k) H[t] = h1[(size_t)r * ldh + t];
  if (t == 64) gk = s.g[(size_t)r * (m + 1) + k];
  if (t == 128) tol = s.abstol[r];
  sum_parts(hs, part + (size_t)r * (k + 2) * nchunk, k + 2, nchunk);
  if (t < 64) {
    const cx<double> v = t <= k ? hs[t] : mk(0.0, 0.0);
    if (t <= k) {
      h2[(size_t)r * ldh + t] = v;
      H[t] = H[t] + v;
    }
    const double n = wave_sum_d(cabs2(v));
    if (t == 0) n2 = fmax(hs[k + 1].r - n, 0.0);
  }
  __syncthreads();
  if (t == 0) {
    const double hn = sqrt(n2);
    inv[r] = (hn > 0.0 && isfinite(hn)) ? 1.0 / hn : 0.0;
    post_flag(host_active, r, finish_column(s, r, k, H, cs, sn, gk, tol, hn) ? 0 : 1);
  }
  __syncthreads();
  if (t <= k + 1) s.H[(size_t)r * (m + 1) * m + (size_t)k * (m + 1) + t] = H[t];
}

// elements per thread: the narrowest of 4, 8, 16, 24 (FP64 to 16: registers)
template <typename T, typename F>
void with_ept(size_t n, F&& f) {
  if (n <= (size_t)AT * 4)
    f(std::integral_constant<int, 4>());
  else if (n <= (size_t)AT * 8)
    f(std::integral_constant<int, 8>());
  else if (n <= (size_t)AT * 16)
    f(std::integral_constant<int, 16>());
  else if constexpr (sizeof(T) == 4)
    f(std::integral_constant<int, 24>());
}

}  // namespace

template <typename T>
bool arnoldi_fits(size_t n) {
  return n <= (size_t)AT * (sizeof(T) == 4 ? 24 : 16);
}

template <typename T>
void launch_coarse_start(ArnoldiState s, cx<T>* V0, size_t vsr, const cx<T>* bo, const cx<T>* cw, size_t bstr, size_t n,
                         cx<T>* xo, size_t xstr, const cx<T>* yc, size_t ystr, size_t n_all, double tol,
                         int* host_active, int nrhs, int nflags, hipStream_t st) {
  if (nrhs <= 0) return;
  with_ept<T>(n, [&](auto e) {
    coarse_start_kernel<T, decltype(e)::value>
        <<<nrhs, AT, 0, st>>>(s, V0, vsr, bo, cw, bstr, (int)n, xo, xstr, yc, ystr, (int)n_all, tol,
                               host_active, nflags);
  });
}

template <typename T>
void launch_coarse_arnoldi(ArnoldiState s, int k, cx<T>* Vb, size_t vsj, size_t vsr, size_t n, int* host_active,
                           int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  with_ept<T>(n, [&](auto e) {
    coarse_arnoldi_kernel<T, decltype(e)::value><<<nrhs, AT, 0, st>>>(s, k, Vb, vsj, vsr, (int)n, host_active);
  });
}

void launch_gs_coef(const cx<double>* part, int nchunk, cx<double>* h, cx<double>* c, const cx<double>* h2, int ldh,
                    const double* sigma, int k, bool correct, double* wsc, int nrhs, const int* active,
                    hipStream_t st) {
  if (nrhs <= 0) return;
  gs_coef_kernel<<<nrhs, AT, 0, st>>>(part, nchunk, h, c, h2, ldh, sigma, k, correct ? 1 : 0, wsc, active);
}

void launch_gs_column(ArnoldiState s, int k, const cx<double>* part, int nchunk, const cx<double>* h1, cx<double>* h2,
                      int ldh, double* inv, int* host_active, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  gs_column_kernel<<<nrhs, AT, 0, st>>>(s, k, part, nchunk, h1, h2, ldh, inv, host_active);
}

template <typename T>
void launch_coarse_finish(ArnoldiState s, const cx<T>* Vb, size_t vsj, size_t vsr, cx<T>* xo, size_t xstr, size_t n,
                          int nrhs, hipStream_t st) {
  if (nrhs <= 0 || n == 0) return;
  coarse_finish_kernel<T>
      <<<dim3((unsigned)((n + F_ELEMS - 1) / F_ELEMS), nrhs), FT, 0, st>>>(s, Vb, vsj, vsr, xo, xstr, n);
}

#define INST(T)                                                                                                        \
  template bool arnoldi_fits<T>(size_t);                                                                               \
  template void launch_coarse_start<T>(ArnoldiState, cx<T>*, size_t, const cx<T>*, const cx<T>*, size_t, size_t,       \
                                       cx<T>*, size_t, const cx<T>*, size_t, size_t, double, int*, int, int,           \
                                       hipStream_t);                                                                   \
  template void launch_coarse_arnoldi<T>(ArnoldiState, int, cx<T>*, size_t, size_t, size_t, int*, int, hipStream_t);   \
  template void launch_coarse_finish<T>(ArnoldiState, const cx<T>*, size_t, size_t, cx<T>*, size_t, size_t, int,       \
                                        hipStream_t);
INST(double)
INST(float)
#undef INST

}  // namespace ddamg
