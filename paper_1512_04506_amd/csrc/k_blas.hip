// Krylov linear algebra on block vectors (one independent system per rhs):
// several inner products in one pass (the classical Gram-Schmidt step of
// GMRES), linear combinations, scaling, and the Arnoldi/Givens state of
// GMRES kept on the device in FP64 (Hessenberg least squares).
//
// Reductions are deterministic: each workgroup writes one partial per
// (rhs, vector, chunk) and a second kernel sums the chunks in a fixed
// order, so repeated runs give bitwise identical results.
#include "krylov_device.h"

namespace ddamg {

namespace {

using namespace dev;

constexpr int BT = 256;
constexpr int JG = 8;  // basis vectors per pass over the chunk
constexpr int MAX_MDOT_VECS = 66;  // restart length 64 plus w itself

// With a single chunk the workgroup's sums are the inner products: they go
// straight to h (row stride ldh) and no final kernel runs.
template <typename T>
__global__ __launch_bounds__(BT) void mdot_partial_kernel(cx<double>* part, const cx<T>* __restrict__ Vb,
                                                          size_t vsj, size_t vsr, int nvec,
                                                          const cx<T>* __restrict__ w, size_t wsr, size_t n,
                                                          size_t chunk, int nchunk, const int* active,
                                                          cx<double>* h, int ldh) {
  __shared__ cx<double> red[MAX_MDOT_VECS][BT / 64];
  const int c = blockIdx.x;
  const int r = blockIdx.y;
  if (active && !active[r]) return;
  const size_t beg = (size_t)c * chunk;
  const size_t end = min(n, beg + chunk);
  const cx<T>* wr = w + (size_t)r * wsr;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int j0 = 0; j0 < nvec; j0 += JG) {
    cx<T> acc[JG];
#pragma unroll
    for (int q = 0; q < JG; ++q) acc[q] = mk((T)0, (T)0);
    for (size_t i = beg + threadIdx.x; i < end; i += BT) {
      const cx<T> wv = wr[i];
#pragma unroll
      for (int q = 0; q < JG; ++q)
        if (j0 + q < nvec) acc[q] = acc[q] + cmulc(Vb[(size_t)(j0 + q) * vsj + (size_t)r * vsr + i], wv);
    }
#pragma unroll
    for (int q = 0; q < JG; ++q) {
      double re = wave_sum_d((double)acc[q].r), im = wave_sum_d((double)acc[q].i);
      if (lane == 0 && j0 + q < nvec) red[j0 + q][wid] = mk(re, im);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nvec; j += BT) {
    cx<double> s = mk(0.0, 0.0);
    for (int k = 0; k < BT / 64; ++k) s = s + red[j][k];
    if (h && nchunk == 1)
      h[(size_t)r * ldh + j] = s;
    else
      part[((size_t)r * nvec + j) * nchunk + c] = s;
  }
}

__global__ void mdot_final_kernel(cx<double>* h, int ldh, const cx<double>* part, int nvec, int nchunk,
                                  const int* active) {
  const int j = blockIdx.x;
  const int r = blockIdx.y;
  if (active && !active[r]) return;
  double re = 0.0, im = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 64) {
    cx<double> v = part[((size_t)r * nvec + j) * nchunk + c];
    re += v.r;
    im += v.i;
  }
  re = wave_sum_d(re);
  im = wave_sum_d(im);
  if (threadIdx.x == 0) h[(size_t)r * ldh + j] = mk(re, im);
}

// w <- (w + sign sum_j h_j V_j) [* post[r] if post], and an FP32 copy of the
// result in w32 (same strides) if w32 is given
template <typename Tw, typename Tv>
__global__ __launch_bounds__(BT) void maxpy_kernel(cx<Tw>* w, size_t wsr, const cx<Tv>* __restrict__ Vb, size_t vsj,
                                                   size_t vsr, int nvec, const cx<double>* __restrict__ h, int ldh,
                                                   double sign, size_t n, const int* active, const double* post,
                                                   cx<float>* w32) {
  const int r = blockIdx.y;
  if (active && !active[r]) return;
  using Tc = typename std::conditional<(sizeof(Tw) > sizeof(Tv)), Tw, Tv>::type;
  const cx<double>* hr = h + (size_t)r * ldh;
  const Tc f = post ? (Tc)post[r] : (Tc)1;
  for (size_t i = (size_t)blockIdx.x * BT + threadIdx.x; i < n; i += (size_t)gridDim.x * BT) {
    cx<Tc> acc = cvt<Tc>(w[(size_t)r * wsr + i]);
    for (int j = 0; j < nvec; ++j)
      acc = acc + cvt<Tc>(sign * hr[j]) * cvt<Tc>(Vb[(size_t)j * vsj + (size_t)r * vsr + i]);
    const cx<Tw> res = cvt<Tw>(f * acc);
    w[(size_t)r * wsr + i] = res;
    if (w32) w32[(size_t)r * wsr + i] = cvt<float>(res);
  }
}

// Second step of classical Gram-Schmidt done twice with the subtraction of
// the previous step's second projection deferred into it.  Slot k holds the
// pending vector u (the previous new vector, projected once); with the
// previous second-projection coefficients c and normalisation sigma it
// becomes v_k = sigma (u - sum_{j<k} c_j V_j), the vector a separate pass
// would have written, and is stored back (correct = false: u is v_k
// already).  In the same pass over the data: w <- w - sum_{j<=k} h_j V_j
// with the corrected v_k, its FP32 copy in w32 if given, and the partial
// sums of V_j^H w (j <= k) and |w|^2 (entry k + 1) as mdot_partial_kernel
// writes them.
// The FP32 copy is scaled by wsc[r] (an estimate of 1 / |w''|) so that the
// preconditioner, which receives it, sees a vector of about unit norm.
template <int MAXV>
__global__ __launch_bounds__(BT) void gs_defer_kernel(cx<double>* part, cx<double>* Vb, size_t vsj, size_t vsr, int k,
                                                      int correct, const cx<double>* __restrict__ c, int ldc,
                                                      const double* __restrict__ sigma, cx<double>* w, size_t wsr,
                                                      const cx<double>* __restrict__ h, int ldh, size_t n,
                                                      size_t chunk, int nchunk, const int* active, cx<float>* w32,
                                                      const double* __restrict__ wsc) {
  __shared__ cx<double> red[MAXV + 1][BT / 64];
  const int cb = blockIdx.x;
  const int r = blockIdx.y;
  if (active && !active[r]) return;
  const int nvec = k + 1;
  const size_t beg = (size_t)cb * chunk;
  const size_t end = min(n, beg + chunk);
  cx<double>* wr = w + (size_t)r * wsr;
  cx<double>* uk = Vb + (size_t)k * vsj + (size_t)r * vsr;
  const cx<double>* hr = h + (size_t)r * ldh;
  const cx<double>* cr = c + (size_t)r * ldc;
  const double sg = sigma[r];
  const double ws = w32 ? wsc[r] : 1.0;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  cx<double> acc[MAXV];
  double nacc = 0.0;
#pragma unroll
  for (int j = 0; j < MAXV; ++j) acc[j] = mk(0.0, 0.0);
  for (size_t i = beg + threadIdx.x; i < end; i += BT) {
    cx<double> v[MAXV];
#pragma unroll
    for (int j = 0; j < MAXV; ++j)
      if (j < k) v[j] = Vb[(size_t)j * vsj + (size_t)r * vsr + i];
    cx<double> u = uk[i];
    if (correct) {
#pragma unroll
      for (int j = 0; j < MAXV; ++j)
        if (j < k) u = u - cr[j] * v[j];
      u = sg * u;
      uk[i] = u;
    }
    cx<double> x = wr[i];
#pragma unroll
    for (int j = 0; j < MAXV; ++j)
      if (j < nvec) {
        if (j == k) v[j] = u;
        x = x - hr[j] * v[j];
      }
    wr[i] = x;
    if (w32) w32[(size_t)r * wsr + i] = cvt<float>(ws * x);
#pragma unroll
    for (int j = 0; j < MAXV; ++j)
      if (j < nvec) acc[j] = acc[j] + cmulc(v[j], x);
    nacc += x.r * x.r + x.i * x.i;
  }
#pragma unroll
  for (int j = 0; j < MAXV; ++j) {
    if (j < nvec) {
      const double re = wave_sum_d(acc[j].r), im = wave_sum_d(acc[j].i);
      if (lane == 0) red[j][wid] = mk(re, im);
    }
  }
  nacc = wave_sum_d(nacc);
  if (lane == 0) red[nvec][wid] = mk(nacc, 0.0);
  __syncthreads();
  for (int j = threadIdx.x; j <= nvec; j += BT) {
    cx<double> sum = mk(0.0, 0.0);
    for (int q = 0; q < BT / 64; ++q) sum = sum + red[j][q];
    part[((size_t)r * (nvec + 1) + j) * nchunk + cb] = sum;
  }
}

// |w''|^2 = |w'|^2 - sum_j |h2_j|^2 (w'' = w' - V h2 with V orthonormal),
// and the factor that normalises w''; zero for a vanishing or non-finite
// norm (the Arnoldi step then stops that rhs)
__global__ void gs_norm_kernel(cx<double>* n2, double* inv, const cx<double>* h2, int ldh, int nvec, int nrhs,
                               const int* active) {
  const int r = threadIdx.x;
  if (r >= nrhs) return;
  if (active && !active[r]) return;
  const cx<double>* hr = h2 + (size_t)r * ldh;
  double t = hr[nvec].r;
  for (int j = 0; j < nvec; ++j) t -= hr[j].r * hr[j].r + hr[j].i * hr[j].i;
  t = fmax(t, 0.0);
  n2[r] = mk(t, 0.0);
  const double nr = sqrt(t);
  inv[r] = (nr > 0.0 && isfinite(nr)) ? 1.0 / nr : 0.0;
}

template <typename Ty, typename Tx>
__global__ __launch_bounds__(BT) void scale_kernel(cx<Ty>* y, size_t ystr, const cx<Tx>* x, size_t xstr,
                                                   const double* s, size_t n, const int* active, cx<float>* y32) {
  const int r = blockIdx.y;
  if (active && !active[r]) return;
  const double f = s[r];
  for (size_t i = (size_t)blockIdx.x * BT + threadIdx.x; i < n; i += (size_t)gridDim.x * BT) {
    cx<double> v = cvt<double>(x[(size_t)r * xstr + i]);
    const cx<Ty> res = cvt<Ty>(f * v);
    y[(size_t)r * ystr + i] = res;
    if (y32) y32[(size_t)r * ystr + i] = cvt<float>(res);
  }
}

template <typename T>
__global__ __launch_bounds__(BT) void sub_kernel(cx<T>* y, size_t ystr, const cx<T>* a, size_t astr, const cx<T>* b,
                                                 size_t bstr, size_t n) {
  const int r = blockIdx.y;
  for (size_t i = (size_t)blockIdx.x * BT + threadIdx.x; i < n; i += (size_t)gridDim.x * BT)
    y[(size_t)r * ystr + i] = a[(size_t)r * astr + i] - b[(size_t)r * bstr + i];
}

template <typename Ty, typename Tx>
__global__ __launch_bounds__(BT) void copy_kernel(cx<Ty>* y, size_t ystr, const cx<Tx>* x, size_t xstr, size_t n) {
  const int r = blockIdx.y;
  for (size_t i = (size_t)blockIdx.x * BT + threadIdx.x; i < n; i += (size_t)gridDim.x * BT)
    y[(size_t)r * ystr + i] = cvt<Ty>(x[(size_t)r * xstr + i]);
}

inline unsigned grid_for(size_t n) {
  size_t b = (n + BT - 1) / BT;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (unsigned)b;
}

// ----------------------------------------------------- Arnoldi / Givens
// the number of active rhs into *any (one 64-lane wave, nrhs <= 64)
__device__ inline void publish_any(const ArnoldiState& s, bool act) {
  const unsigned long long b = __ballot(act);
  if (threadIdx.x == 0) *s.any = __popcll(b);
}

__global__ void arnoldi_start_kernel(ArnoldiState s, const cx<double>* norm2, int ldn, int nrhs) {
  const int r = threadIdx.x;
  bool act = false;
  if (r < nrhs) {
    const int m = s.m;
    const double beta = sqrt(fmax(norm2[(size_t)r * ldn].r, 0.0));
    for (int j = 0; j <= m; ++j) s.g[(size_t)r * (m + 1) + j] = mk(0.0, 0.0);
    s.g[(size_t)r * (m + 1)] = mk(beta, 0.0);
    const double tol = s.abstol[r];
    act = tol < 0.0 ? beta > 0.0 : beta > tol;
    s.active[r] = act ? 1 : 0;
    s.inv_h[r] = act ? 1.0 / beta : 0.0;
    s.kdone[r] = 0;
    s.est[r] = beta;
  }
  publish_any(s, act);
}

__global__ void arnoldi_column_kernel(ArnoldiState s, int k, const cx<double>* h1, const cx<double>* h2, int ldh,
                                      const cx<double>* norm2, int ldn, int nrhs) {
  const int r = threadIdx.x;
  bool act = false;
  if (r < nrhs && !s.active[r]) s.inv_h[r] = 0.0;
  if (r < nrhs && s.active[r]) {
    const int m = s.m;
    cx<double>* H = s.H + (size_t)r * (m + 1) * m + (size_t)k * (m + 1);
    cx<double>* cs = s.cs + (size_t)r * m;
    cx<double>* sn = s.sn + (size_t)r * m;
    cx<double>* g = s.g + (size_t)r * (m + 1);
    for (int j = 0; j <= k; ++j) {
      cx<double> v = h1[(size_t)r * ldh + j];
      if (h2) v = v + h2[(size_t)r * ldh + j];
      H[j] = v;
    }
    const double hn = sqrt(fmax(norm2[(size_t)r * ldn].r, 0.0));
    H[k + 1] = mk(hn, 0.0);
    for (int j = 0; j < k; ++j) {
      const double c = cs[j].r;
      const cx<double> sj = sn[j];
      const cx<double> t = c * H[j] + sj * H[j + 1];
      H[j + 1] = c * H[j + 1] - conj(sj) * H[j];
      H[j] = t;
    }
    double c;
    cx<double> sv, rr;
    givens(H[k], H[k + 1], c, sv, rr);
    cs[k] = mk(c, 0.0);
    sn[k] = sv;
    H[k] = rr;
    H[k + 1] = mk(0.0, 0.0);
    const cx<double> gk = g[k];
    g[k + 1] = neg(conj(sv) * gk);
    g[k] = c * gk;
    const double est = sqrt(cabs2(g[k + 1]));
    s.est[r] = est;
    s.kdone[r] = k + 1;
    const double tol = s.abstol[r];
    const bool stop = !(hn > 0.0) || (tol >= 0.0 && est <= tol) || k + 1 >= m;
    act = !stop;
    s.active[r] = stop ? 0 : 1;
    s.inv_h[r] = stop ? 0.0 : 1.0 / hn;
  }
  publish_any(s, act);
}

__global__ void arnoldi_solve_kernel(ArnoldiState s, int nrhs) {
  const int r = threadIdx.x;
  if (r >= nrhs) return;
  const int m = s.m;
  const int kd = s.kdone[r];
  const cx<double>* H = s.H + (size_t)r * (m + 1) * m;
  const cx<double>* g = s.g + (size_t)r * (m + 1);
  cx<double>* y = s.y + (size_t)r * m;
  for (int j = kd; j < m; ++j) y[j] = mk(0.0, 0.0);
  for (int i = kd - 1; i >= 0; --i) {
    cx<double> v = g[i];
    for (int j = i + 1; j < kd; ++j) v = v - H[(size_t)j * (m + 1) + i] * y[j];
    const cx<double> d = H[(size_t)i * (m + 1) + i];
    const double dn = cabs2(d);
    y[i] = dn > 0.0 ? (1.0 / dn) * (conj(d) * v) : mk(0.0, 0.0);
  }
}

// abstol[r] = tol * sqrt(|n2[r]|) (tol < 0: -1, i.e. never test)
__global__ void set_abstol_kernel(double* abstol, const cx<double>* n2, double tol, int nrhs) {
  const int r = threadIdx.x;
  if (r >= nrhs) return;
  abstol[r] = tol < 0.0 ? -1.0 : tol * sqrt(fmax(n2[r].r, 0.0));
}

// s[r] = 1 / sqrt(n2[r]); flags a zero or non-finite norm in *status
__global__ void inv_norm_kernel(double* s, const cx<double>* n2, int nrhs, int* status) {
  const int r = threadIdx.x;
  if (r >= nrhs) return;
  const double nr = sqrt(fmax(n2[r].r, 0.0));
  if (!(nr > 0.0) || !isfinite(nr)) {
    atomicExch(status, 1);
    s[r] = 0.0;
  } else {
    s[r] = 1.0 / nr;
  }
}

}  // namespace

void launch_set_abstol(double* abstol, const cx<double>* n2, double tol, int nrhs, hipStream_t st) {
  set_abstol_kernel<<<1, 64, 0, st>>>(abstol, n2, tol, nrhs);
}
void launch_inv_norm(double* s, const cx<double>* n2, int nrhs, int* status, hipStream_t st) {
  inv_norm_kernel<<<1, 64, 0, st>>>(s, n2, nrhs, status);
}

template <typename T>
bool launch_mdot(cx<double>* h, int ldh, cx<double>* part, size_t part_cap, const cx<T>* Vb, size_t vsj, size_t vsr,
                 int nvec, const cx<T>* w, size_t wsr, size_t n, int nrhs, const int* active, hipStream_t st) {
  if (nrhs <= 0 || nvec <= 0) return true;
  if (nvec > MAX_MDOT_VECS || mdot_part_entries(n, nvec, nrhs) > part_cap) return false;
  const int nchunk = blas_nchunks(n, nrhs);
  const size_t chunk = (n + nchunk - 1) / nchunk;
  mdot_partial_kernel<T><<<dim3(nchunk, nrhs), BT, 0, st>>>(part, Vb, vsj, vsr, nvec, w, wsr, n, chunk, nchunk,
                                                            active, h, ldh);
  if (h && nchunk > 1) mdot_final_kernel<<<dim3(nvec, nrhs), 64, 0, st>>>(h, ldh, part, nvec, nchunk, active);
  return true;
}

template <typename Tw, typename Tv>
void launch_maxpy(cx<Tw>* w, size_t wsr, const cx<Tv>* Vb, size_t vsj, size_t vsr, int nvec, const cx<double>* h,
                  int ldh, double sign, size_t n, int nrhs, const int* active, hipStream_t st, const double* post,
                  cx<float>* w32) {
  if (nrhs <= 0 || (nvec <= 0 && !post && !w32)) return;
  maxpy_kernel<Tw, Tv>
      <<<dim3(grid_for(n), nrhs), BT, 0, st>>>(w, wsr, Vb, vsj, vsr, nvec, h, ldh, sign, n, active, post, w32);
}

bool launch_gs_defer(int ldh, cx<double>* part, size_t part_cap, cx<double>* Vb, size_t vsj,
                     size_t vsr, int k, bool correct, const cx<double>* c, const double* sigma, cx<double>* w,
                     size_t wsr, const cx<double>* h, size_t n, int nrhs, const int* active, cx<float>* w32,
                     const double* wsc, hipStream_t st) {
  if (nrhs <= 0) return true;
  const int nvec = k + 1;
  if (nvec > GS_FUSED_MAXV || mdot_part_entries(n, nvec + 1, nrhs) > part_cap) return false;
  const int nchunk = blas_nchunks(n, nrhs);
  const size_t chunk = (n + nchunk - 1) / nchunk;
  dim3 grid(nchunk, nrhs);
  const int cr = correct ? 1 : 0;
  if (nvec <= 4)
    gs_defer_kernel<4><<<grid, BT, 0, st>>>(part, Vb, vsj, vsr, k, cr, c, ldh, sigma, w, wsr, h, ldh, n, chunk, nchunk,
                                            active, w32, wsc);
  else if (nvec <= 8)
    gs_defer_kernel<8><<<grid, BT, 0, st>>>(part, Vb, vsj, vsr, k, cr, c, ldh, sigma, w, wsr, h, ldh, n, chunk, nchunk,
                                            active, w32, wsc);
  else if (nvec <= 16)
    gs_defer_kernel<16><<<grid, BT, 0, st>>>(part, Vb, vsj, vsr, k, cr, c, ldh, sigma, w, wsr, h, ldh, n, chunk,
                                             nchunk, active, w32, wsc);
  else
    gs_defer_kernel<GS_FUSED_MAXV><<<grid, BT, 0, st>>>(part, Vb, vsj, vsr, k, cr, c, ldh, sigma, w, wsr, h, ldh, n,
                                                        chunk, nchunk, active, w32, wsc);
  return true;
}

void launch_gs_norm(cx<double>* n2, double* inv, const cx<double>* h2, int ldh, int nvec, int nrhs, const int* active,
                    hipStream_t st) {
  gs_norm_kernel<<<1, 64, 0, st>>>(n2, inv, h2, ldh, nvec, nrhs, active);
}

template <typename Ty, typename Tx>
void launch_scale(cx<Ty>* y, size_t ystr, const cx<Tx>* x, size_t xstr, const double* s, size_t n, int nrhs,
                  const int* active, hipStream_t st, cx<float>* y32) {
  if (nrhs <= 0) return;
  scale_kernel<Ty, Tx><<<dim3(grid_for(n), nrhs), BT, 0, st>>>(y, ystr, x, xstr, s, n, active, y32);
}

template <typename T>
void launch_sub(cx<T>* y, size_t ystr, const cx<T>* a, size_t astr, const cx<T>* b, size_t bstr, size_t n, int nrhs,
                hipStream_t st) {
  if (nrhs <= 0) return;
  sub_kernel<T><<<dim3(grid_for(n), nrhs), BT, 0, st>>>(y, ystr, a, astr, b, bstr, n);
}

template <typename Ty, typename Tx>
void launch_copy(cx<Ty>* y, size_t ystr, const cx<Tx>* x, size_t xstr, size_t n, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  copy_kernel<Ty, Tx><<<dim3(grid_for(n), nrhs), BT, 0, st>>>(y, ystr, x, xstr, n);
}

void launch_arnoldi_start(ArnoldiState s, const cx<double>* norm2, int ldn, int nrhs, hipStream_t st) {
  arnoldi_start_kernel<<<1, 64, 0, st>>>(s, norm2, ldn, nrhs);
}
void launch_arnoldi_column(ArnoldiState s, int k, const cx<double>* h1, const cx<double>* h2, int ldh,
                           const cx<double>* norm2, int ldn, int nrhs, hipStream_t st) {
  arnoldi_column_kernel<<<1, 64, 0, st>>>(s, k, h1, h2, ldh, norm2, ldn, nrhs);
}
void launch_arnoldi_solve(ArnoldiState s, int nrhs, hipStream_t st) {
  arnoldi_solve_kernel<<<1, 64, 0, st>>>(s, nrhs);
}

template bool launch_mdot<double>(cx<double>*, int, cx<double>*, size_t, const cx<double>*, size_t, size_t, int,
                                  const cx<double>*, size_t, size_t, int, const int*, hipStream_t);
template bool launch_mdot<float>(cx<double>*, int, cx<double>*, size_t, const cx<float>*, size_t, size_t, int,
                                 const cx<float>*, size_t, size_t, int, const int*, hipStream_t);
#define INST2(A, B)                                                                                                   \
  template void launch_maxpy<A, B>(cx<A>*, size_t, const cx<B>*, size_t, size_t, int, const cx<double>*, int, double, \
                                   size_t, int, const int*, hipStream_t, const double*, cx<float>*);                  \
  template void launch_scale<A, B>(cx<A>*, size_t, const cx<B>*, size_t, const double*, size_t, int, const int*,      \
                                   hipStream_t, cx<float>*);                                                          \
  template void launch_copy<A, B>(cx<A>*, size_t, const cx<B>*, size_t, size_t, int, hipStream_t);
INST2(double, double)
INST2(float, float)
INST2(double, float)
INST2(float, double)
#undef INST2
template void launch_sub<double>(cx<double>*, size_t, const cx<double>*, size_t, const cx<double>*, size_t, size_t, int,
                                 hipStream_t);
template void launch_sub<float>(cx<float>*, size_t, const cx<float>*, size_t, const cx<float>*, size_t, size_t, int,
                                hipStream_t);

}  // namespace ddamg
