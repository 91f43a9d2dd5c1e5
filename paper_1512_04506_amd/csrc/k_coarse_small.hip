// The whole coarse solve of Alg. 2 for one rhs in one workgroup, on coarse
// lattices of a few dozen sites: the even/odd Schur complement S = D_oo -
// D_oe D_ee^{-1} D_eo, restarted GMRES on S with classical Gram-Schmidt
// twice, the Givens rotations and the convergence test of the many-launch
// solve, the back substitution, then x_e = D_ee^{-1} (y_e - D_eo x_o).
//
// One GMRES iteration is a few microseconds of work; as separate launches it
// is a chain of launch latencies.  Here one compute unit reads the operator
// once per iteration (1.2 MB on 2^4 sites at N_tv 16 in FP32), at most 64
// bytes a cycle from L2, 9 us: what bounds it is that rate and the loads in
// flight.  Every lane therefore takes 16 bytes
// of a column (two rows, one in FP64) with eight columns in flight, the
// columns of all slots are split over as many lanes as the workgroup has,
// and the vectors stay on chip: the operator's input in LDS, where each
// product leaves its result for the next one, the new vector in registers.
// 2^4 sites, N_tv 16, FP32, one rhs, per solve: 98 us (135 with 512 lanes of
// 8-byte loads and the vectors in memory; some 150 as separate launches).
// Every loop is bounded by maxit or by the restart length m <= SG_M.
#include <algorithm>
#include <stdexcept>

#include "krylov_device.h"
#include "mfma_device.h"

namespace ddamg {

namespace {

using namespace dev;

constexpr int SG_M = COARSE_SMALL_MAX_RESTART;
constexpr int SG_EPT = (COARSE_SMALL_MAX_VECTOR + AT - 1) / AT;  // elements of a vector per lane
constexpr int SG_COLS = 8;                                      // columns in flight
// rows of a column per lane: 16 bytes of an FP32 or FP64 operator
template <typename T>
constexpr int sg_rows() { return (int)(16 / sizeof(cx<T>)); }

template <typename T>
struct SmallShared {
  cx<T> x[COARSE_SMALL_MAX_VECTOR];  // a vector of the whole lattice, site-major
  cx<T> part[AT * sg_rows<T>()];     // [column group][element]
  cx<double> H[(SG_M + 1) * SG_M], sn[SG_M], g[SG_M + 1], h1[SG_M + AJ], h2[SG_M + AJ];
  double cs[SG_M], red[8][AW];
  int nbr[COARSE_SMALL_MAX_SITES * 9];
  int stop;
};

// acc[q] += sum over cnt columns of rows q of D (row offset included), inputs x
template <typename T, typename X>
__device__ inline void sg_columns(cx<T> acc[sg_rows<T>()], const X* D, int nc, int cnt, const cx<T>* x) {
  constexpr int RP = sg_rows<T>();
  for (int k0 = 0; k0 < cnt; k0 += SG_COLS) {
    Run<X, RP> d[SG_COLS];
#pragma unroll
    for (int u = 0; u < SG_COLS; ++u) d[u] = load_run<X, RP>(D + (size_t)min(k0 + u, cnt - 1) * nc);
#pragma unroll
    for (int u = 0; u < SG_COLS; ++u) {
      if (k0 + u >= cnt) break;
      const cx<T> xk = x[k0 + u];
#pragma unroll
      for (int q = 0; q < RP; ++q) acc[q] = cfma(ldc<T>(d[u].v, (size_t)q), xk, acc[q]);
    }
  }
}

// The products of a parity with the columns split over G groups of lanes:
// f(acc, ls, row, q, G) gives group q's part of rows row .. row + RP - 1 of
// site ls; done(e, i, sum) receives element e = t + AT i.  Two barriers; the
// inputs may be overwritten by done.
template <typename T, typename F, typename D>
__device__ inline void sg_product(SmallShared<T>& s, int nsite, int nc, int ncol, F&& f, D&& done) {
  constexpr int RP = sg_rows<T>();
  const int t = threadIdx.x, nelem = nsite * nc, np = nelem / RP;  // np <= AT, nc is even
  const int G = min(AT / np, ncol);
  const int q = t / np, p = t - q * np;
  if (q < G) {
    const int ls = RP * p / nc;
    cx<T> acc[RP];
#pragma unroll
    for (int v = 0; v < RP; ++v) acc[v] = mk((T)0, (T)0);
    f(acc, ls, RP * p - ls * nc, q, G);
#pragma unroll
    for (int v = 0; v < RP; ++v) s.part[q * nelem + RP * p + v] = acc[v];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i) {
    const int e = t + AT * i;
    if (e < nelem) {
      cx<T> sum = mk((T)0, (T)0);
      for (int k = 0; k < G; ++k) sum = sum + s.part[k * nelem + e];
      done(e, i, sum);
    }
  }
  __syncthreads();
}

// done(e, i, [D_self x +] cn sum_{slot > 0} D_slot x(nbr)) on the sites
// out_first .. out_first + nsite - 1, x = s.x: group q takes its share of the
// columns of the eight neighbour slots and of the self slot's
template <typename T, typename S, bool SELF, typename D>
__device__ inline void sg_stencil(SmallShared<T>& s, int out_first, int nsite, T cn, const CoarseView<S>& cv, int nc,
                                  D&& done) {
  constexpr int RP = sg_rows<T>();
  const size_t nn = (size_t)nc * nc;
  sg_product<T>(
      s, nsite, nc, 8 * nc,
      [&](cx<T>* acc, int ls, int row, int q, int G) {
        const int ci = out_first + ls;
        const stc_t<S>* Ds = cv.D + (size_t)ci * 9 * nn + row;
        auto run = [&](int slot, int k0, int k1, T coef) {
          if constexpr (is_half<S>()) coef *= (T)cv.Dsc[ci * 9 + slot];
          cx<T> sum[RP];
#pragma unroll
          for (int v = 0; v < RP; ++v) sum[v] = mk((T)0, (T)0);
          const int nb = slot == 0 ? ci : s.nbr[ci * 9 + slot];
          sg_columns<T, stc_t<S>>(sum, Ds + (size_t)slot * nn + (size_t)k0 * nc, nc, k1 - k0,
                                  s.x + (size_t)nb * nc + k0);
#pragma unroll
          for (int v = 0; v < RP; ++v) acc[v] = acc[v] + coef * sum[v];
        };
        const int c1 = (q + 1) * 8 * nc / G;
        for (int c = q * 8 * nc / G; c < c1;) {
          const int sl = c / nc, k0 = c - sl * nc, k1 = min(nc, k0 + c1 - c);
          run(sl + 1, k0, k1, cn);
          c += k1 - k0;
        }
        if constexpr (SELF) {
          const int k0 = q * nc / G, k1 = (q + 1) * nc / G;
          if (k1 > k0) run(0, k0, k1, (T)1);
        }
      },
      done);
}

// x_e = D_ee^{-1} x_e in s.x, or done(e, i, that)
template <typename T, typename D>
__device__ inline void sg_even_inverse(SmallShared<T>& s, const cx<T>* M, int neven, int nc, D&& done) {
  sg_product<T>(
      s, neven, nc, nc,
      [&](cx<T>* acc, int ls, int row, int q, int G) {
        const int k0 = q * nc / G, k1 = (q + 1) * nc / G;
        if (k1 > k0)
          sg_columns<T, cx<T>>(acc, M + ((size_t)ls * nc + k0) * nc + row, nc, k1 - k0, s.x + ls * nc + k0);
      },
      done);
}

// h[j] = V_j^H w, j < nv, summed in FP64
template <typename T>
__device__ inline void sg_dots(cx<double>* h, const cx<T>* V, size_t vsj, int nv, const cx<T> w[SG_EPT], int n,
                               double (*red)[AW]) {
  for (int j0 = 0; j0 < nv; j0 += AJ) {
    cx<double> acc[AJ];
#pragma unroll
    for (int q = 0; q < AJ; ++q) acc[q] = mk(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < SG_EPT; ++i) {
      if ((int)threadIdx.x >= n - AT * i) continue;
      const cx<double> wv = cvt<double>(w[i]);
#pragma unroll
      for (int q = 0; q < AJ; ++q)
        if (j0 + q < nv) acc[q] = acc[q] + cmulc(cvt<double>(V[(size_t)(j0 + q) * vsj + AT * i + threadIdx.x]), wv);
    }
    block_sum(h + j0, acc, min(AJ, nv - j0), red);
  }
}
// |w|^2 into h[0].r (elements beyond n are zero)
template <typename T>
__device__ inline void sg_norm2(cx<double>* h, const cx<T> w[SG_EPT], double (*red)[AW]) {
  cx<double> acc[AJ];
#pragma unroll
  for (int q = 0; q < AJ; ++q) acc[q] = mk(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i) acc[0].r += cabs2(cvt<double>(w[i]));
  block_sum(h, acc, 1, red);
}
// w -= sum_j h_j V_j
template <typename T>
__device__ inline void sg_update(cx<T> w[SG_EPT], const cx<T>* V, size_t vsj, int nv, const cx<double>* h, int n) {
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i) {
    if ((int)threadIdx.x >= n - AT * i) continue;
#pragma unroll 4
    for (int j = 0; j < nv; ++j) w[i] = w[i] + cvt<T>(-1.0 * h[j]) * V[(size_t)j * vsj + AT * i + threadIdx.x];
  }
}

template <typename T, typename S>
__global__ __launch_bounds__(AT) void coarse_gmres_small_kernel(cx<T>* xc, const cx<T>* yc, size_t cstr,
                                                                CoarseView<S> cv, const cx<T>* Dinv, int nc, int neven,
                                                                int nodd, cx<T>* bo_, cx<T>* V_, size_t vsj, int m,
                                                                int maxit, double tol, int* its_stat) {
  __shared__ SmallShared<T> s;
  const int r = blockIdx.x, t = threadIdx.x;
  const int ne = neven * nc, no = nodd * nc;
  const cx<T>* y = yc + (size_t)r * cstr;
  cx<T>* x = xc + (size_t)r * cstr;
  cx<T>* bo = bo_ + (size_t)r * no;
  cx<T>* V = V_ + (size_t)r * no;  // V_j = V + j vsj
  cx<T> w[SG_EPT], xo[SG_EPT];     // elements t + AT i of the odd sites
  // to LDS for the operator (a barrier of the caller's follows)
  auto put_odd = [&](const cx<T>* a) {
#pragma unroll
    for (int i = 0; i < SG_EPT; ++i)
      if (t < no - AT * i) s.x[ne + AT * i + t] = a[i];
  };
  auto to_even = [&](int e, int, cx<T> v) { s.x[e] = v; };
  // w = S (the odd part of s.x); the even part is lost
  auto schur = [&] {
    sg_stencil<T, S, false>(s, 0, neven, (T)1, cv, nc, to_even);
    sg_even_inverse<T>(s, Dinv, neven, nc, to_even);
    sg_stencil<T, S, true>(s, neven, nodd, (T)-1, cv, nc, [&](int, int i, cx<T> v) { w[i] = v; });
  };
  for (int e = t; e < (neven + nodd) * 9; e += AT) s.nbr[e] = cv.nbr[e];
  // |y_c| -> absolute tolerance (tol < 0: never test)
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i) {
    const int e = t + AT * i;
    xo[i] = mk((T)0, (T)0);
    w[i] = e < ne + no ? y[e] : mk((T)0, (T)0);
    if (e < ne) s.x[e] = w[i];
  }
  sg_norm2<T>(s.h1, w, s.red);
  const double abstol = tol < 0.0 ? -1.0 : tol * sqrt(fmax(s.h1[0].r, 0.0));
  __syncthreads();
  // b_o = y_o - D_oe D_ee^{-1} y_e, x_o = 0
  sg_even_inverse<T>(s, Dinv, neven, nc, to_even);
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i) w[i] = mk((T)0, (T)0);
  sg_stencil<T, S, false>(s, neven, nodd, (T)-1, cv, nc, [&](int e, int i, cx<T> v) {
    w[i] = y[ne + e] + v;
    bo[e] = w[i];
  });
  int its = 0;
  bool first = true;
  while (its < maxit) {
    // r = b_o - S x_o into V_0, its norm, the start of a cycle
    if (!first) {
      put_odd(xo);
      __syncthreads();
      schur();
#pragma unroll
      for (int i = 0; i < SG_EPT; ++i)
        if (t < no - AT * i) w[i] = bo[AT * i + t] - w[i];
    }
    first = false;
    sg_norm2<T>(s.h1, w, s.red);
    const double beta = sqrt(fmax(s.h1[0].r, 0.0));
    const bool act = abstol < 0.0 ? beta > 0.0 : beta > abstol;
    if (!act) break;  // uniform: every lane computed beta from the same sum
    if (t <= m) s.g[t] = mk(t == 0 ? beta : 0.0, 0.0);
    double inv = 1.0 / beta;
    int k = 0;
    for (; k < m && its < maxit; ++k) {
      // V_k = w / |w|
#pragma unroll
      for (int i = 0; i < SG_EPT; ++i) {
        w[i] = cvt<T>(inv * cvt<double>(w[i]));
        if (t < no - AT * i) V[(size_t)k * vsj + AT * i + t] = w[i];
      }
      put_odd(w);
      __syncthreads();
      schur();
      // classical Gram-Schmidt twice, then |w|^2
      sg_dots<T>(s.h1, V, vsj, k + 1, w, no, s.red);
      sg_update<T>(w, V, vsj, k + 1, s.h1, no);
      sg_dots<T>(s.h2, V, vsj, k + 1, w, no, s.red);
      sg_update<T>(w, V, vsj, k + 1, s.h2, no);
      if (t <= k) s.H[k * (m + 1) + t] = s.h1[t] + s.h2[t];
      sg_norm2<T>(s.h1 + SG_M, w, s.red);
      const double hn = sqrt(fmax(s.h1[SG_M].r, 0.0));
      if (t == 0) {
        cx<double>* Hk = s.H + k * (m + 1);
        cx<double> a = Hk[0];
        for (int j = 0; j < k; ++j) {
          const double c = s.cs[j];
          const cx<double> sj = s.sn[j], b = Hk[j + 1];
          Hk[j] = c * a + sj * b;
          a = c * b - conj(sj) * a;
        }
        double c;
        cx<double> sv, rr;
        givens(a, mk(hn, 0.0), c, sv, rr);
        s.cs[k] = c;
        s.sn[k] = sv;
        Hk[k] = rr;
        const cx<double> gk = s.g[k], gn = neg(conj(sv) * gk);
        s.g[k + 1] = gn;
        s.g[k] = c * gk;
        s.stop = (!(hn > 0.0) || (abstol >= 0.0 && sqrt(cabs2(gn)) <= abstol) || k + 1 >= m) ? 1 : 0;
      }
      __syncthreads();
      ++its;
      inv = 1.0 / hn;
      if (s.stop) {
        ++k;
        break;
      }
    }
    // y = H^{-1} g (upper triangular, k columns; lane j holds g_j), then x_o += V y
    if (t < 64) {
      cx<double> g = t < k ? s.g[t] : mk(0.0, 0.0);
      for (int i = k - 1; i >= 0; --i) {
        const cx<double> hc = t <= i ? s.H[i * (m + 1) + t] : mk(0.0, 0.0);
        const cx<double> d = mk(__shfl(hc.r, i, 64), __shfl(hc.i, i, 64));
        const cx<double> gi = mk(__shfl(g.r, i, 64), __shfl(g.i, i, 64));
        const double dn = cabs2(d);
        const cx<double> yi = dn > 0.0 ? (1.0 / dn) * (conj(d) * gi) : mk(0.0, 0.0);
        if (t == i) g = yi;
        if (t < i) g = g - hc * yi;
      }
      if (t < k) s.h2[t] = neg(g);
    }
    __syncthreads();
    sg_update<T>(xo, V, vsj, k, s.h2, no);
    __syncthreads();  // H, g and h2 are written again
  }
  // x_e = D_ee^{-1} (y_e - D_eo x_o)
  put_odd(xo);
#pragma unroll
  for (int i = 0; i < SG_EPT; ++i)
    if (t < no - AT * i) x[ne + AT * i + t] = xo[i];
  __syncthreads();
  sg_stencil<T, S, false>(s, 0, neven, (T)-1, cv, nc, [&](int e, int, cx<T> v) { s.x[e] = y[e] + v; });
  sg_even_inverse<T>(s, Dinv, neven, nc, [&](int e, int, cx<T> v) { x[e] = v; });
  if (t == 0) {
    atomicAdd(its_stat, its);
    atomicMax(its_stat + 1, its);
  }
}

}  // namespace

template <typename T, typename S>
void launch_coarse_gmres_small(cx<T>* xc, const cx<T>* yc, size_t cstr, const CoarseView<S>& cv, const cx<T>* Dinv,
                               const Geom& g, cx<T>* bo, cx<T>* V, size_t vsj, int m, int maxit, double tol,
                               int* its_stat, int nrhs, hipStream_t st) {
  if (nrhs <= 0) return;
  const int nodd = g.nblocks - g.neven;
  if (m < 1 || m > SG_M || g.nblocks > COARSE_SMALL_MAX_SITES || g.nblocks * g.nc > COARSE_SMALL_MAX_VECTOR ||
      std::max(g.neven, nodd) * g.nc > AT * sg_rows<T>() || g.neven < 1 || nodd < 1 || g.nc % 2)
    throw std::runtime_error("single-kernel coarse solve: restart length or lattice above its bound");
  coarse_gmres_small_kernel<T, S><<<nrhs, AT, 0, st>>>(xc, yc, cstr, cv, Dinv, g.nc, g.neven, nodd, bo, V, vsj, m,
                                                       maxit, tol, its_stat);
}
#define INST(T, S)                                                                                                     \
  template void launch_coarse_gmres_small<T, S>(cx<T>*, const cx<T>*, size_t, const CoarseView<S>&, const cx<T>*,      \
                                                const Geom&, cx<T>*, cx<T>*, size_t, int, int, double, int*, int,      \
                                                hipStream_t);
INST(double, double)
INST(float, float)
INST(float, __half)
#undef INST

}  // namespace ddamg
