// Setup kernels of Alg. 5: orthonormalisation of the test vectors on every
// aggregate (Gram-Schmidt on the rows of R_i^h) and the storage formats of
// the resulting basis.
//
// The paper uses classical block Gram-Schmidt for fewer global sums and
// better cache reuse.  Here every aggregate (block, chirality h: 6 V_block
// rows, ntv columns) runs CholQR2 in FP64, all aggregates at once: the Gram
// matrix X^H X, its Cholesky factor (positive real diagonal) and X <- X T^{-1};
// doing it twice restores orthogonality to rounding.  The result is the
// unique Q of X = Q T with positive diag(T), i.e. the basis Gram-Schmidt
// produces.
#include <algorithm>
#include <type_traits>

#include "ddamg_internal.h"

namespace ddamg {

namespace {

constexpr int QR_THREADS = 256;
constexpr int MAX_NTV = 32;
constexpr int QR_CS = 8;             // sites per staged chunk of the Gram matrix pass
constexpr int QR_ROWS = QR_CS * 6;   // rows (site, spin-colour) per chunk
constexpr int QR_LD = MAX_NTV + 1;   // padded LDS row
// An aggregate is (internal block ci, chirality h): rows are the 6 V_block
// (spin of chirality h x colour, site) entries, columns the ntv test
// vectors.  The products run on the FP64 matrix cores (16x16x4).  The FP64
// basis is never stored: the test vectors are read three times in their own
// precision and the stored basis is written once,
//   G1 = X^H X, T1 = its Cholesky factor,
//   G2 = Q^H Q with Q = X T1^{-1} formed in registers, T2 = its factor,
//   the stored basis (X T1^{-1}) T2^{-1}, for FP16 with its scales,
// the arithmetic of a stored Q in FP64 step by step.  Storing Q and W in FP64
// and quantising in a pass of its own moved 20 GB on 24^3x48 at N_tv 24
// (FP16, 4.81 ms), now 7 (3.74 ms: 0.62 the first Gram matrix, 1.25 the
// second, 1.66 the store, 0.11 each factor); what bounds it is the FP64 matrix
// cores (0.47, 1.06 and 1.18 ms of products).  8^3x16 at N_tv 16 in FP64: 180
// -> 69 us.
// x rounded once to FP16, in a dozen instructions (the compiler's conversion
// takes forty): to FP32 with the last bit odd if that was inexact, which
// leaves the rounding to FP16 to decide alone
__device__ inline __half half_rn(double x) {
  float f = (float)x;
  const double d = (double)f;
  unsigned u = __float_as_uint(f);
  if (d != x && !(u & 1)) u = fabs(d) < fabs(x) ? u + 1 : u - 1;
  return __float2half_rn(__uint_as_float(u));
}

typedef double qr_v4d __attribute__((ext_vector_type(4)));

// The waves' Gram tiles summed (waves 2, 3 hand theirs to 0, 1, then 1 to 0)
// and the upper triangle of G (n x n) written, row-major
template <int NT>
__device__ inline void gram_out(qr_v4d (&acc)[2 * NT], qr_v4d (*part)[2 * NT][64], int n, cx<double>* G) {
  constexpr int NACC = 2 * NT;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col0 = lane & 15, rsub = lane >> 4;
  if (w >= 2)
#pragma unroll
    for (int t = 0; t < NACC; ++t) part[w - 2][t][lane] = acc[t];
  __syncthreads();
  if (w < 2)
#pragma unroll
    for (int t = 0; t < NACC; ++t) acc[t] += part[w][t][lane];
  __syncthreads();
  if (w == 1)
#pragma unroll
    for (int t = 0; t < NACC; ++t) part[0][t][lane] = acc[t];
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int t = 0; t < NACC; ++t) acc[t] += part[0][t][lane];
    // f64 16x16x4 result v of lane l: row l/16 + 4v (first operand's
    // column), column l%16 (second operand's column)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = rsub + 4 * v, j = col0;
      if constexpr (NT == 1) {
        if (i < n && j < n) G[i * n + j] = mk(acc[0][v], acc[1][v]);
      } else if constexpr (NT == 2) {
        const int ib = 8 + j;  // tile 0: rows 0..15, columns 8..23
        if (i <= ib && ib < n) G[i * n + ib] = mk(acc[0][v], acc[1][v]);
        const int ic = i < 8 ? i : i + 8, jc = j < 8 ? j : j + 8;  // tile 1
        if (ic <= jc && jc < n && !(ic < 8 && jc >= 16)) G[ic * n + jc] = mk(acc[2][v], acc[3][v]);
      } else {
        if (i < n && j < n) G[i * n + j] = mk(acc[0][v], acc[1][v]);
        if (i < n && 16 + j < n) G[i * n + 16 + j] = mk(acc[2][v], acc[3][v]);
        if (16 + i < n && 16 + j < n) G[(16 + i) * n + 16 + j] = mk(acc[4][v], acc[5][v]);
      }
    }
  }
}

// Column layouts of the Gram tiles (upper triangle of G = X^H X, 16x16
// tiles, one lane per column in each operand):
//   NT = 1, ntv <= 16: columns 0..15 x 0..15;
//   NT = 2, ntv <= 24: columns 0..15 x 8..23 and {0..7, 16..23} x {0..7,
//          16..23}: with columns in groups of eight, two tiles hold every
//          pair i <= j (the pairs 0..7 x 16..23 of the second are dropped);
//   NT = 3, ntv <= 32: 0..15 x 0..15, 0..15 x 16..31 and 16..31 x 16..31.
template <typename Tin, int NT>
__global__ __launch_bounds__(QR_THREADS) void qr_gram_kernel(const cx<Tin>* W, Geom g, int part_sites,
                                                             cx<double>* Gout) {
  constexpr int NACC = 2 * NT;  // Re and Im of each tile
  // the staged rows of the Gram matrix pass, later the partial tiles of two
  // waves
  constexpr size_t STAGE_BYTES = sizeof(cx<double>) * QR_ROWS * QR_LD > sizeof(qr_v4d) * 2 * NACC * 64
                                     ? sizeof(cx<double>) * QR_ROWS * QR_LD
                                     : sizeof(qr_v4d) * 2 * NACC * 64;
  __shared__ __attribute__((aligned(32))) char stage_raw[STAGE_BYTES];
  auto Xs = reinterpret_cast<cx<double>(*)[QR_LD]>(stage_raw);
  auto part = reinterpret_cast<qr_v4d(*)[NACC][64]>(stage_raw);
  const int ci = blockIdx.x >> 1;  // internal block: its sites are ci * vblock + [0, vblock)
  const int h = blockIdx.x & 1;
  const int n = g.ntv;
  const size_t V = g.V;
  const int beg = blockIdx.y * part_sites, vb = min(g.vblock, beg + part_sites);  // the sites of this part
  const int l = threadIdx.x, lane = l & 63, w = l >> 6;
  const size_t base = (size_t)ci * g.vblock;
  const int col0 = lane & 15, rsub = lane >> 4;
  // operand columns of this lane: ca (first operand of tile 0), cb (second
  // operand of tile 0), cc (both operands of the last tile)
  const int ca = col0;
  const int cb = NT == 2 ? 8 + col0 : col0;
  const int cc = NT == 2 ? (col0 < 8 ? col0 : col0 + 8) : 16 + col0;
  qr_v4d acc[NACC];
#pragma unroll
  for (int t = 0; t < NACC; ++t) acc[t] = (qr_v4d){0.0, 0.0, 0.0, 0.0};
  // Rows (site, spin-colour) of QR_CS sites at a time are staged in LDS with
  // coalesced loads (QR_CS consecutive sites of one test vector and
  // component); the loads of the next two chunks are in flight, held in the
  // input precision, while the MFMAs consume the current one.  Padded test
  // vectors (a >= ntv) are not loaded.
  constexpr int NQ = QR_ROWS * 32 / 256;
  cx<Tin> xq0[NQ], xq1[NQ];
  auto fetch = [&](cx<Tin>(&xq)[NQ], int s0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = l + 256 * q;
      const int sl = e % QR_CS, rest = e / QR_CS, c = rest % 6, a = rest / 6;
      const int sx = min(s0 + sl, vb - 1);
      xq[q] = a < n ? W[((size_t)a * 12 + 6 * h + c) * V + base + sx] : mk((Tin)0, (Tin)0);
    }
  };
  auto chunk = [&](cx<Tin>(&xq)[NQ], int s0) {
    __syncthreads();  // the previous chunk has been consumed
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = l + 256 * q;
      const int sl = e % QR_CS, rest = e / QR_CS, c = rest % 6, a = rest / 6;
      Xs[sl * 6 + c][a] = s0 + sl < vb ? cvt<double>(xq[q]) : mk(0.0, 0.0);
    }
    if (s0 + 2 * QR_CS < vb) fetch(xq, s0 + 2 * QR_CS);
    __syncthreads();
    // 4-row slices; the two products feeding one accumulator are issued
    // apart so no MFMA waits on the one before it
    for (int t = w; t < QR_ROWS / 4; t += 4) {
      const cx<double> y0 = Xs[4 * t + rsub][ca];
      if constexpr (NT == 1) {
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y0.r, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y0.i, acc[1], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.i, y0.i, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-y0.i, y0.r, acc[1], 0, 0, 0);
      } else if constexpr (NT == 2) {
        const cx<double> yb = Xs[4 * t + rsub][cb];
        const cx<double> yc = Xs[4 * t + rsub][cc];
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, yb.r, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, yb.i, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(yc.r, yc.r, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(yc.r, yc.i, acc[3], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.i, yb.i, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-y0.i, yb.r, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(yc.i, yc.i, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(-yc.i, yc.r, acc[3], 0, 0, 0);
      } else {
        const cx<double> y1 = Xs[4 * t + rsub][cc];
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y0.r, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y0.i, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y1.r, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.r, y1.i, acc[3], 0, 0, 0);
        acc[4] = __builtin_amdgcn_mfma_f64_16x16x4f64(y1.r, y1.r, acc[4], 0, 0, 0);
        acc[5] = __builtin_amdgcn_mfma_f64_16x16x4f64(y1.r, y1.i, acc[5], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.i, y0.i, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-y0.i, y0.r, acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0.i, y1.i, acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(-y0.i, y1.r, acc[3], 0, 0, 0);
        acc[4] = __builtin_amdgcn_mfma_f64_16x16x4f64(y1.i, y1.i, acc[4], 0, 0, 0);
        acc[5] = __builtin_amdgcn_mfma_f64_16x16x4f64(-y1.i, y1.r, acc[5], 0, 0, 0);
      }
    }
  };
  fetch(xq0, beg);
  if (beg + QR_CS < vb) fetch(xq1, beg + QR_CS);
  for (int s0 = beg; s0 < vb; s0 += 2 * QR_CS) {
    chunk(xq0, s0);
    if (s0 + QR_CS < vb) chunk(xq1, s0 + QR_CS);
  }
  __syncthreads();  // the staging buffer is reused for the partial tiles
  gram_out<NT>(acc, part, n, Gout + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * n * n);
}

// Cholesky G = T^H T (T upper, real positive diagonal) and T^{-1}, one
// workgroup of L lanes per aggregate, every entry of the W x W matrix (W >=
// ntv) in the register of one lane: a step hands one row to the others
// through LDS.  G is the sum of nparts upper triangles (pstride
// apart).  T^{-1} goes to Tout (both n x n, row-major), which may be the
// first part of G; a pivot that is not positive sets *status and leaves
// zeros.  Bound: the chain of n steps and reciprocal square roots.  N_tv 24,
// 5184 aggregates 106 us (109 with 64 lanes on a matrix in LDS), N_tv 16, 64
// aggregates 17 (20).
template <int W, int L>
__global__ __launch_bounds__(L) void qr_chol_kernel(const cx<double>* G, size_t pstride, int nparts, cx<double>* Tout,
                                                    Geom g, int* status) {
  __shared__ cx<double> row[2][W];
  __shared__ cx<double> Ts[W][W + 1];
  __shared__ double dinv[W];
  constexpr int NQ = W * W / L, RS = L / W;  // rows RS apart per lane
  const int n = g.ntv, t = threadIdx.x, j = t % W, i0 = t / W;
  const cx<double>* Gg = G + (size_t)blockIdx.x * n * n;
  cx<double>* Tg = Tout + (size_t)blockIdx.x * n * n;
  cx<double> a[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = i0 + RS * q;
    a[q] = mk(0.0, 0.0);
    if (i <= j && j < n)
      for (int p = 0; p < nparts; ++p) a[q] = a[q] + Gg[(size_t)p * pstride + i * n + j];
  }
  // right-looking: step k scales row k by the pivot and updates the rows below
  bool ok = true;
  for (int k = 0; k < n; ++k) {
    cx<double>* rk = row[k & 1];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (i0 + RS * q == k) rk[j] = a[q];
    __syncthreads();
    const double dk = rk[k].r;  // every lane reads the same pivot
    if (!(dk > 0.0)) {
      ok = false;
      break;
    }
    const double inv = rsqrt(dk);
    if (t == 0) dinv[k] = inv;
    const cx<double> tj = inv * rk[j];  // of the diagonal only 1 / d is used
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (RS * q + RS - 1 < k) continue;  // rows that are done
      const int i = i0 + RS * q;
      if (i == k) a[q] = tj;
      if (i > k && i <= j) a[q] = a[q] - cmulc(inv * rk[i], tj);
    }
  }
  if (!ok) {
    if (t == 0) atomicExch(status, 1);
    for (int e = t; e < n * n; e += L) Tg[e] = mk(0.0, 0.0);
    return;
  }
  // T^{-1}: T's rows in LDS, the unit matrix reduced from the last row up
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = i0 + RS * q;
    Ts[i][j] = a[q];
    a[q] = mk(i == j ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  for (int k = n - 1; k >= 0; --k) {
    cx<double>* rk = row[k & 1];
    const double inv = dinv[k];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (i0 + RS * q == k) rk[j] = a[q] = inv * a[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (RS * q >= k) continue;
      const int i = i0 + RS * q;
      if (i < k && j >= k) a[q] = a[q] - Ts[i][k] * rk[j];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int i = i0 + RS * q;
    if (i < n && j < n) Tg[i * n + j] = a[q];
  }
}

// T^{-1} as the matrix cores take it, one 64-entry block per step of four
// rows and tile of 16 columns (lane l: row l / 16, column l % 16).  T^{-1} is
// upper triangular: the columns 0 .. 15 have only the steps below 16.
template <int NQ>
struct TBlocks {
  static constexpr int NT = NQ > 4 ? 2 : 1;           // column tiles
  static constexpr int N = NQ > 4 ? 4 + NQ : NQ;      // blocks
  __device__ static constexpr int at(int q, int tj) { return tj ? 4 + q : q; }
  // does step q of tile tj exist
  __device__ static constexpr bool has(int q, int tj) { return tj || q < 4; }
};
template <int NQ>
__device__ inline void load_tinv(cx<double> (*B)[64], const cx<double>* T, int n) {
  for (int e = threadIdx.x; e < TBlocks<NQ>::N * 64; e += blockDim.x) {
    const int b = e >> 6, l = e & 63, tj = b >= 4 ? 1 : 0;
    const int i = 4 * (b - 4 * tj) + (l >> 4), j = 16 * tj + (l & 15);
    B[b][l] = i < n && j < n ? T[i * n + j] : mk(0.0, 0.0);
  }
}

// A barrier for data exchanged through LDS: global loads and stores stay in
// flight across it (__syncthreads waits for them)
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The rows of X for one tile: site s0 + lane % 16, component comp, vectors 4 q + lane / 16
template <typename Tin, int NQ>
__device__ inline void load_x(cx<Tin> x[NQ], const cx<Tin>* X, int comp, size_t base, int s0, int vb, int n,
                              size_t V) {
  const int lane = threadIdx.x & 63, k4 = lane >> 4, sa = min(s0 + (lane & 15), vb - 1);
  // n > 4 (NQ - 1): only the last step can run past the vectors, it reads the first step's again
  const cx<Tin>* p = X + ((size_t)min(k4, n - 1) * 12 + comp) * V + base + sa;
#pragma unroll
  for (int q = 0; q < NQ; ++q) x[q] = p[q < NQ - 1 || 4 * q + k4 < n ? (size_t)(48 * q) * V : 0];
}

// G = Q^H Q with Q = X T^{-1} of one aggregate (and part of its sites).  A
// wave takes tiles of 16 sites of one component: the products with T^{-1}
// leave site lane / 16 + 4 v, vector lane % 16 in register v, which is the
// operand of the Gram products for the sites 4 v .. 4 v + 3 as it stands.
// The column tiles of the Gram matrix are those of qr_gram_kernel (NT == 2:
// the shifted ones by moves within rows of 16 lanes).
__device__ inline double ror8(double v) {  // lane ^ 8 within rows of 16
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x128, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x128, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename Tin, int NQ>
__global__ __launch_bounds__(QR_THREADS, 2) void qr_gram2_kernel(const cx<Tin>* X, Geom g, int part_sites,
                                                                 const cx<double>* Tinv, cx<double>* Gout) {
  using TB = TBlocks<NQ>;
  constexpr int NT = NQ <= 4 ? 1 : NQ <= 6 ? 2 : 3, NACC = 2 * NT;
  constexpr size_t T_BYTES = sizeof(cx<double>) * TB::N * 64, P_BYTES = sizeof(qr_v4d) * 2 * NACC * 64;
  __shared__ __attribute__((aligned(32))) char raw[T_BYTES > P_BYTES ? T_BYTES : P_BYTES];
  auto Tb = reinterpret_cast<cx<double>(*)[64]>(raw);
  auto part = reinterpret_cast<qr_v4d(*)[NACC][64]>(raw);
  const int ci = blockIdx.x >> 1, h = blockIdx.x & 1, n = g.ntv;
  const size_t V = g.V, base = (size_t)ci * g.vblock;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, k4 = lane >> 4;
  const bool lo8 = (lane & 8) == 0;
  const int beg = blockIdx.y * part_sites, end = min(g.vblock, beg + part_sites);
  const int ntile = 6 * ((end - beg + 15) / 16);  // tile: component tile % 6, sites beg + 16 (tile / 6)
  cx<Tin> xr[NQ];
  if (w < ntile) load_x<Tin, NQ>(xr, X, 6 * h + w % 6, base, beg + 16 * (w / 6), end, n, V);
  load_tinv<NQ>(Tb, Tinv + (size_t)blockIdx.x * n * n, n);
  qr_v4d acc[NACC];
#pragma unroll
  for (int t = 0; t < NACC; ++t) acc[t] = (qr_v4d){0.0, 0.0, 0.0, 0.0};
  __syncthreads();
  for (int tile = w; tile < ntile; tile += QR_THREADS / 64) {
    const int s0 = beg + 16 * (tile / 6), nt = tile + QR_THREADS / 64;
    double xa[NQ], xi[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const bool in = 4 * q + k4 < n;  // padded test vectors add nothing
      xa[q] = in ? (double)xr[q].r : 0.0;
      xi[q] = in ? (double)xr[q].i : 0.0;
    }
    if (nt < ntile) load_x<Tin, NQ>(xr, X, 6 * h + nt % 6, base, beg + 16 * (nt / 6), end, n, V);
    qr_v4d yr[TB::NT], yi[TB::NT];
#pragma unroll
    for (int tj = 0; tj < TB::NT; ++tj) {
      qr_v4d RR, II, RI, IR;
#pragma unroll
      for (int v = 0; v < 4; ++v) RR[v] = II[v] = RI[v] = IR[v] = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (!TB::has(q, tj)) continue;
        const cx<double> b = Tb[TB::at(q, tj)][lane];
        RR = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[q], b.r, RR, 0, 0, 0);
        II = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[q], b.i, II, 0, 0, 0);
        RI = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[q], b.i, RI, 0, 0, 0);
        IR = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[q], b.r, IR, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool in = s0 + k4 + 4 * v < end;
        yr[tj][v] = in ? RR[v] - II[v] : 0.0;
        yi[tj][v] = in ? RI[v] + IR[v] : 0.0;
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double ar = yr[0][v], ai = yi[0][v];
      if constexpr (NT == 1) {
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, ar, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, ai, acc[1], 0, 0, 0);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, ai, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, ar, acc[1], 0, 0, 0);
      } else {
        const double cr = yr[TB::NT - 1][v], cim = yi[TB::NT - 1][v];
        // second operand of tile 0 / both of the last tile
        double br = ar, bi = ai, dr = cr, di = cim;
        if constexpr (NT == 2) {
          const double a8 = ror8(ar), i8 = ror8(ai), c8 = ror8(cr), ci8 = ror8(cim);
          br = lo8 ? a8 : c8;  // columns 8 .. 23
          bi = lo8 ? i8 : ci8;
          dr = lo8 ? ar : c8;  // columns 0 .. 7, 16 .. 23
          di = lo8 ? ai : ci8;
        }
        constexpr int L = NACC - 2;
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, acc[1], 0, 0, 0);
        acc[L] = __builtin_amdgcn_mfma_f64_16x16x4f64(dr, dr, acc[L], 0, 0, 0);
        acc[L + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(dr, di, acc[L + 1], 0, 0, 0);
        if constexpr (NT == 3) {
          acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, cr, acc[2], 0, 0, 0);
          acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, cim, acc[3], 0, 0, 0);
        }
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, br, acc[1], 0, 0, 0);
        acc[L] = __builtin_amdgcn_mfma_f64_16x16x4f64(di, di, acc[L], 0, 0, 0);
        acc[L + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(-di, dr, acc[L + 1], 0, 0, 0);
        if constexpr (NT == 3) {
          acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, cim, acc[2], 0, 0, 0);
          acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, cr, acc[3], 0, 0, 0);
        }
      }
    }
  }
  __syncthreads();  // T^{-1} gives way to the partial tiles
  gram_out<NT>(acc, part, n, Gout + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * n * n);
}

// The stored basis (X T1^{-1}) T2^{-1} of one block (blockIdx.x), both
// chiralities, 16 sites at a time: wave w takes the components 3 w .. 3 w + 2.
// The products are formed transposed (T^T X^T), so that register v of the
// first one, vector lane / 16 + 4 v at site lane % 16, is the operand of step
// v of the second, and the stores are runs of 16 sites.  FP16: the scale of a
// (vector, site), its largest component, is exchanged between the waves, and
// Wt receives scale * half, as quantize_basis_kernel writes them.  Bound: the
// FP64 matrix cores (80 products of 64 cycles per wave, component and 16
// sites at N_tv 24).  Barriers that leave loads and stores in flight, one base
// address per lane and the short FP16 rounding took it from 1.99 to 1.66 ms.
template <typename Tin, typename S, int NQ>
__global__ __launch_bounds__(QR_THREADS, 2) void qr_store_kernel(stc_t<S>* Wq, float* Wsc, cx<float>* Wt,
                                                                 const cx<Tin>* X, Geom g, const cx<double>* T1,
                                                                 const cx<double>* T2) {
  using TB = TBlocks<NQ>;
  __shared__ cx<double> Tb[2][2][TB::N][64];  // [chirality][factor]
  __shared__ float mx[is_half<S>() ? 4 : 1][TB::NT * 4][64];
  const int ci = blockIdx.x, n = g.ntv, vb = g.vblock;
  const size_t V = g.V, base = (size_t)ci * vb;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, k4 = lane >> 4, h = w >> 1;
  for (int e = 0; e < 2; ++e) {
    const size_t agg = (size_t)(2 * ci + e) * n * n;
    load_tinv<NQ>(Tb[e][0], T1 + agg, n);
    load_tinv<NQ>(Tb[e][1], T2 + agg, n);
  }
  const int ngroup = (vb + 15) / 16, step = 16 * gridDim.y;
  int s0 = 16 * blockIdx.y;
  cx<Tin> xr[NQ];  // the next component's rows
  if (blockIdx.y < ngroup) load_x<Tin, NQ>(xr, X, 3 * w, base, s0, vb, n, V);
  __syncthreads();
  // z = T^T x for factor f of this wave's chirality, steps and tiles in registers
  auto product = [&](double zr[TB::NT][4], double zi[TB::NT][4], int f, const double xr_[NQ], const double xi_[NQ]) {
#pragma unroll
    for (int tj = 0; tj < TB::NT; ++tj) {
      qr_v4d RR, II, RI, IR;
#pragma unroll
      for (int v = 0; v < 4; ++v) RR[v] = II[v] = RI[v] = IR[v] = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (!TB::has(q, tj)) continue;
        const cx<double> a = Tb[h][f][TB::at(q, tj)][lane];
        RR = __builtin_amdgcn_mfma_f64_16x16x4f64(a.r, xr_[q], RR, 0, 0, 0);
        II = __builtin_amdgcn_mfma_f64_16x16x4f64(a.i, xi_[q], II, 0, 0, 0);
        RI = __builtin_amdgcn_mfma_f64_16x16x4f64(a.r, xi_[q], RI, 0, 0, 0);
        IR = __builtin_amdgcn_mfma_f64_16x16x4f64(a.i, xr_[q], IR, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        zr[tj][v] = RR[v] - II[v];
        zi[tj][v] = RI[v] + IR[v];
      }
      asm volatile("" ::: "memory");  // one tile's operands at a time: registers
    }
  };
  for (; s0 < vb; s0 += step) {
    const int s = s0 + (lane & 15);
    const size_t o0 = (size_t)(12 * k4 + 3 * w) * V + base + s;  // vector k4, component 3 w
    constexpr int HC = is_half<S>() ? 3 : 1;  // components held until their scale is known
    double wr[HC][TB::NT][4], wi[HC][TB::NT][4];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int hc = c % HC;
      double xd[NQ], xe[NQ], zr[TB::NT][4], zi[TB::NT][4];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const bool in = 4 * q + k4 < n;  // padded test vectors add nothing
        xd[q] = in ? (double)xr[q].r : 0.0;
        xe[q] = in ? (double)xr[q].i : 0.0;
      }
      if (c < 2)
        load_x<Tin, NQ>(xr, X, 3 * w + c + 1, base, s0, vb, n, V);
      else if (s0 + step < vb)
        load_x<Tin, NQ>(xr, X, 3 * w, base, s0 + step, vb, n, V);
      product(zr, zi, 0, xd, xe);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        xd[q] = zr[q >> 2][q & 3];
        xe[q] = zi[q >> 2][q & 3];
      }
      product(wr[hc], wi[hc], 1, xd, xe);
      asm volatile("" ::: "memory");
      if constexpr (!is_half<S>()) {
#pragma unroll
        for (int tj = 0; tj < TB::NT; ++tj)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int a = 16 * tj + k4 + 4 * v;
            if (s < vb && a < n)
              stc_store(Wq, o0 + (size_t)(12 * (16 * tj + 4 * v) + c) * V, mk(wr[0][tj][v], wi[0][tj][v]));
          }
      }
    }
    if constexpr (is_half<S>()) {
      // the largest component of each (vector, site): this wave's three, then all
#pragma unroll
      for (int tj = 0; tj < TB::NT; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double m = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) m = fmax(m, fmax(fabs(wr[c][tj][v]), fabs(wi[c][tj][v])));
          mx[w][4 * tj + v][lane] = (float)m;
        }
      lds_barrier();
#pragma unroll
      for (int tj = 0; tj < TB::NT; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * tj + k4 + 4 * v, e = 4 * tj + v;
          if (s >= vb || a >= n) continue;
          const float fm = fmaxf(fmaxf(mx[0][e][lane], mx[1][e][lane]), fmaxf(mx[2][e][lane], mx[3][e][lane]));
          if (w == 0) Wsc[(size_t)k4 * V + base + s + (size_t)(16 * tj + 4 * v) * V] = fm;
          const double inv = fm > 0.f ? 1.0 / (double)fm : 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const size_t at = o0 + (size_t)(12 * (16 * tj + 4 * v) + c) * V;
            const __half2 hq = __halves2half2(half_rn(wr[c][tj][v] * inv), half_rn(wi[c][tj][v] * inv));
            Wq[at] = hq;
            const float2 f = __half22float2(hq);
            Wt[at] = mk(fm * f.x, fm * f.y);
          }
        }
      lds_barrier();  // mx is written again
    }
  }
}

template <typename S>
__global__ void quantize_basis_kernel(stc_t<S>* Wq, float* Wsc, const cx<double>* W, int V, int ntv, cx<float>* Wt) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ntv * V) return;
  const int s = (int)(idx % V);
  const int a = (int)(idx / V);
  if constexpr (is_half<S>()) {
    cx<double> v[12];  // one read of the 12 entries: max, then the scaled copy
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      v[k] = W[((size_t)a * 12 + k) * V + s];
      m = fmax(m, fmax(fabs(v[k].r), fabs(v[k].i)));
    }
    const float fm = (float)m;
    Wsc[idx] = fm;
    const double inv = fm > 0.f ? 1.0 / (double)fm : 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const __half2 hq = __halves2half2(half_rn(v[k].r * inv), half_rn(v[k].i * inv));
      Wq[((size_t)a * 12 + k) * V + s] = hq;
      if (Wt) {
        const float2 f = __half22float2(hq);
        Wt[((size_t)a * 12 + k) * V + s] = mk(fm * f.x, fm * f.y);
      }
    }
  } else {
    for (int k = 0; k < 12; ++k) stc_store(Wq, ((size_t)a * 12 + k) * V + s, W[((size_t)a * 12 + k) * V + s]);
  }
}

template <typename T, typename S>
__global__ void dequantize_basis_kernel(cx<T>* out, BasisView<S> bv, int V, int ntv) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ntv * 12 * V) return;
  const int s = (int)(idx % V);
  const int a = (int)(idx / ((size_t)12 * V));
  T sc = (T)1;
  if constexpr (is_half<S>()) sc = (T)bv.Wsc[(size_t)a * V + s];
  out[idx] = sc * ldc<T>(bv.W, idx);
}

// the Gram kernel with the fewest column tiles for ntv (ntv <= 32 is validated)
template <typename Tin>
void launch_qr_gram(const cx<Tin>* X, const Geom& g, int nparts, int part_sites, cx<double>* G, hipStream_t st) {
  const dim3 grid(2 * g.nblocks, nparts);
  if (g.ntv <= 16)
    qr_gram_kernel<Tin, 1><<<grid, QR_THREADS, 0, st>>>(X, g, part_sites, G);
  else if (g.ntv <= 24)
    qr_gram_kernel<Tin, 2><<<grid, QR_THREADS, 0, st>>>(X, g, part_sites, G);
  else
    qr_gram_kernel<Tin, 3><<<grid, QR_THREADS, 0, st>>>(X, g, part_sites, G);
}
// f with NQ = ceil(ntv / 4), the steps of four test vectors
template <int NQ = 8, typename F>
void with_nq(int ntv, F&& f) {
  if constexpr (NQ > 1) {
    if ((ntv + 3) / 4 < NQ) {
      with_nq<NQ - 1>(ntv, f);
      return;
    }
  }
  f(std::integral_constant<int, NQ>());
}
}  // namespace

template <typename T>
void launch_aggregate_qr(const cx<T>* X, const Geom& g, int* status, cx<double>* T1, cx<double>* T2, hipStream_t st) {
  // the Gram matrices of a small lattice's few aggregates in parts, about a
  // workgroup per compute unit
  const unsigned nagg = 2 * g.nblocks;
  const int nparts = qr_parts(g), part_sites = ((g.vblock + nparts - 1) / nparts + 15) / 16 * 16;
  cx<double>* G = T2;  // T2 replaces G's first part
  const size_t pstride = qr_factor_entries(g);
  launch_qr_gram<T>(X, g, nparts, part_sites, G, st);
  const auto chol = [&](cx<double>* out) {
    if (g.ntv <= 16)
      qr_chol_kernel<16, 64><<<nagg, 64, 0, st>>>(G, pstride, nparts, out, g, status);
    else
      qr_chol_kernel<MAX_NTV, 256><<<nagg, 256, 0, st>>>(G, pstride, nparts, out, g, status);
  };
  chol(T1);
  with_nq(g.ntv, [&](auto q) {
    qr_gram2_kernel<T, decltype(q)::value><<<dim3(nagg, nparts), QR_THREADS, 0, st>>>(X, g, part_sites, T1, G);
  });
  chol(G);
}
template <typename T, typename S>
void launch_qr_store(stc_t<S>* Wq, float* Wsc, cx<float>* Wt, const cx<T>* X, const Geom& g, const cx<double>* T1,
                     const cx<double>* T2, hipStream_t st) {
  const int ngroup = (g.vblock + 15) / 16;
  const int gy = std::max(1, std::min(ngroup, 1024 / g.nblocks));
  with_nq(g.ntv, [&](auto q) {
    qr_store_kernel<T, S, decltype(q)::value><<<dim3(g.nblocks, gy), QR_THREADS, 0, st>>>(Wq, Wsc, Wt, X, g, T1, T2);
  });
}
template void launch_aggregate_qr<double>(const cx<double>*, const Geom&, int*, cx<double>*, cx<double>*, hipStream_t);
template void launch_aggregate_qr<float>(const cx<float>*, const Geom&, int*, cx<double>*, cx<double>*, hipStream_t);
template void launch_qr_store<double, double>(stc_t<double>*, float*, cx<float>*, const cx<double>*, const Geom&,
                                              const cx<double>*, const cx<double>*, hipStream_t);
template void launch_qr_store<float, float>(stc_t<float>*, float*, cx<float>*, const cx<float>*, const Geom&,
                                            const cx<double>*, const cx<double>*, hipStream_t);
template void launch_qr_store<float, __half>(stc_t<__half>*, float*, cx<float>*, const cx<float>*, const Geom&,
                                             const cx<double>*, const cx<double>*, hipStream_t);

template <typename S>
void launch_quantize_basis(stc_t<S>* Wq, float* Wsc, const cx<double>* W, const Geom& g, hipStream_t st,
                           cx<float>* Wt) {
  size_t n = (size_t)g.ntv * g.V;
  quantize_basis_kernel<S><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(Wq, Wsc, W, g.V, g.ntv, Wt);
}
template <typename T, typename S>
void launch_dequantize_basis(cx<T>* out, const BasisView<S>& bv, const Geom& g, hipStream_t st) {
  size_t n = (size_t)g.ntv * 12 * g.V;
  dequantize_basis_kernel<T, S><<<(unsigned)((n + 255) / 256), 256, 0, st>>>(out, bv, g.V, g.ntv);
}

template void launch_quantize_basis<double>(stc_t<double>*, float*, const cx<double>*, const Geom&, hipStream_t,
                                            cx<float>*);
template void launch_quantize_basis<float>(stc_t<float>*, float*, const cx<double>*, const Geom&, hipStream_t,
                                            cx<float>*);
template void launch_quantize_basis<__half>(stc_t<__half>*, float*, const cx<double>*, const Geom&, hipStream_t,
                                            cx<float>*);
template void launch_dequantize_basis<double, double>(cx<double>*, const BasisView<double>&, const Geom&, hipStream_t);
template void launch_dequantize_basis<float, float>(cx<float>*, const BasisView<float>&, const Geom&, hipStream_t);
template void launch_dequantize_basis<float, __half>(cx<float>*, const BasisView<__half>&, const Geom&, hipStream_t);
template void launch_dequantize_basis<double, __half>(cx<double>*, const BasisView<__half>&, const Geom&, hipStream_t);
template void launch_dequantize_basis<double, float>(cx<double>*, const BasisView<float>&, const Geom&, hipStream_t);
template void launch_dequantize_basis<float, double>(cx<float>*, const BasisView<double>&, const Geom&, hipStream_t);

}  // namespace ddamg
