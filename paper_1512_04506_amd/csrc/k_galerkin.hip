// Block-crossing couplings of the coarse operator, Eq. (cgo):
//
//   (D_c)_{b, b+mu}[i][j] = w_i^{b dag} D_{b, b+mu} w_j^{b+mu}
//     = -1/2 s sum_{x in F} < w_i(x), (1 - g_mu) U_mu(x) w_j(x + mu) >
//
// where F is the last layer of block b in direction mu (its sites are the
// only ones with a forward neighbour in block b + mu) and s = -1 for the hop
// across the time boundary.  With the forward spin projection
// P_mu psi = psi_up - X_mu psi_dn (the 2-spinor a hop multiplies by the link)
// and the reconstruction R u = (u, -X_mu^dag u), (1 - g_mu) v = R P_mu v and
// <w, R u> = <P_mu w, u>, so each term is a 6-component inner product
//
//   < P_mu w_i(x), U_mu(x) P_mu w_j(x + mu) >.
//
// A basis vector lives on one chirality, so P_mu w is two of its spins
// multiplied by phases +-1, +-i: exact copies of stored values.  Per block
// and direction this is a complex contraction of 2 ntv rows by 2 ntv columns
// over 6 |F| terms, which runs on the 16x16x4 matrix cores: one workgroup per
// block and direction, the 2 ntv rows and columns of both chiralities tiled
// together (N_tv 24 is 3 x 3 full tiles; tiled per chirality it would be 4 x 4,
// N_tv 16 in FP64 4 x 4 instead of 2 x 2), the terms of a chunk of face sites
// split over the waves where the tiles' accumulators fit one wave.  Chunks
// are staged through LDS; the loads of the next chunk are issued before the
// matrix products of the current one.
//
// Bound: FP32 at N_tv 24 the matrix cores (0.5 ms of products on 24^3x48)
// and the scattered faces, FP64 the same on small lattices, where one
// workgroup per block and all directions left most compute units idle.
// 24^3x48, N_tv 24, FP16 basis: 1104 us (1872 with a workgroup per block and
// 32x32 tiles per chirality pair); 8^3x16, N_tv 16, FP64: 32 us (308).
#include <type_traits>

#include "galerkin.h"
#include "mfma_device.h"

namespace ddamg {

namespace {

using namespace dev;

// NT tiles of 16 rows and columns; the workgroup's four waves: WK parts of
// the terms by 4 / WK groups of CT tile columns; CS face sites per chunk.  A
// wave's NT x CT tiles of four accumulators are 16 registers each in FP32, 32
// in FP64, beside some 80 of staging.
template <typename T, int NT>
struct GcShape {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr int WK = F64 ? (NT <= 2 ? 4 : 1) : (NT <= 3 ? 4 : 2);
  static constexpr int CT = (NT * WK + 3) / 4;
  static constexpr int CS = F64 && NT > 2 ? 4 : 8;  // LDS
  static constexpr int ROWS = 6 * CS;               // contraction terms per chunk
  static constexpr int TPS = 256 / CS;              // staging threads per site
  static constexpr int NQ = (32 * NT + TPS - 1) / TPS;  // (spin, column) entries per thread and chunk
  static constexpr int LD = 16 * NT + 1;            // padded row length in LDS
};

// P_mu w for w of chirality ch: component sg of the 2-spinor is
// phase * w_spin.  ch = 0: (w_0, w_1).  ch = 1: -X_mu (w_2, w_3), i.e.
// mu = 0: i (w_3, w_2); mu = 1: (w_3, -w_2); mu = 2: (i w_2, -i w_3);
// mu = 3: (w_2, w_3).
__device__ inline void proj_spin(int mu, int ch, int sg, int& spin, float& pr, float& pi) {
  if (ch == 0) {
    spin = sg;
    pr = 1.f;
    pi = 0.f;
  } else if (mu == 0) {
    spin = 3 - sg;
    pr = 0.f;
    pi = 1.f;
  } else if (mu == 1) {
    spin = 3 - sg;
    pr = sg ? -1.f : 1.f;
    pi = 0.f;
  } else if (mu == 2) {
    spin = 2 + sg;
    pr = 0.f;
    pi = sg ? -1.f : 1.f;
  } else {
    spin = 2 + sg;
    pr = 1.f;
    pi = 0.f;
  }
}

__device__ inline int sel4(const int a[4], int mu) { return mu == 0 ? a[0] : mu == 1 ? a[1] : mu == 2 ? a[2] : a[3]; }

template <typename T, typename S, int NT>
__global__ __launch_bounds__(256, 2) void galerkin_cross_kernel(cx<T>* __restrict__ Dc, BasisView<S> bv,
                                                                GaugeView<T> gv, Geom g) {
  using Sh = GcShape<T, NT>;
  using Acc = typename MmAcc<T>::type;
  constexpr int CS = Sh::CS, ROWS = Sh::ROWS, NQ = Sh::NQ, LD = Sh::LD, WK = Sh::WK, CT = Sh::CT;
  constexpr int KW = ROWS / WK;  // terms per wave and chunk
  static_assert(KW % 4 == 0, "terms in fours");
  __shared__ cx<T> PQ[2][ROWS][LD];  // rows P_mu w_i(x), columns U P_mu w_j(x + mu)
  // blocks in lexicographic order, the directions of a block next to each
  // other (through the XCD swizzle): the neighbour blocks read here are
  // processed at about the same time on the same XCD
  const int wg = xcd_swizzle(blockIdx.x, gridDim.x);
  const int mu = wg & 3, bl = wg >> 2;
  int bc[4], nb[4];
  bc[0] = bl % g.NB[0];
  bc[1] = (bl / g.NB[0]) % g.NB[1];
  bc[2] = (bl / (g.NB[0] * g.NB[1])) % g.NB[2];
  bc[3] = bl / (g.NB[0] * g.NB[1] * g.NB[2]);
  for (int d = 0; d < 4; ++d) nb[d] = d == mu ? (bc[d] + 1 == g.NB[d] ? 0 : bc[d] + 1) : bc[d];
  const int ci = block_to_int(g, bc), cn = block_to_int(g, nb);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 15, lg = lane >> 4;
  const int kq = w % WK, c0 = (w / WK) * CT;     // this wave's terms and first tile column
  const int xs = t % CS, rest = t / CS;          // staging: face site and entry
  const int ntv = g.ntv, nc = g.nc, bsm = sel4(g.bs, mu), back = (bsm - 1) * sel4(g.lstr, mu);
  const int nsites = g.vblock / bsm;
  const size_t V = g.V;

  // raw values of one chunk: the basis at x (rows) and at x + mu (columns)
  // for NQ (spin, vector) entries, and the link at x
  cx<T> praw[NQ][3], qraw[NQ][3], uraw[3][3];
  T psc[NQ], qsc[NQ];
  // entry q of this thread: spin component sg of column col (chirality ch, vector av)
  auto entry = [&](int q, int& sg, int& col, int& ch, int& av) {
    const int e = rest + Sh::TPS * q;
    sg = e & 1;
    col = e >> 1;
    ch = col >= ntv ? 1 : 0;
    av = min(col - ch * ntv, ntv - 1);
  };
  auto fetch = [&](int f0) {
    const int lx = face_site(g, mu, bsm - 1, min(f0 + xs, nsites - 1));
    const unsigned x = (unsigned)(ci * g.vblock + lx);
    const unsigned y = (unsigned)(cn * g.vblock + lx - back);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) uraw[a][b] = ldc<T>(gv.U + (size_t)(mu * 9 + 3 * a + b) * V, x);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      int sg, col, ch, av, spin;
      float pr, pi;
      entry(q, sg, col, ch, av);
      proj_spin(mu, ch, sg, spin, pr, pi);
      const stc_t<S>* wb = bv.W + (size_t)(av * 12 + 3 * spin) * V;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        praw[q][c] = ldc<T>(wb + (size_t)c * V, x);
        qraw[q][c] = ldc<T>(wb + (size_t)c * V, y);
      }
      if constexpr (is_half<S>()) {
        psc[q] = bv.Wsc[(size_t)av * V + x];
        qsc[q] = bv.Wsc[(size_t)av * V + y];
      } else {
        psc[q] = qsc[q] = (T)1;
      }
    }
  };
  auto store = [&](int f0) {
    const bool fin = f0 + xs < nsites;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      int sg, col, ch, av, spin;
      float pr, pi;
      entry(q, sg, col, ch, av);
      if (col >= 16 * NT) continue;
      proj_spin(mu, ch, sg, spin, pr, pi);
      const bool ok = fin && col < nc;
      const T tr = (T)pr, ti = (T)pi;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cx<T> pv = psc[q] * praw[q][c];
        cx<T> u = mk((T)0, (T)0);
#pragma unroll
        for (int b = 0; b < 3; ++b) u = cfma(uraw[c][b], qraw[q][b], u);
        u = qsc[q] * u;
        const int row = xs * 6 + sg * 3 + c;
        PQ[0][row][col] = ok ? mk(tr * pv.r - ti * pv.i, tr * pv.i + ti * pv.r) : mk((T)0, (T)0);
        PQ[1][row][col] = ok ? mk(tr * u.r - ti * u.i, tr * u.i + ti * u.r) : mk((T)0, (T)0);
      }
    }
  };

  Acc RR[NT][CT], II[NT][CT], RI[NT][CT], IR[NT][CT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) RR[a][b][v] = II[a][b][v] = RI[a][b][v] = IR[a][b][v] = (T)0;
  const bool work = c0 < NT;  // CT columns do not always divide NT over the waves
  fetch(0);
  for (int f0 = 0; f0 < nsites; f0 += CS) {
    __syncthreads();  // the previous chunk has been consumed
    store(f0);
    if (f0 + CS < nsites) fetch(f0 + CS);
    __syncthreads();
    if (!work) continue;
#pragma unroll
    for (int k0 = 0; k0 < KW; k0 += 4) {
      const int k = kq * KW + k0 + lg;
      cx<T> qv[CT];
#pragma unroll
      for (int b = 0; b < CT; ++b) qv[b] = PQ[1][k][16 * (c0 + b) + li];
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const cx<T> pv = PQ[0][k][16 * a + li];
#pragma unroll
        for (int b = 0; b < CT; ++b) {
          RR[a][b] = mm_mfma(pv.r, qv[b].r, RR[a][b]);
          II[a][b] = mm_mfma(pv.i, qv[b].i, II[a][b]);
          RI[a][b] = mm_mfma(pv.r, qv[b].i, RI[a][b]);
          IR[a][b] = mm_mfma(pv.i, qv[b].r, IR[a][b]);
        }
      }
    }
  }
  // sum conj(p) q = (RR + II, RI - IR), over the parts of the terms in pairs
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        RR[a][b][v] += II[a][b][v];
        RI[a][b][v] -= IR[a][b][v];
      }
  if constexpr (WK > 1) {
    constexpr int PER = NT * CT * 4 * 64;  // entries of a wave
    cx<T>* sum = &PQ[0][0][0];
    static_assert((WK / 2) * (4 / WK) * PER <= 2 * ROWS * LD, "the parts fit the staging memory");
#pragma unroll
    for (int half = WK / 2; half > 0; half /= 2) {
      __syncthreads();
      cx<T>* mine = sum + (size_t)((w / WK) * (WK / 2) + kq % half) * PER + lane;
      if (kq >= half && kq < 2 * half) {
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = 0; b < CT; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[64 * ((a * CT + b) * 4 + v)] = mk(RR[a][b][v], RI[a][b][v]);
      }
      __syncthreads();
      if (kq < half) {
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = 0; b < CT; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const cx<T> o = mine[64 * ((a * CT + b) * 4 + v)];
              RR[a][b][v] += o.r;
              RI[a][b][v] += o.i;
            }
      }
    }
    if (kq) return;
  }
  if (!work) return;
  const T coef = (mu == 3 && bc[3] == g.NB[3] - 1) ? (T)0.5 : (T)-0.5;
  cx<T>* out = Dc + ((size_t)ci * 9 + 1 + 2 * mu) * nc * nc;
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < CT; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * a + mm_row<T>(lg, v), jc = 16 * (c0 + b) + li;
        if (i < nc && jc < nc) out[(size_t)jc * nc + i] = mk(coef * RR[a][b][v], coef * RI[a][b][v]);
      }
}

}  // namespace

template <typename T, typename S>
void launch_galerkin_cross(cx<T>* Dc, const BasisView<S>& bv, const GaugeView<T>& gv, const Geom& g, hipStream_t st) {
  const unsigned n = 4u * (unsigned)g.nblocks;
  if (g.nc <= 16)
    galerkin_cross_kernel<T, S, 1><<<n, 256, 0, st>>>(Dc, bv, gv, g);
  else if (g.nc <= 32)
    galerkin_cross_kernel<T, S, 2><<<n, 256, 0, st>>>(Dc, bv, gv, g);
  else if (g.nc <= 48)
    galerkin_cross_kernel<T, S, 3><<<n, 256, 0, st>>>(Dc, bv, gv, g);
  else  // N_tv <= 32
    galerkin_cross_kernel<T, S, 4><<<n, 256, 0, st>>>(Dc, bv, gv, g);
}
template void launch_galerkin_cross<float, float>(cx<float>*, const BasisView<float>&, const GaugeView<float>&,
                                                  const Geom&, hipStream_t);
template void launch_galerkin_cross<float, __half>(cx<float>*, const BasisView<__half>&, const GaugeView<float>&,
                                                   const Geom&, hipStream_t);
template void launch_galerkin_cross<double, double>(cx<double>*, const BasisView<double>&, const GaugeView<double>&,
                                                    const Geom&, hipStream_t);

}  // namespace ddamg
