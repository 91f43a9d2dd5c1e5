// Gauge-covariant network that proposes test vectors for the adaptive
// setup (the random start of Alg. 4 replaced by a learned map), trained on
// the device: layer applies, their transposes (input gradients), weight
// gradients, the span loss against a target aggregate basis (Sec. 2
// aggregates, Alg. 5 basis) with its gradient, and Adam.
//
// Fields are FP32 complex in the internal layout [channel][12][V].  A
// layer's weights are [C_out][C_in][18] complex: k = 0 multiplies phi,
// k = 1 g5 phi, and hop h = 2 mu + s (s = 0 forward, 1 backward) has
// k = 2 + 2h for T_h phi and k = 3 + 2h for g_mu T_h phi, with the parallel
// transports T_mu,+ phi(x) = U_mu(x) phi(x + mu) and T_mu,- phi(x) =
// U_mu(x - mu)^dag phi(x - mu) under the boundary conditions of D.  Between
// layers every channel passes the gate phi / sqrt(1 + |phi(x)|^2 / 12); the
// kernels apply it when they load a hidden layer's stored pre-gate output.
#include <algorithm>
#include <cmath>

#include "blas_sizes.h"
#include "dirac_device.h"
#include "mfma_device.h"

namespace ddamg {

namespace {

using namespace dev;
constexpr int NTPB = 256;
constexpr int NFEAT = 18;

// spinor of one channel (plane base f = channel * 12 V) at internal site s,
// times sign; GATE: the stored value is a pre-gate activation, apply the gate
template <bool GATE>
__device__ inline void load_in(cx<float> p[4][3], const cx<float>* f, int s, size_t V, float sign) {
  float n = 0.f;
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      p[sp][c] = elem(f + (size_t)(3 * sp + c) * V, (unsigned)s);
      n += p[sp][c].r * p[sp][c].r + p[sp][c].i * p[sp][c].i;
    }
  float sc = sign;
  if (GATE) sc *= 1.f / sqrtf(1.f + n * (1.f / 12.f));
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int c = 0; c < 3; ++c) p[sp][c] = sc * p[sp][c];
}

// t = U p (FWD) or U^dag p on the colour index of every spin
template <bool FWD>
__device__ inline void transport(cx<float> t[4][3], const cx<float> p[4][3], const cx<float> U[3][3]) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<float> acc = mk(0.f, 0.f);
#pragma unroll
      for (int b = 0; b < 3; ++b) acc = FWD ? cfma(U[a][b], p[sp][b], acc) : cfmac(U[b][a], p[sp][b], acc);
      t[sp][a] = acc;
    }
}

// The layers and their weight gradients run on the FP32 matrix cores
// (16x16x4): both are products over channels of spinor fields that a lane
// transports itself.  g_mu is a phase times a permutation of the spins, so
// g_mu T_h phi is the same operand at another spin with the phase on the
// other side.
struct SpinMap {
  int src[4];    // (g_mu p)[s] = i^phase[s] p[src[s]]
  int phase[4];
};
template <int MU>
__device__ constexpr SpinMap gamma_map() {
  if constexpr (MU == 0) return {{3, 2, 1, 0}, {3, 3, 1, 1}};
  if constexpr (MU == 1) return {{3, 2, 1, 0}, {2, 0, 0, 2}};
  if constexpr (MU == 2) return {{2, 3, 0, 1}, {3, 1, 1, 3}};
  return {{2, 3, 0, 1}, {2, 2, 2, 2}};
}

// re + i im += (wr + i wi) x, with n... the negatives (the instructions negate nothing)
__device__ inline void mm_c(mm_f4& re, mm_f4& im, float wr, float wi, float nwi, cx<float> x) {
  re = mm_mfma(wr, x.r, re);
  im = mm_mfma(wr, x.i, im);
  re = mm_mfma(nwi, x.i, re);
  im = mm_mfma(wi, x.r, im);
}
// the same with the weight times i^ph
__device__ inline void mm_cp(mm_f4& re, mm_f4& im, int ph, cx<float> w, cx<float> nw, cx<float> x) {
  if (ph == 0)
    mm_c(re, im, w.r, w.i, nw.i, x);
  else if (ph == 1)
    mm_c(re, im, nw.i, w.r, nw.r, x);
  else if (ph == 2)
    mm_c(re, im, nw.r, nw.i, w.i, x);
  else
    mm_c(re, im, w.i, nw.r, w.r, x);
}

// neighbour, boundary sign and link of hop (MU, FWD) at site p
template <int MU, bool FWD>
__device__ inline int hop_link(cx<float> U[3][3], float& sign, const SitePos& p, const Geom& g,
                               const GaugeView<float>& gv, size_t V) {
  const int sn = FWD ? nbr_fwd(g, p, MU) : nbr_bwd(g, p, MU);
  const bool wrap = MU == 3 && (FWD ? p.lc[3] == g.bs[3] - 1 && p.bc[3] == g.NB[3] - 1 : p.lc[3] == 0 && p.bc[3] == 0);
  sign = wrap ? -1.f : 1.f;
  load_link<float, float>(U, gv, MU, FWD ? p.S : sn, V);
  return sn;
}

// hop (MU, FWD) of every input channel for 16 sites and 16 output channels
template <int MU, bool FWD, bool GATE>
__device__ inline void layer_hop(mm_f4 re[12], mm_f4 im[12], const cx<float>* in, int cin, const cx<float>* Wi,
                                 const SitePos& p, const Geom& g, const GaugeView<float>& gv, size_t V, int lg) {
  constexpr SpinMap G = gamma_map<MU>();
  cx<float> U[3][3];
  float sign;
  const int sn = hop_link<MU, FWD>(U, sign, p, g, gv, V);
  constexpr int k = 2 + 2 * (2 * MU + (FWD ? 0 : 1));
  for (int j0 = 0; j0 < cin; j0 += 4) {
    const int j = min(j0 + lg, cin - 1);
    const float on = j0 + lg < cin ? 1.f : 0.f;  // channels beyond the last weigh nothing
    const Run<cx<float>, 2> w = load_run<cx<float>, 2>(Wi + (size_t)j * NFEAT + k);
    cx<float> ph[4][3], t[4][3];
    load_in<GATE>(ph, in + (size_t)j * 12 * V, sn, V, sign);
    transport<FWD>(t, ph, U);
    const cx<float> c = on * w.v[0], d = on * w.v[1], nc = neg(c), nd = neg(d);
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        mm_c(re[3 * sp + q], im[3 * sp + q], c.r, c.i, nc.i, t[sp][q]);
        mm_cp(re[3 * sp + q], im[3 * sp + q], G.phase[sp], d, nd, t[G.src[sp]][q]);
      }
  }
  asm volatile("" ::: "memory");
}

// o, the gradient with respect to the gate's output, becomes the one with
// respect to the pre-gate value psi of channel plane f at site s:
// psi -> psi g(n), n = |psi|^2 / 12, g = (1 + n)^(-1/2):
// g o + (rho g'(n) / 6) psi with rho = Re <psi, o>, g' = -g^3 / 2
__device__ inline void gate_backward(cx<float> o[12], const cx<float>* f, int s, size_t V) {
  cx<float> ps[12];
  float n = 0.f, rho = 0.f;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    ps[c] = elem(f + (size_t)c * V, (unsigned)s);
    n += ps[c].r * ps[c].r + ps[c].i * ps[c].i;
    rho += ps[c].r * o[c].r + ps[c].i * o[c].i;
  }
  const float gg = 1.f / sqrtf(1.f + n * (1.f / 12.f));
  const float cr = rho * (-0.5f * gg * gg * gg) * (1.f / 6.f);
#pragma unroll
  for (int c = 0; c < 12; ++c) o[c] = gg * o[c] + cr * ps[c];
}

// out[i] = sum_jk W[i][j][k] F_k(in_j) for 16 output channels (blockIdx.y).
// A wave takes 16 sites: lane (li, lg) transports channel 4 jj + lg at site
// li, which makes it the B operand (K = 4 channels, N = 16 sites) of the
// products with the weights of 16 outputs, one tile per spin and colour; the
// result holds four output channels of a site with all twelve components, as
// the gate's backward wants them.  Bound: the FP32 matrix cores (816 products
// of 32 cycles per 16 sites and 4 channels beside some 1200 cycles of
// vector work).  16 -> 16 channels on 16^4: 420 us (first layer without gate
// 270), from 850 (500) with a lane per site and four output channels that
// repeated loads, gate and transport for each group of four.  The sum runs in
// two chains of half the length: one chain of this order was up to 1.24e-6
// off in the gradients where the vector units were 1.19e-6, two are 0.88e-6.
// GATE_IN: the input planes hold pre-gate activations (gate applied on load).
// GATE_BWD: the result is the gradient with respect to the gate's output of
// the channels whose pre-gate values are in pre; store instead the gradient
// with respect to those pre-gate values (the gate's backward).
template <bool GATE_IN, bool GATE_BWD>
__global__ __launch_bounds__(NTPB, 2) void net_layer_kernel(cx<float>* __restrict__ out,
                                                            const cx<float>* __restrict__ in,
                                                            const cx<float>* __restrict__ W, int cin, int cout,
                                                            GaugeView<float> gv, Geom g,
                                                            const cx<float>* __restrict__ pre) {
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int unit = blockIdx.x * (NTPB / 64) + (threadIdx.x >> 6);
  if (unit * 16 >= g.V) return;  // V is a multiple of 16: two or more blocks in each direction
  const int s = unit * 16 + li;
  const int i0 = blockIdx.y * 16;
  const size_t V = g.V;
  const SitePos p = site_pos(g, s);
  const cx<float>* Wi = W + (size_t)min(i0 + li, cout - 1) * cin * NFEAT;  // rows beyond the last are dropped
  mm_f4 re[12], im[12];
#pragma unroll
  for (int c = 0; c < 12; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) re[c][v] = im[c][v] = 0.f;
  for (int j0 = 0; j0 < cin; j0 += 4) {
    const int j = min(j0 + lg, cin - 1);
    const float on = j0 + lg < cin ? 1.f : 0.f;
    const Run<cx<float>, 2> w = load_run<cx<float>, 2>(Wi + (size_t)j * NFEAT);
    cx<float> ph[4][3];
    load_in<GATE_IN>(ph, in + (size_t)j * 12 * V, s, V, 1.f);
    // a phi + b g5 phi, g5 = diag(-1, -1, +1, +1)
    const cx<float> lo = on * (w.v[0] - w.v[1]), hi = on * (w.v[0] + w.v[1]);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const cx<float> ww = c < 6 ? lo : hi;
      mm_c(re[c], im[c], ww.r, ww.i, -ww.i, ph[c / 3][c % 3]);
    }
  }
  layer_hop<0, true, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<0, false, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<1, true, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<1, false, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  // two chains of half the length: the first half of the sum waits, as far as
  // they go in registers, the other components in the output planes
  constexpr int HOLD = 8;
  mm_f4 hr[HOLD], hi[HOLD];
#pragma unroll
  for (int c = 0; c < 12; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + 4 * lg + v;
      if (c < HOLD) {
        hr[c][v] = re[c][v];
        hi[c][v] = im[c][v];
      } else if (i < cout) {
        out[((size_t)i * 12 + c) * V + s] = mk(re[c][v], im[c][v]);
      }
      re[c][v] = im[c][v] = 0.f;
    }
  layer_hop<2, true, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<2, false, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<3, true, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  layer_hop<3, false, GATE_IN>(re, im, in, cin, Wi, p, g, gv, V, lg);
  // lane: site li, output channels i0 + 4 lg + v
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + 4 * lg + v;
    if (i >= cout) continue;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const cx<float> o = c < HOLD ? mk(hr[c][v], hi[c][v]) : out[((size_t)i * 12 + c) * V + s];
      re[c][v] += o.r;
      im[c][v] += o.i;
    }
    cx<float> o[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) o[c] = mk(re[c][v], im[c][v]);
    if (GATE_BWD) gate_backward(o, pre + (size_t)i * 12 * V, s, V);
#pragma unroll
    for (int c = 0; c < 12; ++c) out[((size_t)i * 12 + c) * V + s] = o[c];
  }
}

// i^ph a
__device__ inline cx<float> times_ip(int ph, cx<float> a) {
  return ph == 0 ? a : ph == 1 ? times_i(a) : ph == 2 ? neg(a) : times_mi(a);
}

// hop (MU, FWD) of every input channel for a lane's site and OG output channels
constexpr int OG = 4;
template <int MU, bool FWD, bool GATE>
__device__ inline void thin_hop(cx<float> acc[OG][12], const cx<float>* in, int cin, const cx<float>* const w[OG],
                                const SitePos& p, const Geom& g, const GaugeView<float>& gv, size_t V) {
  constexpr SpinMap G = gamma_map<MU>();
  constexpr int k = 2 + 2 * (2 * MU + (FWD ? 0 : 1));
  cx<float> U[3][3];
  float sign;
  const int sn = hop_link<MU, FWD>(U, sign, p, g, gv, V);
  for (int j = 0; j < cin; ++j) {
    cx<float> ph[4][3], t[4][3];
    load_in<GATE>(ph, in + (size_t)j * 12 * V, sn, V, sign);
    transport<FWD>(t, ph, U);
#pragma unroll
    for (int q = 0; q < OG; ++q) {
      const cx<float> c = w[q][(size_t)j * NFEAT + k], d = w[q][(size_t)j * NFEAT + k + 1];
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a)
          acc[q][3 * sp + a] = cfma(d, times_ip(G.phase[sp], t[G.src[sp]][a]), cfma(c, t[sp][a], acc[q][3 * sp + a]));
    }
  }
  asm volatile("" ::: "memory");
}

// The same layer for few channels: a lane per site and four output channels
// (blockIdx.y), which repeats loads, gate and transport for every four outputs
// but computes no channels that are not there.  Bound: loads and transports.  1
// to 1 channels on 16^3x32 63 us (192 on the matrix cores), 4 to 4 195 (270).
template <bool GATE_IN, bool GATE_BWD>
__global__ __launch_bounds__(NTPB, 2) void net_thin_layer_kernel(cx<float>* __restrict__ out,
                                                                 const cx<float>* __restrict__ in,
                                                                 const cx<float>* __restrict__ W, int cin, int cout,
                                                                 GaugeView<float> gv, Geom g,
                                                                 const cx<float>* __restrict__ pre) {
  const int s = blockIdx.x * NTPB + threadIdx.x;
  if (s >= g.V) return;
  const int i0 = blockIdx.y * OG;
  const size_t V = g.V;
  const SitePos p = site_pos(g, s);
  cx<float> acc[OG][12], half[OG][12];
  const cx<float>* w[OG];  // weights of input channel 0
#pragma unroll
  for (int q = 0; q < OG; ++q) {
    w[q] = W + (size_t)min(i0 + q, cout - 1) * cin * NFEAT;
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[q][c] = mk(0.f, 0.f);
  }
  for (int j = 0; j < cin; ++j) {
    cx<float> ph[4][3];
    load_in<GATE_IN>(ph, in + (size_t)j * 12 * V, s, V, 1.f);
    // a phi + b g5 phi, g5 = diag(-1, -1, +1, +1)
#pragma unroll
    for (int q = 0; q < OG; ++q) {
      const cx<float> a = w[q][(size_t)j * NFEAT], b = w[q][(size_t)j * NFEAT + 1];
      const cx<float> lo = a - b, hi = a + b;
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[q][c] = cfma(c < 6 ? lo : hi, ph[c / 3][c % 3], acc[q][c]);
    }
  }
  thin_hop<0, true, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<0, false, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<1, true, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<1, false, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  // two chains of half the length, as above
#pragma unroll
  for (int q = 0; q < OG; ++q)
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      half[q][c] = acc[q][c];
      acc[q][c] = mk(0.f, 0.f);
    }
  thin_hop<2, true, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<2, false, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<3, true, GATE_IN>(acc, in, cin, w, p, g, gv, V);
  thin_hop<3, false, GATE_IN>(acc, in, cin, w, p, g, gv, V);
#pragma unroll
  for (int q = 0; q < OG; ++q) {
    const int i = i0 + q;
    if (i >= cout) break;
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[q][c] = acc[q][c] + half[q][c];
    if (GATE_BWD) gate_backward(acc[q], pre + (size_t)i * 12 * V, s, V);
#pragma unroll
    for (int c = 0; c < 12; ++c) out[((size_t)i * 12 + c) * V + s] = acc[q][c];
  }
}

// Wb[j][i][k]: the weights of the transposed layer (input gradients):
// conj(W[i][j][k]) with the hop direction reversed (T_mu,s^dag = T_mu,-s;
// g5 and g_mu are Hermitian and commute with the transports)
__global__ void net_transpose_kernel(cx<float>* Wb, const cx<float>* W, int cin, int cout) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= cin * cout * NFEAT) return;
  const int k = e % NFEAT, i = (e / NFEAT) % cout, j = e / (NFEAT * cout);
  int ks = k;
  if (k >= 2) {
    const int h = (k - 2) >> 1, t = (k - 2) & 1;
    ks = 2 + 2 * (h ^ 1) + t;
  }
  Wb[((size_t)j * cout + i) * NFEAT + k] = conj(W[((size_t)i * cin + j) * NFEAT + ks]);
}

// Partial weight gradients Gamma_w[i][j][k] = sum_x <F_k(in_j)(x), gam_i(x)>
// over the sites of one chunk (blockIdx.x) for the two features of one hop
// (blockIdx.y = 0 .. 7) or of the site itself (8):
// part[(chunk cout + i) cin + j][k] (FP64).
// A wave takes 16 sites at a time: lane (li, lg) transports channel 4 jj + lg
// at site li, spin by spin into the wave's LDS tile, from which lane (li, lg)
// reads channel li at the sites 4 lg .. 4 lg + 3: the A operand of products
// over sites (K) with gam_i at the same sites, read as 32-byte runs.  FP32
// accumulators are emptied into FP64 ones after each spin, chains of 48 products.
// Bound: the FP32 matrix cores (768 products per hop and 16 sites at 24
// output channels).  16 x 16 channels on 16^4: 762 us (first layer without gate 510),
// from 1997 (1074) with one site and 2 x 2 channels per lane.
constexpr int WG_LD = 18;  // padded row (16 sites) of the LDS tile

template <int JOB, bool GATE>
__device__ inline void wgrad_job(cx<double>* __restrict__ part, const cx<float>* __restrict__ in,
                                 const cx<float>* __restrict__ gam, int cin, int cout, const GaugeView<float>& gv,
                                 const Geom& g, int jb, int ctot, int ib, cx<float>* smem) {
  constexpr bool SELF = JOB == 8;
  constexpr int MU = SELF ? 0 : JOB / 2;
  constexpr bool FWD = JOB % 2 == 0;
  constexpr SpinMap G = gamma_map<MU>();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
  const size_t V = g.V;
  cx<float>* tile = smem + (size_t)w * 3 * 16 * WG_LD;
  double* red = reinterpret_cast<double*>(smem);
  const int nunit = g.V / 16, stride = gridDim.x * (NTPB / 64);
  mm_f4 acc[4];  // feature 0 re, im, feature 1 re, im
  double tot[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        acc[q][v] = 0.f;
        tot[q][v] = 0.0;
      }
    const cx<float>* gp = gam + (size_t)min(ib + li, cout - 1) * 12 * V + 4 * lg;
  for (int unit = blockIdx.x * (NTPB / 64) + w; unit < nunit; unit += stride) {
    const int s0 = unit * 16, s = s0 + li;
    const SitePos p = site_pos(g, s);
    cx<float> U[3][3];
    int sn = s;
    float sign = 1.f;
    if constexpr (!SELF) sn = hop_link<MU, FWD>(U, sign, p, g, gv, V);
    float sc[4];  // sign and gate of channel 4 jj + lg at sn
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      sc[jj] = sign;
      if constexpr (GATE) {
        const cx<float>* f = in + (size_t)min(4 * jj + lg, cin - 1) * 12 * V;
        float n = 0.f;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
          const cx<float> v = elem(f + (size_t)c * V, (unsigned)sn);
          n += v.r * v.r + v.i * v.i;
        }
        sc[jj] *= 1.f / sqrtf(1.f + n * (1.f / 12.f));
        asm volatile("" ::: "memory");  // one channel's loads at a time: registers
      }
    }
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const cx<float>* f = in + ((size_t)min(4 * jj + lg, cin - 1) * 12 + 3 * sp) * V;
        cx<float> x[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) x[c] = sc[jj] * elem(f + (size_t)c * V, (unsigned)sn);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          cx<float> t = x[c];
          if constexpr (!SELF) {
            t = mk(0.f, 0.f);
#pragma unroll
            for (int b = 0; b < 3; ++b) t = FWD ? cfma(U[c][b], x[b], t) : cfmac(U[b][c], x[b], t);
          }
          tile[(c * 16 + 4 * jj + lg) * WG_LD + li] = t;
        }
      }
      // the tile is the wave's own: order its writes before the reads below
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // spin d of g_mu t is i^ph times this spin (g5: -1, -1, +1, +1 in place)
      int d = sp, ph = sp < 2 ? 2 : 0;
      if constexpr (!SELF) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (G.src[q] == sp) {
            d = q;
            ph = G.phase[q];
          }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Run<cx<float>, 4> t;
#pragma unroll
        for (int i = 0; i < 4; ++i) t.v[i] = tile[(c * 16 + li) * WG_LD + 4 * lg + i];
        const Run<cx<float>, 4> g0 = load_run<cx<float>, 4>(gp + (size_t)(3 * sp + c) * V + s0);
        const Run<cx<float>, 4> g1 = load_run<cx<float>, 4>(gp + (size_t)(3 * d + c) * V + s0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // conj(t) gam: (tr gr + ti gi) + i (tr gi - ti gr)
            const cx<float> a = t.v[i], na = neg(a);
            mm_c(acc[0], acc[1], a.r, na.i, a.i, g0.v[i]);
            // conj(i^ph t) gam = i^-ph conj(t) gam
            mm_cp(acc[2], acc[3], (4 - ph) & 3, mk(a.r, na.i), mk(na.r, a.i), g1.v[i]);
          }
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          tot[q][v] += (double)acc[q][v];
          acc[q][v] = 0.f;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the reads are done before the next spin is written
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  // the waves' sums, one after the other in a fixed order: red [16][64],
  // in the tiles' place
  __syncthreads();
  for (int k = 0; k < NTPB / 64; ++k) {
    if (w == k) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double& r = red[(q * 4 + v) * 64 + lane];
            const double t = tot[q][v];
            r = k == 0 ? t : r + t;
          }
    }
    __syncthreads();
  }
  // lane: rows j = 4 lg + v, column i = li + 16 n
  if (w == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = 4 * lg + v, i = ib + li;
        if (j >= cin || i >= cout) continue;
        cx<double>* o = part + (((size_t)blockIdx.x * cout + i) * ctot + jb + j) * NFEAT + (SELF ? 0 : 2 + 2 * JOB);
        auto at = [&](int q) { return red[(q * 4 + v) * 64 + lane]; };
        o[0] = mk(at(0), at(1));
        o[1] = mk(at(2), at(3));
      }
  }
}

// blockIdx: chunk, job, tile of 16 input channels and 16 output channels
template <bool GATE>
__global__ __launch_bounds__(NTPB, 2) void net_wgrad_kernel(cx<double>* __restrict__ part,
                                                            const cx<float>* __restrict__ in,
                                                            const cx<float>* __restrict__ gam, int cin, int cout,
                                                            GaugeView<float> gv, Geom g) {
  __shared__ __attribute__((aligned(16))) cx<float> smem[(NTPB / 64) * 3 * 16 * WG_LD];
  static_assert(sizeof(smem) >= sizeof(double) * 16 * 64, "reduction area");
  const int nj = (cin + 15) / 16, jb = 16 * (blockIdx.z % nj), ib = 16 * (blockIdx.z / nj), cl = min(16, cin - jb);
  const cx<float>* ij = in + (size_t)jb * 12 * g.V;
  switch (blockIdx.y) {
    case 0: wgrad_job<0, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 1: wgrad_job<1, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 2: wgrad_job<2, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 3: wgrad_job<3, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 4: wgrad_job<4, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 5: wgrad_job<5, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 6: wgrad_job<6, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    case 7: wgrad_job<7, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
    default: wgrad_job<8, GATE>(part, ij, gam, cl, cout, gv, g, jb, cin, ib, smem); break;
  }
}

// <t, gam> and <g_mu t, gam> of both hops of direction MU, added to acc
template <int MU, bool FWD, bool GATE>
__device__ inline void thin_wgrad_hop(cx<float> acc[2][NFEAT], const cx<float>* f, const cx<float> gm[2][12],
                                      const SitePos& p, const Geom& g, const GaugeView<float>& gv, size_t V) {
  constexpr SpinMap G = gamma_map<MU>();
  constexpr int k = 2 + 2 * (2 * MU + (FWD ? 0 : 1));
  cx<float> U[3][3], ph[4][3], t[4][3];
  float sign;
  const int sn = hop_link<MU, FWD>(U, sign, p, g, gv, V);
  load_in<GATE>(ph, f, sn, V, sign);
  transport<FWD>(t, ph, U);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    cx<float> a = mk(0.f, 0.f), b = mk(0.f, 0.f);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      a = cfmac(t[c / 3][c % 3], gm[q][c], a);
      b = cfmac(times_ip(G.phase[c / 3], t[G.src[c / 3]][c % 3]), gm[q][c], b);
    }
    acc[q][k] = acc[q][k] + a;
    acc[q][k + 1] = acc[q][k + 1] + b;
  }
  asm volatile("" ::: "memory");
}

// The same for few channels: a lane per site, one input and two output
// channels (blockIdx.y), all features; at most 16 sites per lane in FP32,
// then FP64.  Bound: loads and transports, repeated for every two outputs.  The
// backward pass of a layer of 1 to 1 channels on 16^3x32 266 us (970 on the matrix
// cores), 4 to 4 354 (1013).
template <bool GATE>
__global__ __launch_bounds__(NTPB) void net_thin_wgrad_kernel(cx<double>* __restrict__ part,
                                                              const cx<float>* __restrict__ in,
                                                              const cx<float>* __restrict__ gam, int cin, int cout,
                                                              GaugeView<float> gv, Geom g) {
  __shared__ cx<double> red[NTPB / 64][2 * NFEAT];
  const int ngroup = (cout + 1) / 2, j = blockIdx.y / ngroup, i0 = 2 * (blockIdx.y % ngroup);
  const size_t V = g.V;
  const cx<float>* f = in + (size_t)j * 12 * V;
  cx<float> acc[2][NFEAT];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int k = 0; k < NFEAT; ++k) acc[q][k] = mk(0.f, 0.f);
  for (int s = blockIdx.x * NTPB + threadIdx.x; s < g.V; s += gridDim.x * NTPB) {
    const SitePos p = site_pos(g, s);
    cx<float> gm[2][12], ph[4][3];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int c = 0; c < 12; ++c) gm[q][c] = elem(gam + ((size_t)min(i0 + q, cout - 1) * 12 + c) * V, (unsigned)s);
    load_in<GATE>(ph, f, s, V, 1.f);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      cx<float> lo = mk(0.f, 0.f), hi = mk(0.f, 0.f);  // spins 0, 1 and 2, 3
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        lo = cfmac(ph[c / 3][c % 3], gm[q][c], lo);
        hi = cfmac(ph[2 + c / 3][c % 3], gm[q][6 + c], hi);
      }
      acc[q][0] = acc[q][0] + (hi + lo);
      acc[q][1] = acc[q][1] + (hi - lo);
    }
    thin_wgrad_hop<0, true, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<0, false, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<1, true, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<1, false, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<2, true, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<2, false, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<3, true, GATE>(acc, f, gm, p, g, gv, V);
    thin_wgrad_hop<3, false, GATE>(acc, f, gm, p, g, gv, V);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int k = 0; k < NFEAT; ++k) {
      double re = acc[q][k].r, im = acc[q][k].i;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
      }
      if (lane == 0) red[w][q * NFEAT + k] = mk(re, im);
    }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * NFEAT; e += NTPB) {
    const int q = e / NFEAT, k = e % NFEAT;
    if (i0 + q >= cout) continue;
    cx<double> sum = red[0][e];
    for (int x = 1; x < NTPB / 64; ++x) sum = sum + red[x][e];
    part[(((size_t)blockIdx.x * cout + i0 + q) * cin + j) * NFEAT + k] = sum;
  }
}

// grad[e] = 2 sum_chunk part[chunk][e] (dL/dRe w + i dL/dIm w from the
// Wirtinger sums), summed in a fixed order
__global__ void net_wgrad_final_kernel(cx<float>* grad, const cx<double>* part, size_t n, int nchunk) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  cx<double> s = mk(0.0, 0.0);
  for (int c = 0; c < nchunk; ++c) s = s + part[(size_t)c * n + e];
  grad[e] = cvt<float>(2.0 * s);
}

// Span loss of the proposal X against the target basis T on one aggregate
// per workgroup (blockIdx.x = 2 ci + h), N_tv <= 32, in FP64:
//   G = X^H X, C = X^H T, Z = G^-1 C (Cholesky),
//   loss_agg = ||T||^2 - Re tr(C^H Z),
//   gam = -scale (T - X Z) Z^H = T M_T + X M_X on the aggregate's components,
//   M_T = -scale Z^H, M_X = scale Z Z^H.
// status is set to 1 if G is not positive definite.
// The products over the aggregate's rows run on the FP64 matrix cores
// (16x16x4), fed from memory: for G and C lane (li, lg) holds vector li and
// the sites 4 lg .. 4 lg + 3 of a 16-site run (the K order is the same for both
// operands), for gam vector 4 k + lg and site li, so that the results leave
// in 128-byte runs.  Cholesky and the triangular solves go by columns, all
// lanes on the rest.  One lane did the Cholesky and one lane per row the
// gradient, with X read again for every entry of Z: 16^4, N_tv 24 (512
// aggregates): 455 us, from 3130.
constexpr int SLT = 256;  // lanes
constexpr int SLD = 33;   // padded row of the LDS matrices

template <int MT>
__global__ __launch_bounds__(SLT, 2) void net_span_loss_kernel(cx<float>* __restrict__ gam,
                                                               double* __restrict__ loss_agg,
                                                               const cx<float>* __restrict__ X,
                                                               const cx<float>* __restrict__ T, Geom g, int ntv,
                                                               double scale, int* status) {
  constexpr int NP = MT * (MT + 1) / 2 + MT * MT;  // tiles of G (m <= n) and of C
  // G, C and Z, and in their place before them the tiles of the waves, which
  // need more than one matrix's room: one array, whose parts may overlap
  __shared__ cx<double> mats[3 * 32 * SLD];
  __shared__ double wsum[SLT / 64];
  cx<double>*Gs = mats, *Cs = mats + 32 * SLD, *Zs = mats + 2 * 32 * SLD;
  double* red = reinterpret_cast<double*>(mats);
  static_assert(sizeof(double) * NP * 8 * 64 <= sizeof(mats), "reduction area");
  const int ci = blockIdx.x >> 1, h = blockIdx.x & 1;
  const size_t V = g.V;
  const int vb = g.vblock;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 15, lg = lane >> 4;
  const size_t base = (size_t)(6 * h) * V + (size_t)ci * vb;
  mm_d4 re[NP], im[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) re[q][v] = im[q][v] = 0.0;
  double tn = 0.0;
  {
    const cx<float>*Xp[MT], *Tp[MT];
    bool real[MT];  // vectors beyond the last are read as the last
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int a = min(li + 16 * m, ntv - 1);
      real[m] = li + 16 * m < ntv;
      Xp[m] = X + (size_t)a * 12 * V + base;
      Tp[m] = T + (size_t)a * 12 * V + base;
    }
    for (int s0 = 16 * w; s0 < vb; s0 += 16 * (SLT / 64)) {
      const int s = s0 + 4 * lg;
      const bool full = s0 + 16 <= vb;
      for (int k = 0; k < 6; ++k) {
        Run<cx<float>, 4> xv[MT], tv[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          if (full) {
            xv[m] = load_run<cx<float>, 4>(Xp[m] + (size_t)k * V + s);
            tv[m] = load_run<cx<float>, 4>(Tp[m] + (size_t)k * V + s);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {  // sites beyond the block contribute zero
              const bool in = s + i < vb;
              const size_t at = (size_t)k * V + min(s + i, vb - 1);
              const cx<float> xa = Xp[m][at], ta = Tp[m][at];
              xv[m].v[i] = in ? xa : mk(0.f, 0.f);
              tv[m].v[i] = in ? ta : mk(0.f, 0.f);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          cx<double> x[MT], y[MT];
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            x[m] = cvt<double>(xv[m].v[i]);
            y[m] = cvt<double>(tv[m].v[i]);
            if (real[m]) tn += y[m].r * y[m].r + y[m].i * y[m].i;
          }
          int q = 0;
          auto tile = [&](cx<double> a, cx<double> b) {  // conj(a) b
            re[q] = mm_mfma(a.r, b.r, re[q]);
            im[q] = mm_mfma(a.r, b.i, im[q]);
            re[q] = mm_mfma(a.i, b.i, re[q]);
            im[q] = mm_mfma(-a.i, b.r, im[q]);
            ++q;
          };
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = m; n < MT; ++n) tile(x[m], x[n]);
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < MT; ++n) tile(x[m], y[n]);
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) tn += __shfl_xor(tn, o, 64);
  if (lane == 0) wsum[w] = tn;
  for (int k = 0; k < SLT / 64; ++k) {
    if (w == k)
#pragma unroll
      for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double& r = red[(q * 8 + v) * 64 + lane];
          double& i = red[(q * 8 + 4 + v) * 64 + lane];
          r = k == 0 ? re[q][v] : r + re[q][v];
          i = k == 0 ? im[q][v] : i + im[q][v];
        }
    __syncthreads();
  }
  if (w == 0)
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        re[q][v] = red[(q * 8 + v) * 64 + lane];
        im[q][v] = red[(q * 8 + 4 + v) * 64 + lane];
      }
  __syncthreads();
  if (w == 0) {
    int q = 0;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = m; n < MT; ++n, ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * m + mm_row<double>(lg, v), b = 16 * n + li;
          const cx<double> e = mk(re[q][v], im[q][v]);
          Gs[a * SLD + b] = e;
          if (n > m) Gs[b * SLD + a] = conj(e);
        }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < MT; ++n, ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * m + mm_row<double>(lg, v), b = 16 * n + li;
          Cs[a * SLD + b] = Zs[a * SLD + b] = mk(re[q][v], im[q][v]);
        }
  }
  __syncthreads();
  // G = L L^H in place (lower triangle), right-looking; every lane reads the
  // same pivot, so a failure is uniform
  for (int k = 0; k < ntv; ++k) {
    const double d = Gs[k * SLD + k].r;
    if (!(d > 0.0)) {
      if (t == 0) {
        atomicExch(status, 1);
        loss_agg[blockIdx.x] = 0.0;
      }
      return;
    }
    const double lk = sqrt(d);
    __syncthreads();
    for (int i = k + t; i < ntv; i += SLT)
      Gs[i * SLD + k] = i == k ? mk(lk, 0.0) : (1.0 / lk) * Gs[i * SLD + k];
    __syncthreads();
    const int m = ntv - k - 1;
    for (int e = t; e < m * m; e += SLT) {
      const int i = k + 1 + e / m, j = k + 1 + e % m;
      if (j <= i) Gs[i * SLD + j] = Gs[i * SLD + j] - Gs[i * SLD + k] * conj(Gs[j * SLD + k]);
    }
    __syncthreads();
  }
  // Z = L^-H L^-1 C, column by column of L
  for (int k = 0; k < ntv; ++k) {
    const double inv = 1.0 / Gs[k * SLD + k].r;
    if (t < ntv) Zs[k * SLD + t] = inv * Zs[k * SLD + t];
    __syncthreads();
    for (int e = t; e < (ntv - k - 1) * ntv; e += SLT) {
      const int i = k + 1 + e / ntv, b = e % ntv;
      Zs[i * SLD + b] = Zs[i * SLD + b] - Gs[i * SLD + k] * Zs[k * SLD + b];
    }
    __syncthreads();
  }
  for (int k = ntv - 1; k >= 0; --k) {
    const double inv = 1.0 / Gs[k * SLD + k].r;
    if (t < ntv) Zs[k * SLD + t] = inv * Zs[k * SLD + t];
    __syncthreads();
    for (int e = t; e < k * ntv; e += SLT) {
      const int i = e / ntv, b = e % ntv;
      Zs[i * SLD + b] = Zs[i * SLD + b] - conj(Gs[k * SLD + i]) * Zs[k * SLD + b];
    }
    __syncthreads();
  }
  // loss: ||T||^2 - Re tr(C^H Z)
  double tr = 0.0;
  for (int e = t; e < ntv * ntv; e += SLT) {
    const int at = e / ntv * SLD + e % ntv;
    tr += Cs[at].r * Zs[at].r + Cs[at].i * Zs[at].i;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o, 64);
  double tt = 0.0;
  for (int k = 0; k < SLT / 64; ++k) tt += wsum[k];
  __syncthreads();
  if (lane == 0) wsum[w] = tr;
  __syncthreads();
  if (t == 0) {
    for (int k = 0; k < SLT / 64; ++k) tt -= wsum[k];
    loss_agg[blockIdx.x] = tt;
  }
  // M_X = scale (Z Z^H) into Gs (row c, column a: what multiplies X_c in
  // gam_a), M_T into Cs (row b, column a), zero rows up to a multiple of 4
  const int nk = (ntv + 3) / 4;
  for (int e = t; e < 4 * nk * 32; e += SLT) {
    const int c = e / 32, a = e % 32;
    cx<double> q = mk(0.0, 0.0), m = q;
    if (c < ntv && a < ntv) {
      for (int b = 0; b < ntv; ++b) q = q + Zs[c * SLD + b] * conj(Zs[a * SLD + b]);
      m = conj(Zs[a * SLD + c]);
    }
    Gs[c * SLD + a] = scale * q;
    Cs[c * SLD + a] = -scale * m;
  }
  __syncthreads();
  // gam_a = sum_c M_X[c][a] X_c + sum_b M_T[b][a] T_b, units of 16 sites of one component
  const int nrun = (vb + 15) / 16;
  for (int u = w; u < 6 * nrun; u += SLT / 64) {
    const int k = u / nrun, s0 = 16 * (u % nrun);
    const bool in = s0 + li < vb;
    const size_t at = base + (size_t)k * V + min(s0 + li, vb - 1);
    mm_d4 gr[MT], gi[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) gr[m][v] = gi[m][v] = 0.0;
#pragma unroll 2
    for (int kk = 0; kk < nk; ++kk) {
      const int c = 4 * kk + lg;  // rows beyond ntv are zero in the matrices
      const size_t plane = (size_t)min(c, ntv - 1) * 12 * V;
      const cx<double> x = cvt<double>(X[plane + at]), y = cvt<double>(T[plane + at]);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const cx<double> ax = Gs[c * SLD + 16 * m + li], ay = Cs[c * SLD + 16 * m + li];
        gr[m] = mm_mfma(ax.r, x.r, gr[m]);
        gi[m] = mm_mfma(ax.r, x.i, gi[m]);
        gr[m] = mm_mfma(-ax.i, x.i, gr[m]);
        gi[m] = mm_mfma(ax.i, x.r, gi[m]);
        gr[m] = mm_mfma(ay.r, y.r, gr[m]);
        gi[m] = mm_mfma(ay.r, y.i, gi[m]);
        gr[m] = mm_mfma(-ay.i, y.i, gr[m]);
        gi[m] = mm_mfma(ay.i, y.r, gi[m]);
      }
    }
    if (in)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * m + mm_row<double>(lg, v);
          if (a < ntv) gam[(size_t)a * 12 * V + at] = mk((float)gr[m][v], (float)gi[m][v]);
        }
  }
}

// out = scale * sum in[i], one wave, summed in a fixed order
__global__ void sum_kernel(double* out, const double* in, int n, double scale) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += in[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (threadIdx.x == 0) *out = scale * s;
}

// Adam on the real and imaginary parts (n reals), bias corrections c1, c2
__global__ void adam_kernel(float* w, float* m, float* v, const float* grad, size_t n, float lr, float b1, float b2,
                            float c1, float c2, float eps) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const float gr = grad[e];
  const float mm = b1 * m[e] + (1.f - b1) * gr;
  const float vv = b2 * v[e] + (1.f - b2) * gr * gr;
  m[e] = mm;
  v[e] = vv;
  w[e] -= lr * (mm * c1) / (sqrtf(vv * c2) + eps);
}

inline unsigned cdiv(size_t a, size_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

void launch_net_layer(cx<float>* out, const cx<float>* in, const cx<float>* W, int cin, int cout, bool gate_in,
                      const cx<float>* gate_bwd_pre, const GaugeView<float>& gv, const Geom& g, hipStream_t st) {
  const bool thin = net_layer_thin(cin, cout, g.V);
  const dim3 grid(thin ? cdiv(g.V, NTPB) : cdiv(g.V, 16 * (NTPB / 64)), cdiv(cout, thin ? OG : 16));
  auto go = [&](auto kernel) { kernel<<<grid, NTPB, 0, st>>>(out, in, W, cin, cout, gv, g, gate_bwd_pre); };
  if (gate_bwd_pre)
    go(thin ? net_thin_layer_kernel<false, true> : net_layer_kernel<false, true>);
  else if (gate_in)
    go(thin ? net_thin_layer_kernel<true, false> : net_layer_kernel<true, false>);
  else
    go(thin ? net_thin_layer_kernel<false, false> : net_layer_kernel<false, false>);
}

void launch_net_transpose(cx<float>* Wb, const cx<float>* W, int cin, int cout, hipStream_t st) {
  const int n = cin * cout * NFEAT;
  net_transpose_kernel<<<cdiv(n, 256), 256, 0, st>>>(Wb, W, cin, cout);
}

// chunks of the weight gradients: with the nine jobs some 600 workgroups on
// lattices from 16^4 up, and at least eight units of 16 sites per wave; for few
// channels 256 workgroups or 16 sites per lane, whichever is more
int net_wgrad_chunks(int cin, int cout, const Geom& g) {
  if (net_wgrad_thin(cin, cout, g.V)) {
    const int jobs = cin * (int)cdiv(cout, 2);
    return std::max((int)cdiv(g.V, 16 * NTPB), std::min((int)cdiv(g.V, NTPB), 256 / jobs));
  }
  return std::max(1, std::min(64, g.V / 512));
}

void launch_net_wgrad(cx<float>* grad, cx<double>* part, const cx<float>* in, bool gate_in, const cx<float>* gam,
                      int cin, int cout, const GaugeView<float>& gv, const Geom& g, hipStream_t st) {
  const int nchunk = net_wgrad_chunks(cin, cout, g);
  const bool thin = net_wgrad_thin(cin, cout, g.V);
  const dim3 grid(nchunk, thin ? cin * cdiv(cout, 2) : 9, thin ? 1 : cdiv(cin, 16) * cdiv(cout, 16));
  auto go = [&](auto kernel) { kernel<<<grid, NTPB, 0, st>>>(part, in, gam, cin, cout, gv, g); };
  if (gate_in)
    go(thin ? net_thin_wgrad_kernel<true> : net_wgrad_kernel<true>);
  else
    go(thin ? net_thin_wgrad_kernel<false> : net_wgrad_kernel<false>);
  const size_t n = (size_t)cout * cin * NFEAT;
  net_wgrad_final_kernel<<<cdiv(n, 256), 256, 0, st>>>(grad, part, n, nchunk);
}

void launch_net_span_loss(cx<float>* gam, double* loss_agg, double* loss, const cx<float>* X, const cx<float>* T,
                          const Geom& g, int ntv, int* status, hipStream_t st) {
  const int nagg = 2 * g.nblocks;
  const double scale = 1.0 / ((double)nagg * ntv);
  if (ntv <= 16)
    net_span_loss_kernel<1><<<nagg, SLT, 0, st>>>(gam, loss_agg, X, T, g, ntv, scale, status);
  else
    net_span_loss_kernel<2><<<nagg, SLT, 0, st>>>(gam, loss_agg, X, T, g, ntv, scale, status);
  sum_kernel<<<1, 64, 0, st>>>(loss, loss_agg, nagg, scale);
}

void launch_adam(float* w, float* m, float* v, const float* grad, size_t n, float lr, int64_t step, hipStream_t st) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)step)));
  adam_kernel<<<cdiv(n, 256), 256, 0, st>>>(w, m, v, grad, n, lr, b1, b2, c1, c2, eps);
}

}  // namespace ddamg
