// SAP colour phase (Alg. 3, multiplicative Schwarz) on 4^4 blocks, the
// workload's blocks and half of its time.
//
// The residual is carried from phase to phase.  A phase that solves the
// blocks of one colour changes the other colour's residual only through the
// hops across the block faces, so it leaves, beside its own residual after
// the solve, the projected correction (1 -+ g_mu) e on its eight faces (6
// complex per face site), and the next phase subtracts U times that instead
// of forming y - D x anew.  Forming it took half of a phase (24 rhs on 16^4 in
// FP16: 104 of 205 us, the four MR steps the rest): eight hops and both
// clover blocks per site, with strided reads of the neighbours' faces.  Now
// eight compact face reads and two link products per lane do.  Only the
// first visit of a colour from a nonzero x forms y - D x; from x = 0 none.
//
// Two kernels share this.  sap4_site_kernel: one lane per site, four waves
// per block, the gauge field read from L2 in every MR step; four workgroups
// share a CU (two in FP64) and fill each other's waits.  sap4_lane_kernel
// (FP32 arithmetic): two lanes per site and the gauge field in registers, for
// grids that leave the CUs one workgroup each.
#include "dirac_device.h"
#include "sap_device.h"

namespace ddamg {

namespace {

using namespace dev;

constexpr int S4 = 256;    // sites of a block
constexpr int S4T = 512;   // lanes of a workgroup with two per site
constexpr int S4F = 64;    // sites of a face
static_assert(SAP4_FACE_ENTRIES == 8 * 6 * S4F, "face buffer of a block");

// local site of face site i on the layer of direction MU, and the inverse
template <int MU>
__device__ inline int face_l(int layer, int i) {
  if constexpr (MU == 0) return layer + 4 * i;
  if constexpr (MU == 1) return (i & 3) + 4 * layer + 16 * (i >> 2);
  if constexpr (MU == 2) return (i & 15) + 16 * layer + 64 * (i >> 4);
  return i + 64 * layer;
}
template <int MU>
__device__ inline int face_i(int l) {
  if constexpr (MU == 0) return l >> 2;
  if constexpr (MU == 1) return (l & 3) | ((l >> 4) << 2);
  if constexpr (MU == 2) return (l & 15) | ((l >> 6) << 4);
  return l & 63;
}
template <int MU>
__device__ inline int loc(int l) { return (l >> (2 * MU)) & 3; }
constexpr int lstride(int mu) { return mu == 0 ? 1 : mu == 1 ? 4 : mu == 2 ? 16 : 64; }

template <typename S>
__device__ inline cx<float> up(const stc_t<S>& v) {
  if constexpr (is_half<S>()) {
    const float2 f = __half22float2(v);
    return mk(f.x, f.y);
  } else {
    return v;
  }
}

// The links and the clover block of a lane in storage precision: U of its
// site on a lower lane, U^dag of the backward neighbour's on an upper one
template <typename S>
struct Gauge4 {
  stc_t<S> u[4][9];
  stc_t<S> a[CLOVER_PAIRS];
  float cu[4];  // -1/2 times the link's scale, 0 for a hop that leaves the block
  float ca;     // the clover block's scale
  // The values are the same in every MR step: hide that, or the compiler
  // keeps them converted to FP32 across the loop, twice the registers.
  __device__ void launder() {
    if constexpr (is_half<S>()) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int k = 0; k < 9; ++k) asm volatile("" : "+v"(*reinterpret_cast<unsigned*>(&u[m][k])));
#pragma unroll
      for (int k = 0; k < CLOVER_PAIRS; ++k) asm volatile("" : "+v"(*reinterpret_cast<unsigned*>(&a[k])));
    }
  }
};

// conj(v) on upper lanes (mask = the sign bit there, 0 on lower ones)
__device__ inline __half2 conj_if(__half2 v, unsigned mask) {
  unsigned u;
  __builtin_memcpy(&u, &v, 4);
  u ^= mask;
  __builtin_memcpy(&v, &u, 4);
  return v;
}
__device__ inline cx<float> conj_if(cx<float> v, unsigned mask) {
  v.i = __uint_as_float(__float_as_uint(v.i) ^ mask);
  return v;
}

template <int MU, typename S>
__device__ inline void load_u(Gauge4<S>& G, const GaugeView<S>& gv, int s, size_t V, bool upper) {
  stc_t<S> t[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) t[k] = elem(gv.U + (size_t)(MU * 9 + k) * V, (unsigned)s);
  const unsigned mask = upper ? 0x80000000u : 0u;
#pragma unroll
  for (int k = 0; k < 9; ++k) G.u[MU][k] = conj_if(upper ? t[3 * (k % 3) + k / 3] : t[k], mask);
  G.cu[MU] = -0.5f;
  if constexpr (is_half<S>()) G.cu[MU] *= elem(gv.Usc, (unsigned)s);
}

// out = U h for a link as held by the lane
template <typename S>
__device__ inline void mul_link(Half2<float>& o, const stc_t<S> u[9], const Half2<float>& h) {
#pragma unroll
  for (int sp = 0; sp < 2; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<float> t = mk(0.f, 0.f);
#pragma unroll
      for (int b = 0; b < 3; ++b) t = cfma(up<S>(u[3 * a + b]), h.h[sp][b], t);
      o.h[sp][a] = t;
    }
}

// one component of a -+ X_mu b on the way to the projection and of the
// reconstruction X_mu^dag: see project and reconstruct in dirac_device.h,
// whose forward forms these are for sg = 1, the backward ones for sg = -1
template <int MU>
__device__ inline void project_sg(Half2<float>& o, const cx<float> p[4][3], float sg) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cx<float> d0, d1;
    if constexpr (MU == 0) {
      d0 = times_i(p[3][c]);
      d1 = times_i(p[2][c]);
    } else if constexpr (MU == 1) {
      d0 = p[3][c];
      d1 = neg(p[2][c]);
    } else if constexpr (MU == 2) {
      d0 = times_i(p[2][c]);
      d1 = times_mi(p[3][c]);
    } else {
      d0 = p[2][c];
      d1 = p[3][c];
    }
    o.h[0][c] = mk(fmaf(sg, d0.r, p[0][c].r), fmaf(sg, d0.i, p[0][c].i));
    o.h[1][c] = mk(fmaf(sg, d1.r, p[1][c].r), fmaf(sg, d1.i, p[1][c].i));
  }
}
// X_mu^dag h, the lower spins of the backward hop
template <int MU, typename T>
__device__ inline void lower(cx<T>& l0, cx<T>& l1, cx<T> h0, cx<T> h1) {
  if constexpr (MU == 0) {
    l0 = times_i(h1);
    l1 = times_i(h0);
  } else if constexpr (MU == 1) {
    l0 = h1;
    l1 = neg(h0);
  } else if constexpr (MU == 2) {
    l0 = times_i(h0);
    l1 = times_mi(h1);
  } else {
    l0 = neg(h0);
    l1 = neg(h1);
  }
}
__device__ inline cx<float> axpy(float c, cx<float> x, cx<float> y) { return mk(fmaf(c, x.r, y.r), fmaf(c, x.i, y.i)); }

// acc += cu times the hop of direction MU from the 12 components in q
template <int MU, typename S>
__device__ inline void hop4(cx<float> acc[4][3], const cx<float> q[4][3], const stc_t<S> link[9], float cu, float sg) {
  Half2<float> h, u;
  project_sg<MU>(h, q, sg);
  mul_link<S>(u, link, h);
  const float cd = -sg * cu;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cx<float> l0, l1;
    lower<MU>(l0, l1, u.h[0][c], u.h[1][c]);
    acc[0][c] = axpy(cu, u.h[0][c], acc[0][c]);
    acc[1][c] = axpy(cu, u.h[1][c], acc[1][c]);
    acc[2][c] = axpy(cd, l0, acc[2][c]);
    acc[3][c] = axpy(cd, l1, acc[3][c]);
  }
}

template <typename T>
__device__ inline void read12(cx<T> q[4][3], const cx<T>* lds, int l) {
#pragma unroll
  for (int k = 0; k < 12; ++k) q[k / 3][k % 3] = lds[k * S4 + l];
}

// clover block of the lane's chirality times its six components
template <typename S>
__device__ inline void clover4(cx<float> o[6], const cx<float> p[6], const Gauge4<S>& G) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const cx<float> d = up<S>(G.a[k]);
    o[2 * k] = d.r * p[2 * k];
    o[2 * k + 1] = d.i * p[2 * k + 1];
  }
  int q = 3;
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = i + 1; j < 6; ++j) {
      const cx<float> a = up<S>(G.a[q]);
      o[i] = cfma(a, p[j], o[i]);
      o[j] = cfmac(a, p[i], o[j]);
      ++q;
    }
}

// q = the lane's half of acc, both lanes of the site added, plus ca times o:
// the lower halves' lower spins trade places with the upper halves' upper ones
__device__ inline void meet(cx<float> q[6], const cx<float> acc[4][3], const cx<float> o[6], float ca) {
  auto trade = [](float& x, float& y) {  // lanes 32..63 of x <-> lanes 0..31 of y
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(t[0]);
    y = __uint_as_float(t[1]);
  };
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    cx<float> u = acc[k / 3][k % 3], d = acc[2 + k / 3][k % 3];
    trade(u.r, d.r);
    trade(u.i, d.i);
    q[k] = axpy(ca, o[k], u + d);
  }
}

// neighbour block of block coordinates bc in direction mu
__device__ inline int nbr_block(const Geom& g, const int bc[4], int mu, bool fwd) {
  int c[4] = {bc[0], bc[1], bc[2], bc[3]};
  if (fwd)
    c[mu] = c[mu] + 1 == g.NB[mu] ? 0 : c[mu] + 1;
  else
    c[mu] = c[mu] == 0 ? g.NB[mu] - 1 : c[mu] - 1;
  return block_to_int(g, c);
}

// ---- residual from the previous one: one wave per face f = MU (forward) or
// 4 + MU multiplies the neighbour block's face with the link ...
template <int MU, bool FWD, typename T, typename S>
__device__ inline void face_in(cx<T>* halo, const cx<T>* faces, const GaugeView<S>& gv, const Geom& g,
                               const int bc[4], int ci, int i) {
  constexpr int f = FWD ? MU : 4 + MU;
  const int nb = nbr_block(g, bc, MU, FWD);
  const cx<T>* fp = faces + (size_t)nb * SAP4_FACE_ENTRIES + f * 6 * S4F;
  Half2<T> h;
#pragma unroll
  for (int k = 0; k < 6; ++k) h.h[k / 3][k % 3] = elem(fp + k * S4F, (unsigned)i);
  // the link leaves the block forward (own site) or enters it from the neighbour's last layer
  const int s = (FWD ? ci : nb) * S4 + face_l<MU>(3, i);
  cx<T> U[3][3];
  load_link<T, S>(U, gv, MU, s, (size_t)g.V);
  T c = (T)-0.5;
  if constexpr (is_half<S>()) c *= (T)elem(gv.Usc, (unsigned)s);
  if (MU == 3 && bc[3] == (FWD ? g.NB[3] - 1 : 0)) c = -c;
#pragma unroll
  for (int sp = 0; sp < 2; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<T> t = mk((T)0, (T)0);
#pragma unroll
      for (int b = 0; b < 3; ++b) t = FWD ? cfma(U[a][b], h.h[sp][b], t) : cfmac(U[b][a], h.h[sp][b], t);
      halo[(f * 6 + 3 * sp + a) * S4F + i] = c * t;
    }
}
// ... and every site subtracts the reconstruction for the (at most one) face
// of direction MU that it lies on
template <int MU, typename T>
__device__ inline void face_add(cx<T> rho[4][3], const cx<T>* halo, int l) {
  const int c = loc<MU>(l);
  if (c != 0 && c != 3) return;
  const cx<T>* hp = halo + (c == 3 ? MU : 4 + MU) * 6 * S4F + face_i<MU>(l);
  const T sl = c == 3 ? (T)1 : (T)-1;  // lower spins: -X^dag (forward hop) or X^dag (backward), subtracted
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const cx<T> h0 = hp[q * S4F], h1 = hp[(3 + q) * S4F];
    cx<T> l0, l1;
    lower<MU>(l0, l1, h0, h1);
    rho[0][q] = rho[0][q] - h0;
    rho[1][q] = rho[1][q] - h1;
    rho[2][q] = rho[2][q] + sl * l0;
    rho[3][q] = rho[3][q] + sl * l1;
  }
}
// the same for a lane that holds the upper or the lower two spins
template <int MU>
__device__ inline void face_add_half(cx<float> rho[6], const cx<float>* halo, int l, bool upper) {
  const int c = loc<MU>(l);
  if (c != 0 && c != 3) return;
  const cx<float>* hp = halo + (c == 3 ? MU : 4 + MU) * 6 * S4F + face_i<MU>(l);
  const float sl = c == 3 ? 1.f : -1.f;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const cx<float> h0 = hp[q * S4F], h1 = hp[(3 + q) * S4F];
    cx<float> l0, l1;
    lower<MU>(l0, l1, h0, h1);
    rho[q] = axpy(upper ? sl : -1.f, upper ? l0 : h0, rho[q]);
    rho[3 + q] = axpy(upper ? sl : -1.f, upper ? l1 : h1, rho[3 + q]);
  }
}

// the projected correction on face MU: low layer for the neighbour's forward
// hop, high layer for its backward hop
template <int MU, bool FWD, typename T>
__device__ inline void face_out(cx<T>* faces, const cx<T>* lds, int ci, int i) {
  constexpr int f = FWD ? MU : 4 + MU;
  cx<T> q[4][3];
  read12(q, lds, face_l<MU>(FWD ? 0 : 3, i));
  Half2<T> h;
  project<MU, FWD, T>(h, q);
  cx<T>* fp = faces + (size_t)ci * SAP4_FACE_ENTRIES + f * 6 * S4F;
#pragma unroll
  for (int k = 0; k < 6; ++k) fp[k * S4F + i] = h.h[k / 3][k % 3];
}

// a lane's hop of direction MU: whether it stays in the block, and the
// internal site it comes from
template <int MU>
__device__ inline bool stays(int l, bool upper) { return upper ? loc<MU>(l) > 0 : loc<MU>(l) < 3; }
template <int MU>
__device__ inline int hop_site(const Geom& g, const int bc[4], int ci, int l, bool upper) {
  if (stays<MU>(l, upper)) return ci * S4 + (upper ? l - lstride(MU) : l + lstride(MU));
  return nbr_block(g, bc, MU, !upper) * S4 + (upper ? l + 3 * lstride(MU) : l - 3 * lstride(MU));
}

// hop of the full operator: across a face the neighbour block's x from memory
template <int MU, typename S>
__device__ inline void hop_full(cx<float> acc[4][3], const cx<float>* lds, const cx<float>* x, int ci, int l,
                                bool upper, const Geom& g, const int bc[4], const Gauge4<S>& G, float sg) {
  const bool live = g.V > 0;  // opaque: each hop keeps its loads with its arithmetic
  if (live) {
    cx<float> q[4][3];
    float cu = G.cu[MU];
    if (stays<MU>(l, upper)) {
      read12(q, lds, upper ? l - lstride(MU) : l + lstride(MU));
    } else {
      const int s = hop_site<MU>(g, bc, ci, l, upper);
#pragma unroll
      for (int k = 0; k < 12; ++k) q[k / 3][k % 3] = elem(x + (size_t)k * (size_t)g.V, (unsigned)s);
      if (MU == 3 && bc[3] == (upper ? 0 : g.NB[3] - 1)) cu = -cu;
    }
    hop4<MU, S>(acc, q, G.u[MU], cu, sg);
  }
  asm volatile("" ::: "memory");
}

// Two lanes per site, 32 apart in one wave, eight waves per block: the lower
// lane applies the four forward hops and keeps the upper two spins (chirality
// 0) of the residual, the correction and B times the residual, the upper lane
// the backward hops and the lower two spins.  The roles differ in data only
// (the upper lane's links are U^dag, its projection sign is the opposite), and
// the halves of a product meet by swapping the two halves of the wave.  So a
// lane needs four links and one chirality's clover block, and holds them in
// registers (108 values: FP32 108 registers, FP16 54) for the whole phase: the
// MR steps read nothing but LDS.  Where a CU has one workgroup there is no
// other to fill the round trips to L2 of the kernel below, nine per MR step.
// An MR step alone on a CU: 2.4 us in FP32 (issue-bound: 720 instructions,
// two waves per SIMD) against 4.9, 3.2 in FP16.  A phase of 8^4, one rhs: 32.2
// -> 20.8 us; of 16^3x32, one rhs, FP16 (256 workgroups): 39.1 -> 27.4 us.
template <typename S>
__global__ __launch_bounds__(S4T, 2) void sap4_lane_kernel(Sap4Args<float, S> a) {
  __shared__ cx<float> lds[12 * S4];  // the block's field under work; the neighbours' faces [8][6][64] before it
  __shared__ float red[S4T / 64][4];
  const Geom& g = a.g;
  const size_t V = g.V;
  // the rhs of a block side by side on one XCD: they read the same links
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = a.colour * g.neven + wl / a.nrhs, r = wl % a.nrhs;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = threadIdx.x & 63;
  const bool upper = i >= 32;
  const int l = 32 * w + (i & 31), s = ci * S4 + l;
  const int own = upper ? 6 : 0;  // first of the lane's six components
  const float sg = upper ? -1.f : 1.f;
  int bc[4];
  int_block_coords(g, ci, bc);
  cx<float>* x = a.x + (size_t)r * 12 * V;
  const cx<float>* src = a.src + (size_t)r * 12 * V;
  cx<float>* rs = a.r + (size_t)r * 12 * V;
  cx<float>* faces = a.faces + (size_t)r * g.nblocks * SAP4_FACE_ENTRIES;
  cx<float> rho[6], e[6];
  Gauge4<S> G;
  // the lane's gauge field
  load_u<0, S>(G, a.gv, upper ? hop_site<0>(g, bc, ci, l, true) : s, V, upper);
  load_u<1, S>(G, a.gv, upper ? hop_site<1>(g, bc, ci, l, true) : s, V, upper);
  load_u<2, S>(G, a.gv, upper ? hop_site<2>(g, bc, ci, l, true) : s, V, upper);
  load_u<3, S>(G, a.gv, upper ? hop_site<3>(g, bc, ci, l, true) : s, V, upper);
  const stc_t<S>* A = a.gv.A + (size_t)(upper ? CLOVER_PAIRS : 0) * V + s;
#pragma unroll
  for (int k = 0; k < CLOVER_PAIRS; ++k) G.a[k] = A[(size_t)k * V];
  G.ca = 1.f;
  if constexpr (is_half<S>()) G.ca = elem(a.gv.Asc, (unsigned)s);
#pragma unroll
  for (int k = 0; k < 6; ++k) rho[k] = src[(size_t)(own + k) * V + s];
  if (a.mode == SAP4_FULL) {
    cx<float> p[6], o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      p[k] = x[(size_t)(own + k) * V + s];
      lds[(own + k) * S4 + l] = p[k];
    }
    __syncthreads();
    cx<float> acc[4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k / 3][k % 3] = mk(0.f, 0.f);
    clover4<S>(o, p, G);
    hop_full<0, S>(acc, lds, x, ci, l, upper, g, bc, G, sg);
    hop_full<1, S>(acc, lds, x, ci, l, upper, g, bc, G, sg);
    hop_full<2, S>(acc, lds, x, ci, l, upper, g, bc, G, sg);
    hop_full<3, S>(acc, lds, x, ci, l, upper, g, bc, G, sg);
    meet(p, acc, o, G.ca);
#pragma unroll
    for (int k = 0; k < 6; ++k) rho[k] = rho[k] - p[k];
    __syncthreads();  // lds is written again
  } else if (a.mode == SAP4_FACES) {
    switch (w) {
      case 0: face_in<0, true, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 1: face_in<1, true, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 2: face_in<2, true, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 3: face_in<3, true, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 4: face_in<0, false, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 5: face_in<1, false, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      case 6: face_in<2, false, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
      default: face_in<3, false, float, S>(lds, faces, a.gv, g, bc, ci, i); break;
    }
    __syncthreads();
    face_add_half<0>(rho, lds, l, upper);
    face_add_half<1>(rho, lds, l, upper);
    face_add_half<2>(rho, lds, l, upper);
    face_add_half<3>(rho, lds, l, upper);
    __syncthreads();  // lds is written again
  }
  // from here on the hops stay in the block: the others get the factor 0
  // instead of a branch, so that the reads of one hop overlap the products of
  // the one before (their lanes would idle either way)
  int ln[4];
  auto inside = [&](auto mu) {
    constexpr int MU = decltype(mu)::value;
    if (!stays<MU>(l, upper)) G.cu[MU] = 0.f;
    ln[MU] = (l + (upper ? -lstride(MU) : lstride(MU))) & (S4 - 1);
  };
  inside(std::integral_constant<int, 0>());
  inside(std::integral_constant<int, 1>());
  inside(std::integral_constant<int, 2>());
  inside(std::integral_constant<int, 3>());
#pragma unroll
  for (int k = 0; k < 6; ++k) e[k] = mk(0.f, 0.f);
  for (int it = 0; it < a.n_mr; ++it) {
    G.launder();
#pragma unroll
    for (int k = 0; k < 6; ++k) lds[(own + k) * S4 + l] = rho[k];
    __syncthreads();
    cx<float> acc[4][3], q[6], p[4][3], o[6];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k / 3][k % 3] = mk(0.f, 0.f);
    read12(p, lds, ln[0]);
    clover4<S>(o, rho, G);
    hop4<0, S>(acc, p, G.u[0], G.cu[0], sg);
    read12(p, lds, ln[1]);
    hop4<1, S>(acc, p, G.u[1], G.cu[1], sg);
    read12(p, lds, ln[2]);
    hop4<2, S>(acc, p, G.u[2], G.cu[2], sg);
    read12(p, lds, ln[3]);
    hop4<3, S>(acc, p, G.u[3], G.cu[3], sg);
    meet(q, acc, o, G.ca);
    float d0 = 0.f, d1 = 0.f, d2 = 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      d0 = fmaf(q[k].r, rho[k].r, fmaf(q[k].i, rho[k].i, d0));
      d1 = fmaf(q[k].r, rho[k].i, fmaf(-q[k].i, rho[k].r, d1));
      d2 = fmaf(q[k].r, q[k].r, fmaf(q[k].i, q[k].i, d2));
    }
    d0 = wave_sum63(d0);
    d1 = wave_sum63(d1);
    d2 = wave_sum63(d2);
    if (i == 63) {
      red[w][0] = d0;
      red[w][1] = d1;
      red[w][2] = d2;
    }
    __syncthreads();  // the sums are there, and every neighbour has been read
    float a_re = 0.f, a_im = 0.f, n2 = 0.f;
#pragma unroll
    for (int k = 0; k < S4T / 64; ++k) {
      a_re += red[k][0];
      a_im += red[k][1];
      n2 += red[k][2];
    }
    const float inv = n2 > 0.f ? 1.f / n2 : 0.f;
    const cx<float> alpha = mk(a_re * inv, a_im * inv);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      e[k] = cfma(alpha, rho[k], e[k]);
      rho[k] = cfma(neg(alpha), q[k], rho[k]);
    }
  }
  // x += e (x = e from a zero start), the residual, the faces of e
  x += (size_t)own * V + s;
  if (a.x_zero) {
#pragma unroll
    for (int k = 0; k < 6; ++k) x[(size_t)k * V] = e[k];
  } else {
#pragma unroll
    for (int k = 0; k < 6; ++k) x[(size_t)k * V] = x[(size_t)k * V] + e[k];
  }
  if (a.store_r) {
#pragma unroll
    for (int k = 0; k < 6; ++k) rs[(size_t)(own + k) * V + s] = rho[k];
  }
  if (a.store_faces) {
#pragma unroll
    for (int k = 0; k < 6; ++k) lds[(own + k) * S4 + l] = e[k];
    __syncthreads();
    switch (w) {
      case 0: face_out<0, true, float>(faces, lds, ci, i); break;
      case 1: face_out<1, true, float>(faces, lds, ci, i); break;
      case 2: face_out<2, true, float>(faces, lds, ci, i); break;
      case 3: face_out<3, true, float>(faces, lds, ci, i); break;
      case 4: face_out<0, false, float>(faces, lds, ci, i); break;
      case 5: face_out<1, false, float>(faces, lds, ci, i); break;
      case 6: face_out<2, false, float>(faces, lds, ci, i); break;
      default: face_out<3, false, float>(faces, lds, ci, i); break;
    }
  }
}

// One lane per site, four waves per block.  Bound: vector-ALU issue (83 % of
// the SIMD cycles; 6.7 k instructions per wave and phase, 7.7 k with the full
// residual each time).  24^3x48, FP16, 12 and 24 rhs: 1535 -> 1391 us per
// phase; 16^4, FP32, 8 rhs 96 -> 86 us; FP64, 4 rhs 77 -> 71 us.
template <typename T, typename S>
__global__ __launch_bounds__(S4, sizeof(T) == 8 ? 2 : 4) void sap4_site_kernel(Sap4Args<T, S> a) {
  __shared__ cx<T> lds[12 * S4];  // the block's field under work; the neighbours' faces [8][6][64] before it
  __shared__ T red[S4 / 64][3];
  const Geom& g = a.g;
  const size_t V = g.V;
  // the rhs of a block side by side on one XCD: they read the same links
  const int wl = xcd_swizzle(blockIdx.x, gridDim.x);
  const int ci = a.colour * g.neven + wl / a.nrhs, r = wl % a.nrhs;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = threadIdx.x & 63, l = threadIdx.x, s = ci * S4 + l;
  const SitePos pos = site_pos(g, s);
  cx<T>* x = a.x + (size_t)r * 12 * V;
  const cx<T>* src = a.src + (size_t)r * 12 * V;
  cx<T>* rs = a.r + (size_t)r * 12 * V;
  cx<T>* faces = a.faces + (size_t)r * g.nblocks * SAP4_FACE_ENTRIES;
  GaugeLd<S, true> gl(a.gv, V);
  cx<T> rho[1][4][3], e[1][4][3];
  if (a.mode == SAP4_FULL) {
    // the block's x in LDS for the in-block hops, the halo (not written in this phase) from memory
#pragma unroll
    for (int k = 0; k < 12; ++k) lds[k * S4 + l] = elem(x + (size_t)k * V, (unsigned)s);
    __syncthreads();
    cx<T> acc[1][4][3], p[1][4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      acc[0][k / 3][k % 3] = mk((T)0, (T)0);
      p[0][k / 3][k % 3] = lds[k * S4 + l];
    }
    sap_clover<1, T, S>(acc, p, gl, s);
    staged_hops<0, 1, 4, T, S>(acc, lds, x, 0, 1, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<1, 1, 4, T, S>(acc, lds, x, 0, 1, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<2, 1, 4, T, S>(acc, lds, x, 0, 1, pos, g, gl, V);
    asm volatile("" ::: "memory");
    staged_hops<3, 1, 4, T, S>(acc, lds, x, 0, 1, pos, g, gl, V);
#pragma unroll
    for (int k = 0; k < 12; ++k)
      rho[0][k / 3][k % 3] = elem(src + (size_t)k * V, (unsigned)s) - acc[0][k / 3][k % 3];
    __syncthreads();  // lds is written again
  } else {
    if (a.mode == SAP4_FACES) {
      switch (w) {
        case 0:
          face_in<0, true, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          face_in<0, false, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          break;
        case 1:
          face_in<1, true, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          face_in<1, false, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          break;
        case 2:
          face_in<2, true, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          face_in<2, false, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          break;
        default:
          face_in<3, true, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          face_in<3, false, T, S>(lds, faces, a.gv, g, pos.bc, ci, i);
          break;
      }
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) rho[0][k / 3][k % 3] = elem(src + (size_t)k * V, (unsigned)s);
    if (a.mode == SAP4_FACES) {
      __syncthreads();
      face_add<0, T>(rho[0], lds, l);
      face_add<1, T>(rho[0], lds, l);
      face_add<2, T>(rho[0], lds, l);
      face_add<3, T>(rho[0], lds, l);
      __syncthreads();  // lds is written again
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) e[0][k / 3][k % 3] = mk((T)0, (T)0);
  for (int it = 0; it < a.n_mr; ++it) {
    // Launder the gauge loader: the loads of B below are the same in every
    // MR step, and hoisting them out of the loop would pin them in registers
    // for the whole kernel.
    auto gli = gl;
    gli.launder();
#pragma unroll
    for (int k = 0; k < 12; ++k) lds[k * S4 + l] = rho[0][k / 3][k % 3];
    __syncthreads();
    cx<T> q[1][4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) q[0][k / 3][k % 3] = mk((T)0, (T)0);
    sap_clover<1, T, S>(q, rho, gli, s);
    block_hops<0, 1, 4, T, S>(q, lds, pos, g, gli);
    block_hops<1, 1, 4, T, S>(q, lds, pos, g, gli);
    block_hops<2, 1, 4, T, S>(q, lds, pos, g, gli);
    block_hops<3, 1, 4, T, S>(q, lds, pos, g, gli);
    T dots[3] = {(T)0, (T)0, (T)0};
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const cx<T> qk = q[0][k / 3][k % 3], t = cmulc(qk, rho[0][k / 3][k % 3]);
      dots[0] += t.r;
      dots[1] += t.i;
      dots[2] += qk.r * qk.r + qk.i * qk.i;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T v = wave_sum63(dots[c]);
      if (i == 63) red[w][c] = v;
    }
    __syncthreads();  // the sums are there, and every neighbour has been read
    T a_re = 0, a_im = 0, n2 = 0;
#pragma unroll
    for (int k = 0; k < S4 / 64; ++k) {
      a_re += red[k][0];
      a_im += red[k][1];
      n2 += red[k][2];
    }
    const T inv = n2 > (T)0 ? (T)1 / n2 : (T)0;
    const cx<T> alpha = mk(a_re * inv, a_im * inv);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      e[0][k / 3][k % 3] = e[0][k / 3][k % 3] + alpha * rho[0][k / 3][k % 3];
      rho[0][k / 3][k % 3] = rho[0][k / 3][k % 3] - alpha * q[0][k / 3][k % 3];
    }
  }
  // x += e (x = e from a zero start), the residual, the faces of e
  if (a.x_zero) {
#pragma unroll
    for (int k = 0; k < 12; ++k) x[(size_t)k * V + s] = e[0][k / 3][k % 3];
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const size_t at = (size_t)k * V + s;
      x[at] = x[at] + e[0][k / 3][k % 3];
    }
  }
  if (a.store_r) {
#pragma unroll
    for (int k = 0; k < 12; ++k) rs[(size_t)k * V + s] = rho[0][k / 3][k % 3];
  }
  if (a.store_faces) {
#pragma unroll
    for (int k = 0; k < 12; ++k) lds[k * S4 + l] = e[0][k / 3][k % 3];
    __syncthreads();
    switch (w) {
      case 0:
        face_out<0, true, T>(faces, lds, ci, i);
        face_out<0, false, T>(faces, lds, ci, i);
        break;
      case 1:
        face_out<1, true, T>(faces, lds, ci, i);
        face_out<1, false, T>(faces, lds, ci, i);
        break;
      case 2:
        face_out<2, true, T>(faces, lds, ci, i);
        face_out<2, false, T>(faces, lds, ci, i);
        break;
      default:
        face_out<3, true, T>(faces, lds, ci, i);
        face_out<3, false, T>(faces, lds, ci, i);
        break;
    }
  }
}

}  // namespace

// 4^4 blocks whose gauge planes the buffer descriptors cover (9 link planes of
// a direction, 18 clover planes of a chirality below 2^31 bytes each)
template <typename S>
bool sap4_applies(const Geom& g) {
  return g.bs[0] == 4 && g.bs[1] == 4 && g.bs[2] == 4 && g.bs[3] == 4 &&
         (double)CLOVER_PAIRS * (double)g.V * sizeof(stc_t<S>) < 2147483648.0;
}

// Two lanes per site up to one workgroup per CU: 256 of them take 27.7 us in
// FP32 and FP16 against 41 and 39 us of the one-lane kernel (with the full
// residual), 512 take 51.2 and 51.4 us, two rounds, against 51.3 and 47.3 us.
constexpr int SAP4_LANE_MAX_GROUPS = 256;

template <typename T, typename S>
void launch_sap4(const Sap4Args<T, S>& a, hipStream_t st) {
  if (a.nrhs <= 0) return;
  const unsigned groups = (unsigned)(a.g.nblocks / 2) * (unsigned)a.nrhs;
  if constexpr (sizeof(T) == 4) {
    if (groups <= SAP4_LANE_MAX_GROUPS) {
      sap4_lane_kernel<S><<<groups, S4T, 0, st>>>(a);
      return;
    }
  }
  sap4_site_kernel<T, S><<<groups, S4, 0, st>>>(a);
}
#define INST(T, S)                            \
  template bool sap4_applies<S>(const Geom&); \
  template void launch_sap4<T, S>(const Sap4Args<T, S>&, hipStream_t);
INST(double, double)
INST(float, float)
INST(float, __half)
#undef INST

}  // namespace ddamg
