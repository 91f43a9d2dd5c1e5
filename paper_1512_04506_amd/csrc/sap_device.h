// Shared by the smoother's kernels: wave reductions, gauge-field loads and the
// hops of a block.
#pragma once
#include "dirac_device.h"

namespace ddamg {
namespace dev {

// Sum over the 64 lanes of a wave by DPP lane moves (no LDS round trips):
// quad sums, then row sums (lanes 15, 31, 47, 63), then the row broadcasts;
// lane 63 ends with the total.
template <int CTRL, int ROWS>
__device__ inline float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, true));
}
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename T>
__device__ inline T wave_sum63(T v) {
  v += dpp_move<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
  v += dpp_move<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0x114, 0xF>(v);  // row_shr:4
  v += dpp_move<0x118, 0xF>(v);  // row_shr:8
  v += dpp_move<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Gauge-field loads of the smoother.  GaugeLd<S, false> reads the planes
// with global loads (a 64-bit address per load and lane); GaugeLd<S, true>
// reads them with buffer loads, one descriptor per link direction and per
// clover chirality, the plane's offset in a scalar register and the site's
// byte offset shared by all loads of a site: no vector instruction per load
// for its address.  A descriptor covers at most 2^31 bytes (checked by the
// launcher) and returns zeros beyond its range instead of faulting.
template <typename S, bool BUF>
struct GaugeLd;

template <typename S>
struct GaugeLd<S, false> {
  GaugeView<S> gv;
  size_t V;
  __device__ GaugeLd(const GaugeView<S>& g, size_t v) : gv(g), V(v) {}
  __device__ void launder() {
    int zero = 0;
    asm volatile("" : "+s"(zero));
    gv.U += zero;
    gv.A += zero;
  }
  template <int MU, typename Tc>
  __device__ void link(cx<Tc> u[3][3], int s) const {
    load_link<Tc, S>(u, gv, MU, s, V);
  }
  template <typename Tc>
  __device__ void clover(cx<Tc> a[CLOVER_PAIRS], int h, int s) const {
    const stc_t<S>* Ah = gv.A + (size_t)h * CLOVER_PAIRS * V;
#pragma unroll
    for (int e = 0; e < CLOVER_PAIRS; ++e) a[e] = ldc<Tc>(Ah + (size_t)e * V, (unsigned)s);
  }
  __device__ float link_scale(int s) const { return gv.Usc[s]; }
  __device__ float clover_scale(int s) const { return gv.Asc[s]; }
};

constexpr int BUF_WORD3 = 0x00020000;  // CDNA buffer descriptor word 3: 32-bit dword format

template <typename X>
__device__ inline X buf_ld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
  X x;
  if constexpr (sizeof(X) == 4) {
    const unsigned v = __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0);
    __builtin_memcpy(&x, &v, 4);
  } else if constexpr (sizeof(X) == 8) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
    __builtin_memcpy(&x, &v, 8);
  } else {
    static_assert(sizeof(X) == 16, "complex entry of 4, 8 or 16 bytes");
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0);
    __builtin_memcpy(&x, &v, 16);
  }
  return x;
}

template <typename Tc, typename X>
__device__ inline cx<Tc> to_cx(const X& v) {
  if constexpr (std::is_same<X, __half2>::value) {
    const float2 f = __half22float2(v);
    return mk((Tc)f.x, (Tc)f.y);
  } else {
    return mk((Tc)v.r, (Tc)v.i);
  }
}

template <typename S>
struct GaugeLd<S, true> {
  using E = stc_t<S>;
  __amdgpu_buffer_rsrc_t U[4], A[2];
  const float* Usc;
  const float* Asc;
  unsigned plane;  // bytes of one component plane, V entries
  __device__ GaugeLd(const GaugeView<S>& g, size_t V) : Usc(g.Usc), Asc(g.Asc), plane((unsigned)(V * sizeof(E))) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
      U[mu] = __builtin_amdgcn_make_buffer_rsrc((void*)(g.U + (size_t)mu * 9 * V), (short)0, (int)(9 * plane),
                                                BUF_WORD3);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      A[h] = __builtin_amdgcn_make_buffer_rsrc((void*)(g.A + (size_t)h * CLOVER_PAIRS * V), (short)0,
                                               (int)(CLOVER_PAIRS * plane), BUF_WORD3);
  }
  __device__ void launder() { asm volatile("" : "+s"(plane)); }
  template <int MU, typename Tc>
  __device__ void link(cx<Tc> u[3][3], int s) const {
    const unsigned vo = (unsigned)s * (unsigned)sizeof(E);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) u[a][b] = to_cx<Tc>(buf_ld<E>(U[MU], vo, (unsigned)(3 * a + b) * plane));
  }
  template <typename Tc>
  __device__ void clover(cx<Tc> a[CLOVER_PAIRS], int h, int s) const {
    const unsigned vo = (unsigned)s * (unsigned)sizeof(E);
#pragma unroll
    for (int e = 0; e < CLOVER_PAIRS; ++e) a[e] = to_cx<Tc>(buf_ld<E>(h ? A[1] : A[0], vo, (unsigned)e * plane));
  }
  __device__ float link_scale(int s) const { return elem(Usc, (unsigned)s); }
  __device__ float clover_scale(int s) const { return elem(Asc, (unsigned)s); }
};

// Block shape: B4 > 0 is a block of B4^4 sites known at compile time (LDS
// offsets of the neighbours become instruction immediates), B4 = 0 the
// shape of the geometry.
template <int B4>
struct Blk {
  __device__ static int vb(const Geom& g) {
    if constexpr (B4 > 0) return B4 * B4 * B4 * B4;
    else return g.vblock;
  }
  template <int MU>
  __device__ static int bs(const Geom& g) {
    if constexpr (B4 > 0) return B4;
    else return g.bs[MU];
  }
  template <int MU>
  __device__ static int lstr(const Geom& g) {
    if constexpr (B4 > 0) return MU == 0 ? 1 : MU == 1 ? B4 : MU == 2 ? B4 * B4 : B4 * B4 * B4;
    else return g.lstr[MU];
  }
};

// hop of direction MU (forward or backward) for NR spinors, link at slink
template <int MU, bool FWD, int NR, typename T, typename S, typename GL>
__device__ inline void sap_hop(cx<T> acc[NR][4][3], const cx<T> q[NR][4][3], const GL& gl, int slink) {
  cx<T> U[3][3];
  gl.template link<MU, T>(U, slink);
  T coef = (T)-0.5;
  if constexpr (is_half<S>()) coef *= (T)gl.link_scale(slink);
  hop_spinor_multi_u<MU, FWD, NR, T>(acc, q, U, coef);
}

// acc[r] += A(s) p[r] for NR spinors
template <int NR, typename T, typename S, typename GL>
__device__ inline void sap_clover(cx<T> acc[NR][4][3], const cx<T> p[NR][4][3], const GL& gl, int s) {
  T sc = (T)1;
  if constexpr (is_half<S>()) sc = (T)gl.clover_scale(s);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    cx<T> a[CLOVER_PAIRS];
    gl.template clover<T>(a, h, s);
    clover_half_multi<NR, T>(acc, p, a, h, sc);
  }
}

// in-block hops of direction MU for NR residual vectors from LDS
template <int MU, int NR, int B4, typename T, typename S, typename GL>
__device__ inline void block_hops(cx<T> acc[NR][4][3], const cx<T>* lds, const SitePos& p, const Geom& g,
                                  const GL& gl) {
  const int vb = Blk<B4>::vb(g);
  const int ls = Blk<B4>::template lstr<MU>(g);
  cx<T> q[NR][4][3];
  if (p.lc[MU] < Blk<B4>::template bs<MU>(g) - 1) {
    const int ln = p.l + ls;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k) q[r][sp][k] = lds[(r * 12 + 3 * sp + k) * vb + ln];
    sap_hop<MU, true, NR, T, S>(acc, q, gl, p.S);
  }
  if (p.lc[MU] > 0) {
    const int ln = p.l - ls;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int k = 0; k < 3; ++k) q[r][sp][k] = lds[(r * 12 + 3 * sp + k) * vb + ln];
    sap_hop<MU, false, NR, T, S>(acc, q, gl, p.S - ls);
  }
}

// hops of the full operator for NR vectors whose in-block values are staged
// in LDS: a neighbour inside the block is read there, one across the face
// from global memory (the other colour's blocks, not written in this phase)
template <int MU, int NR, int B4, typename T, typename S, typename GL>
__device__ inline void staged_hops(cx<T> acc[NR][4][3], const cx<T>* lds, const cx<T>* x, size_t rs, int nr,
                                   const SitePos& p, const Geom& g, const GL& gl, size_t V) {
  const int vb = Blk<B4>::vb(g);
  const int ls = Blk<B4>::template lstr<MU>(g);
  const bool live = g.V > 0;  // opaque: keeps each hop's loads with its arithmetic
  cx<T> q[NR][4][3];
  if (live) {
    const bool inside = p.lc[MU] < Blk<B4>::template bs<MU>(g) - 1;
    if (inside) {
      const int ln = p.l + ls;
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int k = 0; k < 3; ++k) q[r][sp][k] = lds[(r * 12 + 3 * sp + k) * vb + ln];
    } else {
      const int sn = nbr_fwd(g, p, MU);
      const bool wrap = MU == 3 && p.bc[3] == g.NB[3] - 1;
#pragma unroll
      for (int r = 0; r < NR; ++r)
        load_spinor(q[r], x + (size_t)min(r, nr - 1) * rs, sn, V, wrap ? (T)-1 : (T)1);
    }
    sap_hop<MU, true, NR, T, S>(acc, q, gl, p.S);
  }
  asm volatile("" ::: "memory");
  if (live) {
    const bool inside = p.lc[MU] > 0;
    const int sb = nbr_bwd(g, p, MU);
    if (inside) {
      const int ln = p.l - ls;
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int k = 0; k < 3; ++k) q[r][sp][k] = lds[(r * 12 + 3 * sp + k) * vb + ln];
    } else {
      const bool wrap = MU == 3 && p.bc[3] == 0;
#pragma unroll
      for (int r = 0; r < NR; ++r)
        load_spinor(q[r], x + (size_t)min(r, nr - 1) * rs, sb, V, wrap ? (T)-1 : (T)1);
    }
    sap_hop<MU, false, NR, T, S>(acc, q, gl, sb);
  }
}

}  // namespace dev
}  // namespace ddamg
