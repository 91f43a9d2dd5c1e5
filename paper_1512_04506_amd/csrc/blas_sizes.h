// Sizes of the partial-sum workspace that the Krylov multi-dot kernels
// (k_blas.hip) write: one partial per (rhs, vector, chunk of the vector).
// Plain host arithmetic without HIP, shared by the launchers (which refuse
// to launch into a buffer that is too small), the allocation of every such
// buffer, and a CPU test of the allocation rules.
#pragma once
#include <cstddef>

namespace ddamg {

// workgroups per rhs (chunks) of a multi-dot over n elements per rhs: one per
// 8192 elements (more of them cost long vectors of many rhs their overhead:
// 16^4, 8 rhs, 79 us against 87 at 1024 elements each), at most 512, but
// about 1024 over all rhs while each keeps 1024 elements (8^4, one rhs: six
// workgroups took 27 us, 48 take 7.6 us; 16^3x32: 192, 41 us, 1024, 25 us).
inline int blas_nchunks(size_t n, int nrhs) {
  size_t c = (n + 8191) / 8192;
  if (c > 512) c = 512;
  size_t fill = nrhs > 0 ? 1024 / (size_t)nrhs : 1;
  if (fill > (n + 1023) / 1024) fill = (n + 1023) / 1024;
  if (c < fill) c = fill;
  if (c < 1) c = 1;
  return (int)c;
}

// partial sums written by a multi-dot of nvec vectors over n elements per
// rhs for nrhs rhs (the fused second Gram-Schmidt pass over nvec vectors
// writes nvec + 1 of them per rhs and chunk: the extra one is |w|^2)
inline size_t mdot_part_entries(size_t n, int nvec, int nrhs) {
  return (size_t)(nrhs > 0 ? nrhs : 0) * (size_t)(nvec > 0 ? nvec : 0) * (size_t)blas_nchunks(n, nrhs);
}

// the largest of them over calls of up to nrhs rhs (fewer rhs take more chunks each)
inline size_t mdot_part_capacity(size_t n, int nvec, int nrhs) {
  size_t c = 0;
  for (int r = 1; r <= nrhs; ++r) {
    const size_t e = mdot_part_entries(n, nvec, r);
    if (e > c) c = e;
  }
  return c;
}

// Whether coarse GMRES step k on vectors of n elements runs in one workgroup
// per rhs (k_arnoldi.hip) or in the ten many-workgroup launches.  A step reads
// k + 1 basis vectors four times: one compute unit takes 0.59 us per 1000
// elements and vector, the many workgroups 2.6 us per vector whatever its
// length (up to 24576 elements) and some 18 us more to begin with.  So the one
// workgroup wins for any k up to about 4096 elements and for ever fewer
// vectors beyond.  FP32, one rhs, us per step (with the operator, one workgroup
// against many): 6144 elements k = 8..11 73/80, k = 24..29 145/130; 12288
// elements k = 3 61/59, k = 24..29 253/140; 24576 elements k = 1 81/76, k =
// 24..29 777/145.  FP64 and 4 or 12 rhs cross within two vectors of it.
inline bool arnoldi_one_group(size_t n, int k) { return n <= 4096 || (size_t)(k + 1) * (n - 4096) <= 32768; }

// Shape of the coarse stencil's vector kernel (k_stencil.hip): rows of a
// column per lane and waves per workgroup; waves = 0: the matrix cores.
struct GemvShape {
  int rows, waves;
};
// esize: bytes of a complex entry of the vectors; half: D_c stored in FP16;
// nslot slots of nc columns; nrhs rhs, nout output sites.
// Sixteen waves hide the chain of a workgroup while there are few of them.
// Once they fill the chip, the sum over the waves and their column groups is
// all that more waves add, so four do (eight for the longest columns), each
// group with four columns at least: 2 rhs on 4096 sites, FP32, N_tv 8 126 us
// with sixteen waves, 18 with four; N_tv 24 192 and 127; 256 sites, N_tv 24, one
// rhs 9.8 and 13.5.  Two rows per lane where four would leave lanes idle or,
// with the sums of four rhs, fill the registers: FP32, 4 rhs, 4096 sites, N_tv
// 16 58 us against 64.  The matrix cores compute 16 rhs at one price: FP16, 4
// rhs, 4096 sites, N_tv 24 92 us against 114, 2 rhs 89 against 73.
inline GemvShape stencil_gemv_shape(size_t esize, bool half, int nc, int nslot, int nrhs, int nout) {
  if (nrhs > 4 || (nrhs == 4 && half && nc >= 32)) return {0, 0};
  const bool f32 = esize == 8;
  const bool four = f32 && nc % 4 == 0 && (nrhs == 1 || nc > (half ? 16 : 32)) && !(nrhs == 4 && nout > 512 && nc <= 48);
  const int rows = four ? 4 : 2;
  int waves = 16, lanes = 1;  // lanes for the rows of a column
  while (lanes * rows < nc) lanes *= 2;
  const size_t col = (size_t)nc * nrhs * esize;
  if ((nslot + waves) * col > 49152) waves /= 2;
  if (nout > 512 && nc * esize <= 384) {
    waves = waves < 4 ? waves : 4;
  } else if (nout > 256 && nrhs > 1) {
    waves = waves < 8 ? waves : 8;
  }
  const int groups = 64 / lanes, least = nslot > 1 || nout > 256 ? 4 : 1;
  while (waves > 1 && waves * groups * least > nslot * nc) waves /= 2;
  return {rows, waves};
}

// Whether the stencil of 5 and more rhs in FP32 arithmetic takes a wave per 16
// rows (at most two) instead of the kernel that deals columns in chunks of 16
// to four or eight waves; groups: output sites times groups of 16 rhs.  The
// chunks and row tiles of the latter are partly empty for few rows, and its
// sum over the waves costs a grid that fills the chip without it (us, row
// tiles against chunks): FP32, 5 rhs, 4096 sites, N_tv 4 12/24, 8 22/25, 10
// 43/59, 12 50/59, and 12 rhs, 8192 sites, N_tv 12 157/135; FP16, 5 rhs, 8192
// sites, N_tv 6 29/36, 12 88/72; FP32, 5 rhs, 256 sites, N_tv 12 13/8.
inline bool stencil_by_tiles(bool half, int nc, int nrhs, int groups) {
  if (half) return nc <= 12 && groups > 2048;
  if (nc <= 12) return groups > 512;
  if (nc <= 16) return groups > 2048;
  return nc <= 20 ? groups > 1000 : nc <= 24 && (nrhs - 1) % 16 < 8 && groups > 1500;
}

// Whether the restriction runs on the vector units, a lane per site, instead
// of the matrix cores (k_coarse.hip).  4 rhs in FP32 and 2 in FP64 fit the
// registers, so the basis is read once; the matrix cores do 16 rhs and 16 test
// vectors at one price.  Up to four test vectors, that price is more than a
// second pass over their few planes on all but the smallest blocks (us, matrix
// cores against lanes): N_tv 4, 16^3x32 on 4^4, FP16, 5 rhs 69/58, 12 rhs
// 135/138; FP64, 3 rhs 92/68, 8 rhs 153/169; 16^4 on 2^4, FP32, 5 rhs 41/54; N_tv
// 8, 16^3x32 on 4^4, FP32, 5 rhs 82/85.
inline bool restrict_by_lanes(bool f32, int ntv, int vblock, int nrhs) {
  const bool thin = ntv <= 4 && vblock > 16;
  return nrhs <= (f32 ? 4 : 2) * (thin ? 2 : 1);
}

// Whether a layer of the network runs on the vector units, a lane per site and
// four output channels, instead of the matrix cores (k_learn.hip).  The matrix
// cores compute 4 input and 16 output channels at one price, so few
// channels in either place leave them mostly idle; the lanes need some 8000 sites
// to fill the chip with two or more input channels and repeat gate and
// transport for every four outputs (us, matrix cores against lanes): 16^3x32, 1
// to 1 channels 192/63, 4 to 4 270/195, 3 to 12 348/394, 16 to 2 770/553, 8 to
// 8 493/546; 16^3x8, 4 to 4 86/81, 8 to 4 127/128; 8^3x16, 1 to 8 51/41, 4 to 4
// 50/68.
inline bool net_layer_thin(int cin, int cout, int V) {
  const int lanes = cin * ((cout + 3) / 4), tiles = ((cin + 3) / 4) * ((cout + 15) / 16);
  if (cin <= 4) return (cin == 1 || V >= (cin == 2 ? 8192 : 32768)) && lanes <= 8 * tiles;
  return V >= 65536 && lanes <= 6 * tiles;
}

// The same for its weight gradients, tiles of 16 by 16 channels against a lane
// per site, one input and two output channels: 16^3x32, 1 to 1 channels 970/266,
// 8 to 8 1094/900, 12 to 8 1163/1261, 4 to 24 2328/1777, 8 to 24 2374/2903.
inline bool net_wgrad_thin(int cin, int cout, int V) {
  return V >= 65536 && cin * ((cout + 1) / 2) <= 32 * ((cin + 15) / 16) * ((cout + 15) / 16);
}

// Krylov workspace of GMRES(m) on vectors of n elements per rhs: the
// widest multi-dot is the Gram-Schmidt of a new vector against all m + 1
// basis vectors of a cycle; the norm of a coarse right-hand side runs over
// more elements than the basis vectors, so n is the longest of a call
inline size_t krylov_part_entries(int m, int nrhs, size_t n) { return mdot_part_capacity(n, m + 1, nrhs); }

// normalisation of the ntv fine test vectors of the setup (one norm per
// vector over 12 V elements)
inline size_t setup_norm_part_entries(int ntv, size_t fine_elems) { return mdot_part_capacity(fine_elems, 1, ntv); }

}  // namespace ddamg
