// Checks the rules by which a call takes one kernel or another against times
// measured for both (us).  Prints one line per point; exit status 1 where a
// rule takes the slower side by more than a twentieth.
#include <cstdio>
#include <initializer_list>

#include "blas_sizes.h"

using namespace ddamg;

static int fails = 0;

static void point(const char* what, size_t n, int k, bool first, double t_first, double t_second) {
  const double mine = first ? t_first : t_second, other = first ? t_second : t_first;
  const bool ok = mine <= 1.05 * other;
  std::printf("%-14s %6zu %3d  %7.1f against %7.1f  %s\n", what, n, k, mine, other, ok ? "ok" : "FAIL");
  if (!ok) ++fails;
}

int main() {
  // coarse GMRES step k on n elements, FP32, one rhs: one workgroup, many
  const struct {
    size_t n;
    int k;
    double one, many;
  } steps[] = {{1536, 26, 59.9, 97.1},   {3072, 26, 82.2, 107.7},   {6144, 1, 35.1, 57.5},    {6144, 9, 73.0, 80.2},
               {6144, 27, 144.8, 129.6}, {8192, 5, 58.9, 63.6},     {8192, 13, 103.8, 88.3},  {8192, 27, 176.8, 127.7},
               {12288, 1, 48.6, 68.0},   {12288, 3, 61.5, 59.1},    {12288, 6, 91.9, 77.2},   {12288, 27, 253.0, 140.2},
               {16384, 1, 53.8, 64.3},   {16384, 3, 74.3, 64.0},    {16384, 27, 316.6, 135.0}, {20480, 1, 71.6, 69.9},
               {20480, 3, 89.5, 68.6},   {24576, 1, 81.4, 75.7},    {24576, 27, 777.1, 144.9}};
  for (const auto& s : steps) point("coarse step", s.n, s.k, arnoldi_one_group(s.n, s.k), s.one, s.many);
  // a longer basis or a longer vector never brings the one workgroup back
  for (size_t n = 16; n <= 24576; n += 16)
    for (int k = 0; k < 64; ++k)
      if (!arnoldi_one_group(n, k) && (arnoldi_one_group(n, k + 1) || arnoldi_one_group(n + 16, k))) ++fails;
  // coarse stencil of few rhs, sites and rows: four waves per workgroup, sixteen
  const struct {
    int nout, nc, nrhs;
    bool half;
    double four, sixteen;
  } gemv[] = {{4096, 8, 2, false, 11.0, 34.3},   {4096, 16, 2, false, 20.0, 125.8}, {4096, 16, 4, true, 19.6, 126.6},
              {4096, 24, 3, false, 32.1, 121.0}, {8192, 32, 2, true, 66.0, 122.6},  {8192, 48, 2, true, 141.0, 172.0},
              {256, 48, 1, false, 13.5, 9.8},    {256, 48, 2, false, 19.2, 13.3},   {256, 64, 1, true, 16.0, 8.5}};
  for (const auto& g : gemv) {
    const int w = stencil_gemv_shape(8, g.half, g.nc, 9, g.nrhs, g.nout).waves;
    point("coarse stencil", g.nc, g.nrhs, w <= 4, g.four, g.sixteen);
  }
  // every shape: lanes for the rows of a column within a wave, the rows of a
  // lane within a column, the partial results in LDS
  for (int ntv = 1; ntv <= 32; ++ntv)
    for (int nslot : {1, 8, 9})
      for (int nrhs = 1; nrhs <= 5; ++nrhs)
        for (int nout = 1; nout <= 16384; nout *= 2)
          for (int type = 0; type < 3; ++type) {
            const int nc = 2 * ntv;
            const size_t es = type == 0 ? 16 : 8;
            const GemvShape g = stencil_gemv_shape(es, type == 2, nc, nslot, nrhs, nout);
            if (g.waves == 0 ? nrhs < 4 : nrhs > 4) ++fails;
            if (g.waves == 0) continue;
            int lanes = 1;
            while (lanes * g.rows < nc) lanes *= 2;
            const size_t lds = (size_t)(nslot + g.waves) * nc * nrhs * es;
            if (lanes > 64 || nc % g.rows || g.rows < 2 || (es == 16 && g.rows != 2) || g.waves > 16 ||
                (g.waves & (g.waves - 1)) || lds > 80 * 1024) {
              std::printf("shape ntv %d nslot %d nrhs %d nout %d type %d: rows %d waves %d lds %zu FAIL\n", ntv, nslot,
                          nrhs, nout, type, g.rows, g.waves, lds);
              ++fails;
            }
          }
  // a wave per row tile (at most two), chunks of columns; FP32, 5 and 12 rhs, FP16
  for (int nc = 2; nc <= 64; nc += 2)
    for (bool half : {false, true})
      if (stencil_by_tiles(half, nc, 5, 1 << 20) && nc > 32) ++fails;
  point("row tiles", 8, 5, stencil_by_tiles(false, 8, 5, 4096), 12.5, 24.0);
  point("row tiles", 16, 5, stencil_by_tiles(false, 16, 5, 4096), 22.1, 25.4);
  point("row tiles", 20, 5, stencil_by_tiles(false, 20, 5, 4096), 42.5, 58.8);
  point("row tiles", 24, 5, stencil_by_tiles(false, 24, 5, 4096), 50.2, 59.4);
  point("row tiles", 24, 12, stencil_by_tiles(false, 24, 12, 8192), 157.7, 134.9);
  point("row tiles", 24, 5, stencil_by_tiles(false, 24, 5, 256), 12.7, 7.6);
  point("row tiles", 12, 5, stencil_by_tiles(true, 12, 5, 8192), 28.9, 35.7);
  point("row tiles", 24, 5, stencil_by_tiles(true, 24, 5, 8192), 88.4, 72.3);
  // restriction by lanes, on the matrix cores
  point("restriction", 4, 5, restrict_by_lanes(true, 4, 256, 5), 58.0, 69.0);
  point("restriction", 4, 8, restrict_by_lanes(true, 4, 90, 8), 107.0, 126.0);
  point("restriction", 4, 12, restrict_by_lanes(true, 4, 256, 12), 148.0, 140.0);
  point("restriction", 4, 5, restrict_by_lanes(true, 4, 16, 5), 54.0, 41.0);
  point("restriction", 8, 5, restrict_by_lanes(true, 8, 256, 5), 85.0, 82.0);
  point("restriction", 24, 4, restrict_by_lanes(true, 24, 256, 4), 106.0, 134.0);
  point("restriction", 4, 3, restrict_by_lanes(false, 4, 256, 3), 68.0, 92.0);
  point("restriction", 4, 8, restrict_by_lanes(false, 4, 256, 8), 169.0, 153.0);
  point("restriction", 24, 3, restrict_by_lanes(false, 24, 256, 3), 261.0, 202.0);
  // network layers on the vector units, on the matrix cores
  const struct {
    int cin, cout, V;
    double lanes, cores;
  } layer[] = {{1, 1, 8192, 35, 43},     {4, 4, 8192, 68, 50},      {2, 12, 8192, 54, 58},     {4, 4, 32768, 81, 86},
               {8, 4, 32768, 128, 127},  {12, 1, 32768, 172, 158},  {1, 1, 131072, 63, 192},   {4, 4, 131072, 195, 270},
               {3, 12, 131072, 394, 348}, {16, 2, 131072, 553, 770}, {8, 8, 131072, 546, 493},  {16, 16, 131072, 1760, 958},
               {2, 24, 131072, 559, 609}, {4, 24, 131072, 865, 641}},
    wgrad[] = {{1, 1, 131072, 266, 970},     {8, 8, 131072, 900, 1094},  {12, 8, 131072, 1261, 1163},
               {4, 24, 131072, 1777, 2328}, {8, 24, 131072, 2903, 2374}, {16, 16, 131072, 3147, 1393}};
  for (const auto& x : layer) point("network layer", x.cin, x.cout, net_layer_thin(x.cin, x.cout, x.V), x.lanes, x.cores);
  for (const auto& x : wgrad) point("weight gradient", x.cin, x.cout, net_wgrad_thin(x.cin, x.cout, x.V), x.lanes, x.cores);
  return fails ? 1 : 0;
}
