// Checks the rules by which a call takes one kernel or another against times
// measured for both (us).  Prints one line per point; exit status 1 where a
// rule takes the slower side by more than a twentieth.
#include <cstdio>

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
  return fails ? 1 : 0;
}
