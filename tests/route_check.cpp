// Host check of the rules that pick a call's launches, from the library's own
// headers.  Prints the number of failures.
#include <cstdio>

#include "k_setup.h"
#include "routes.h"

static int bad = 0;
#define CHECK(x)                                     \
  do {                                               \
    if (!(x)) {                                      \
      std::printf("line %d: %s\n", __LINE__, #x);    \
      ++bad;                                         \
    }                                                \
  } while (0)

using namespace fc;

// eigen-decompositions: one launch where 256 MB hold the blocks, and never more
static void eigen_chunks() {
  CHECK(jacobi_chunk(27, 13824) == 13824);
  CHECK(jacobi_chunk(8, 110592) == 110592);
  for (int m = 1; m <= 192; ++m) {
    const int64_t c = jacobi_chunk(m, int64_t(1) << 30);
    CHECK(c >= 2048);
    CHECK(m > 64 || (c * m * m * 8 <= int64_t(256) << 20));
    CHECK(jacobi_chunk(m, 1) == 1);
  }
}

// rows, stored entries, longest row and slices of n^3 cells at degree p, scalar
struct Cube {
  int64_t rows, nnz = 1, slices = 0;
  int32_t longest = 1;
  Cube(int64_t n, int64_t p) {
    const int64_t n1 = p * n + 1, nv = n - 1, nn = n1 - nv;
    rows = n1 * n1 * n1;
    for (int d = 0; d < 3; ++d) {
      nnz *= nv * (2 * p + 1) + nn * (p + 1);
      longest *= (int32_t)(n > 1 ? 2 * p + 1 : p + 1);
    }
    for (int c = 0; c < 8; ++c) {
      int64_t k = 1;
      for (int d = 0; d < 3; ++d) k *= c >> d & 1 ? nv : nn;
      slices += (k + 63) / 64;
    }
  }
  bool joins() const { return step_joins(nnz, longest); }
  bool few_long() const { return few_long_rows(nnz, rows, slices); }
  bool rows_in_step() const { return joins() ? rows_beat_join(nnz, rows, slices) : few_long(); }
};

// the layout of a step's product, where the launch that the joined p update saves
// counts, is not that of the product alone
static void step_layouts() {
  for (int n = 4; n <= 9; ++n) CHECK(Cube(n, 2).few_long() && !Cube(n, 2).rows_in_step());
  for (int n = 10; n <= 15; ++n) CHECK(Cube(n, 2).few_long() && Cube(n, 2).rows_in_step());
  for (int n = 16; n <= 64; ++n) CHECK(!Cube(n, 2).few_long() && !Cube(n, 2).rows_in_step());
  for (int n = 2; n <= 100; ++n) CHECK(!Cube(n, 1).few_long());
  // rows too long for the joined form: the product alone decides
  for (int n = 2; n <= 13; ++n) CHECK(!Cube(n, 3).joins() && Cube(n, 3).rows_in_step());
  CHECK(!Cube(14, 3).rows_in_step());
}

int main() {
  eigen_chunks();
  step_layouts();
  std::printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
