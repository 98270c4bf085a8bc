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

// n^dim cells at degree p, scalar: rows, stored entries, longest row, slices, cells
// and unknowns of a cell
struct Grid {
  int64_t rows = 1, nnz = 1, slices = 0, cells = 1;
  int32_t longest = 1, m = 1;
  Grid(int dim, int64_t n, int64_t p) {
    const int64_t n1 = p * n + 1, nv = n - 1, nn = n1 - nv;
    for (int d = 0; d < dim; ++d) {
      rows *= n1;
      nnz *= nv * (2 * p + 1) + nn * (p + 1);
      longest *= (int32_t)(n > 1 ? 2 * p + 1 : p + 1);
      cells *= n;
      m *= (int32_t)(p + 1);
    }
    for (int c = 0; c < 1 << dim; ++c) {
      int64_t k = 1;
      for (int d = 0; d < dim; ++d) k *= c >> d & 1 ? nv : nn;
      slices += (k + 63) / 64;
    }
  }
  bool joins() const { return step_joins(nnz, longest); }
  bool few_long() const { return few_long_rows(nnz, rows, slices); }
  bool rows_in_step() const { return joins() ? rows_beat_join(nnz, rows, slices) : few_long(); }
  bool tiny() const { return tiny_sizes(nnz, rows, cells, m); }
};
struct Cube : Grid {
  Cube(int64_t n, int64_t p) : Grid(3, n, p) {}
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

// the sizes of test_gpu_routes.py and test_gpu_tiny.py take the kernels they are there
// for
static void tested_sizes() {
  CHECK(Cube(13, 3).few_long() && !Cube(14, 3).few_long());
  CHECK(Cube(12, 4).few_long() && !Cube(13, 4).few_long());
  const int tiny[][3] = {{2, 1, 1}, {2, 7, 1}, {2, 31, 1}, {2, 44, 1}, {2, 1, 2}, {2, 16, 2},
                         {2, 25, 2}, {2, 5, 3}, {2, 13, 3}, {2, 1, 4}, {2, 9, 4}, {3, 1, 1},
                         {3, 9, 1}, {3, 1, 2}, {3, 2, 2}, {3, 3, 2}, {3, 4, 2}, {2, 47, 1},
                         {2, 26, 2}, {2, 16, 3}, {2, 10, 4}, {3, 11, 1}};
  for (auto& t : tiny) {
    CHECK(Grid(t[0], t[1], t[2]).tiny());
    if (!Grid(t[0], t[1], t[2]).tiny()) std::printf("  %d %d %d\n", t[0], t[1], t[2]);
  }
  const int more[][3] = {{2, 48, 1}, {2, 27, 2}, {2, 17, 3}, {2, 11, 4}, {3, 12, 1}, {3, 5, 2}};
  for (auto& t : more) {
    CHECK(!Grid(t[0], t[1], t[2]).tiny());
    if (Grid(t[0], t[1], t[2]).tiny()) std::printf("  %d %d %d\n", t[0], t[1], t[2]);
  }
}

// chunks of the block products: whole 16-byte pieces, and a tile of at most 20 KB
static void staged_chunks() {
  for (int f64 = 0; f64 < 2; ++f64)
    for (int m = 65; m <= 192; ++m)
      for (int64_t n : {1, 640, 641, 1024, 1025, 100000}) {
        const int r = staged_rows(f64, m, n), most = m <= 96 ? 96 : m <= 128 ? 128 : 192;
        CHECK(r >= 4 && r % (f64 ? 2 : 4) == 0 && r * most * (f64 ? 8 : 4) <= 20 * 1024);
        CHECK(staged_rows(f64, m, 1) >= r);
      }
}

int main() {
  staged_chunks();
  tested_sizes();
  eigen_chunks();
  step_layouts();
  std::printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
