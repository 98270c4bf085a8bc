// Host check of the rules that pick a call's launches, from the library's own
// headers.  Prints the number of failures.
#include <cstdio>

#include "k_setup.h"

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

int main() {
  eigen_chunks();
  std::printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
