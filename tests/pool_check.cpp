// Host check of the memory kept between preconditioners (dev_pool.hip) over a
// stand-in for the HIP allocator.  Prints the number of failures.
#include <cstdio>

#include "dev_pool.hip"

static int bad = 0;
#define CHECK(x)                                          \
  do {                                                    \
    if (!(x)) {                                           \
      std::printf("line %d: %s\n", __LINE__, #x);         \
      ++bad;                                              \
    }                                                     \
  } while (0)

using namespace fc;
constexpr size_t kMB = size_t(1) << 20;

static void* get(size_t bytes) {
  void* p = nullptr;
  return pool_malloc(&p, bytes) == hipSuccess ? p : nullptr;
}

// an idle buffer is handed out again, and all go back with the last problem
static void reuse() {
  pool_problem_created();
  void* a = get(8 * kMB);
  pool_free(a, true);
  CHECK(get(7 * kMB) == a);
  pool_free(a, true);
  CHECK(stub::used == 8 * kMB);
  pool_problem_destroyed();
  CHECK(stub::used == 0);
}

// a buffer whose wait failed is handed out only after a wait that came later
static void failed_wait() {
  pool_problem_created();
  void* a = get(8 * kMB);
  stub::may_wait = false;
  const bool idle = device_idle() == hipSuccess;
  CHECK(!idle);
  pool_free(a, idle);
  void* b = get(8 * kMB);
  CHECK(b && b != a);
  stub::may_wait = true;
  void* c = get(8 * kMB);
  CHECK(c && c != a && c != b);
  CHECK(device_idle() == hipSuccess);
  CHECK(get(8 * kMB) == a);
  pool_free(a, true);
  pool_free(b, true);
  pool_free(c, true);
  pool_problem_destroyed();
  CHECK(stub::used == 0);
}

// buffers that cannot be given back stay parked and go later
static void parked_to_the_end() {
  pool_problem_created();
  void* a = get(8 * kMB);
  stub::may_wait = false;
  pool_free(a, false);
  pool_problem_destroyed();
  CHECK(stub::live.count(a));
  stub::may_wait = true;
  pool_problem_created();
  pool_problem_destroyed();
  CHECK(!stub::live.count(a));
}

// memory runs out: parked buffers are given back as well as kept ones
static void out_of_memory() {
  pool_problem_created();
  const size_t old = stub::budget;
  stub::budget = stub::used + 10 * kMB;
  pool_free(get(4 * kMB), true);
  stub::may_wait = false;
  pool_free(get(5 * kMB), false);
  stub::may_wait = true;
  void* a = get(9 * kMB);
  CHECK(a);
  pool_free(a, false);   // the device may be waited for: gone at once
  CHECK(!stub::live.count(a));
  stub::budget = old;
  pool_problem_destroyed();
}

// .. and for memory that is not itself kept
static void out_of_memory_elsewhere() {
  pool_problem_created();
  const size_t old = stub::budget;
  stub::budget = stub::used + 10 * kMB;
  pool_free(get(4 * kMB), true);
  double* d = nullptr;
  CHECK(dev_malloc(&d, 9 * kMB) == hipSuccess && d);
  CHECK(dev_malloc(&d, 9 * kMB) == hipErrorOutOfMemory && !d);
  stub::budget = old;
  pool_problem_destroyed();
}

int main() {
  reuse();
  failed_wait();
  parked_to_the_end();
  out_of_memory();
  out_of_memory_elsewhere();
  std::printf("failures %d\n", bad);
  return bad ? 1 : 0;
}
