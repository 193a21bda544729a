// CPU tests of the dispatch rules (cdd_rules.h).
#include <cstdio>

#include "cdd_rules.h"

using namespace cdd;

static int g_fail = 0;
#define CHECK(cond)                                                   \
  do {                                                                \
    if (!(cond)) {                                                    \
      std::printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond);     \
      ++g_fail;                                                       \
    }                                                                 \
  } while (0)

static bool two(int N, int trials, int64_t nchan, int64_t n) {
  return two_blocks_pay(N, trials, nchan * n, nchan * ((n + 1) / 2 * 2));
}

// Two blocks per workgroup never where the spare ones cost more than sharing gains.
static void test_two_blocks() {
  for (int N : {512, 1024, 2048, 4096}) {
    for (int trials : {1, 2, 3, 8, 16, 32, 64}) {
      if (N == 4096 && trials <= 4) continue;     // faster throughout
      CHECK(!two(N, trials, 2048, 1));            // twice the transforms
      CHECK(two(N, trials, 2048, 2));             // nothing spare
      CHECK(two(N, trials, 512, 131) && two(N, trials, 512, 33));
      CHECK(!two(N, trials, 16, 9) && !two(N, trials, 16, 10));  // a compute unit per block
      bool last = false;  // once two pay at an odd count, they do at every larger one
      for (int64_t n = 1; n < 200; n += 2) {
        const bool t = two(N, trials, 1024, n);
        CHECK(t || !last);
        last = t;
      }
    }
    CHECK(!two(N, 16, 1024, 3) || N == 512);
    CHECK(!two(N, 48, 1024, 3));
    CHECK(!two(N, 48, 1024, 5) || N == 4096);
  }
}

// Detection straight from the record: the sizes measured on both sides of the line.
static void test_detection() {
  for (int f = 0; f < 2; ++f) {
    CHECK(!detect_from_record(f, 1, 1 << 20, 4) && !detect_from_record(f, 512, 1 << 20, 65));
    for (int n_int = 1; n_int <= 16; ++n_int)
      CHECK(detect_from_record(f, 2, 16, n_int) && detect_from_record(f, 64, 4000, n_int) &&
            detect_from_record(f, 4096, 100000, n_int));
    for (int64_t c : {2, 4, 16, 32, 64})
      for (int64_t t : {4000, 40000})
        for (int n_int : {25, 32, 48, 64}) CHECK(!detect_from_record(f, c, t, n_int));
    for (int n_int : {17, 24, 32, 48, 64}) {
      CHECK(detect_from_record(f, 512, 40000, n_int) && detect_from_record(f, 16, 400000, n_int));
      CHECK(detect_from_record(f, 2, 400000, n_int) == (f || n_int <= 32));
    }
    CHECK(detect_from_record(f, 2, 500, 48) && detect_from_record(f, 512, 500, 64));
  }
  CHECK(detect_from_record(false, 16, 4000, 20) && !detect_from_record(true, 16, 4000, 20));
  CHECK(detect_from_record(false, 128, 4000, 16) && !detect_from_record(true, 128, 4000, 16));
  CHECK(detect_from_record(true, 128, 4000, 12) && detect_from_record(true, 512, 4000, 16));
}

static void test_fold() {
  CHECK(fold_threads(1000, 1000.0, 1) == 256 && fold_threads(1000, 1.5, 1024) == 256);
  CHECK(fold_threads(1000, 500.0, 1025) == 64 && fold_threads(1000, 501.0, 1025) == 1);
  CHECK(fold_threads(999, 333.0, 4096) == 64 && fold_threads(999, 334.0, 4096) == 1);
  CHECK(fold_threads(1000, 250.0, 8192) == 64 && fold_threads(1000, 251.0, 8192) == 1);
  CHECK(fold_threads(1000000, 1.5, 8192) == 64 && fold_threads(1000, 1e6, 8192) == 1);
  CHECK(fold_threads(1000, 1.5, 8193) == 1);
}

// Each beam's units are taken by their own length.
static void test_units_per_value() {
  int32_t take[2];
  // 64 trials at 2048 points beside 2 trials of many blocks at the same length
  const double points[] = {2048.0 * 65, 2048.0 * 3};
  const int64_t units[] = {5000, 400000};
  units_per_value(2, points, units, 1024, take);
  CHECK(take[0] == 1 && take[1] == 4);
  const double small[] = {256.0 * 4 * 65, 256.0 * 4 * 3};
  units_per_value(2, small, units, 2048, take);
  CHECK(take[0] == 1 && take[1] == 15);
  // short units alone: at most 16 at once, and four values per workgroup to the end
  for (int64_t n : {1, 100, 2048, 8191, 8192, 40000, 250000, 100000000}) {
    const double p = 256.0 * 3;
    units_per_value(1, &p, &n, 2048, take);
    CHECK(take[0] >= 1 && take[0] <= 16);
    CHECK(take[0] == 1 || n / take[0] >= 4 * 2048);
    CHECK(n < 250000 || take[0] == 16);
  }
  // the last beam of a launch is handed out evenly, however many went before
  const double same[] = {768.0, 768.0};
  const int64_t tail[] = {1000000, 3000};
  units_per_value(2, same, tail, 2048, take);
  CHECK(take[0] == 16 && take[1] == 1);
}

int main() {
  test_two_blocks();
  test_units_per_value();
  test_fold();
  test_detection();
  if (g_fail) {
    std::printf("%d failures\n", g_fail);
    return 1;
  }
  std::printf("all passed\n");
  return 0;
}
