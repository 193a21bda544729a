// CPU test of the matrix fragments of the first pass (cdd_mfma.h): every entry of
// F, put together from its parts, against the long-double value, and the mean
// power gain of F, which gain_of takes as exactly 1.
#include <cmath>
#include <cstdio>

#include "cdd_mfma.h"

using namespace cdd;

int main() {
  const std::vector<float2> tab = make_mf_table();
  const _Float16* h = (const _Float16*)tab.data();
  int bad = 0;
  for (int kind = 0; kind < kMfKinds; ++kind) {
    double worst = 0, power = 0;
    for (int s = 0; s < 2; ++s)
      for (int l = 0; l < 64; ++l)
        for (int e = 0; e < 8; ++e) {
          const int row = l & 31, m = row >> 1, c = row & 1;
          const int k = (m & 9) | ((m & 2) << 1) | ((m & 4) >> 1);
          const int r = 8 * s + 4 * (l >> 5) + (e >> 1), ci = e & 1;
          const long double turn = kind == kMfPlain ? (long double)(r * k) / 16.0L
                                                    : (long double)(k * (2 * r + 1)) / 32.0L;
          const long double ang = -2.0L * acosl(-1.0L) * turn;
          const long double want = c == ci ? cosl(ang) : c ? sinl(ang) : -sinl(ang);
          long double got = 0;
          for (int p = 0; p < kMfParts; ++p)
            got += (long double)h[(((size_t)(kind * 2 + s) * kMfParts + p) * 64 + l) * 8 + e];
          got /= (long double)kMfScale;
          worst = std::fmax(worst, (double)fabsl(got - want));
          power += (double)(got * got);
        }
    power /= 2.0 * 16 * 16;  // |F_kr|^2 twice (re and im rows), 16 x 16 entries
    std::printf("kind %d: largest error %.2e, power gain - 1 %.2e\n", kind, worst, power - 1.0);
    if (!(worst <= 0x1p-29)) ++bad;                 // 1.9e-9; half a unit of FP32 is 3e-8 to 7e-9
    if (!(std::fabs(power - 1.0) <= 2e-9)) ++bad;  // well below the correction's 1e-8
  }
  std::printf(bad ? "%d failures\n" : "all passed\n", bad);
  return bad ? 1 : 0;
}
