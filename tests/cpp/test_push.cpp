// CPU tests of fill_slot (cdd_sched.h) with a fake copy engine: transfers stay
// under way until drained, and any of them, or the event behind them, may fail.
#include <cstdio>
#include <vector>

#include "cdd_sched.h"

struct Engine {
  int fail_at = -1;  // number of the call of send or mark that fails
  int calls = 0;
  size_t staged = 0, next = 0;
  int in_flight = 0, drains = 0;
  bool marked = false, in_order = true;
  int step() { return calls++ == fail_at ? 700 + fail_at : 0; }
};

static int run(Engine& g, size_t bytes) {
  return cdd::fill_slot(
      bytes,
      [&](size_t at, size_t n) {
        g.in_order &= at == g.staged;
        g.staged += n;
      },
      [&](size_t at, size_t n) {
        g.in_order &= at == g.next && at + n <= g.staged;
        const int e = g.step();
        if (e == 0) {
          g.next += n;
          ++g.in_flight;
        }
        return e;
      },
      [&] {
        const int e = g.step();
        g.marked = e == 0;
        return e;
      },
      [&] {
        ++g.drains;
        g.in_flight = 0;
      });
}

int main() {
  int bad = 0;
  const size_t sizes[] = {1, 4096, (4u << 20) - 1, 4u << 20, (4u << 20) + 2, 9000001};
  for (size_t bytes : sizes) {
    const int pieces = bytes >= (4u << 20) ? 2 : 1;
    for (int fail = -1; fail <= pieces; ++fail) {
      Engine g;
      g.fail_at = fail;
      const int e = run(g, bytes);
      bool ok = g.in_order;
      if (fail < 0)
        ok = ok && e == 0 && g.marked && g.next == bytes && g.in_flight == pieces && g.drains == 0;
      else  // the error, and nothing that still reads the slot
        ok = ok && e == 700 + fail && !g.marked && g.in_flight == 0 && g.drains == 1;
      if (!ok) {
        std::printf("FAIL bytes %zu fail %d: e %d, in flight %d\n", bytes, fail, e, g.in_flight);
        ++bad;
      }
    }
  }
  std::printf(bad ? "%d failures\n" : "all passed\n", bad);
  return bad ? 1 : 0;
}
