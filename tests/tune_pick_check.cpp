// Host check of the autotuner's choice (tune_pick.h).  Prints "ok" and exits 0, or prints the
// failing case and exits 1.
#include <cstdio>

#include "tune_pick.h"

int main() {
  struct Case {
    double time[3];
    int base;
    double margin;
    int want;
  };
  const Case cases[] = {
      {{3.0, 2.0, 1.0}, 0, 0.0, 2},     // no margin: the fastest
      {{1.0, 1.0, 1.0}, 0, 0.0, 0},     // ties: the lower index
      {{1.0, 1.0, 2.0}, 1, 0.0, 1},     // ... but the base where nothing is faster
      {{1.0, 0.99, 2.0}, 0, 0.02, 0},   // within the margin: the base
      {{1.0, 0.97, 2.0}, 0, 0.02, 1},
      {{0.99, 1.0, 2.0}, 1, 0.02, 1},   // the margin is against the base, whichever that is
      {{0.90, 1.0, 2.0}, 1, 0.02, 0},   // shape 0 clearly faster than the base: shape 0
      {{1.0, 0.5, 0.4}, 1, 0.02, 2},
  };
  for (const Case& c : cases) {
    const int got = pick_variant(c.time, 3, c.base, c.margin);
    if (got != c.want) {
      std::printf("times %g %g %g base %d margin %g: %d, not %d\n", c.time[0], c.time[1], c.time[2], c.base, c.margin,
                  got, c.want);
      return 1;
    }
  }
  std::printf("ok\n");
  return 0;
}
