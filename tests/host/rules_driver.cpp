// Host-only rules of the planning code, one question a line of input:
//   rows slo1 slo2 slo3 shi1 shi2 shi3 n1 n2 n3 pitch tail
//   count lo1 lo2 lo3 hi1 hi2 hi3 step |e3|
// Prints 1 or 0 a line.
#include <cstdio>
#include <cstring>

#include "plan.h"

int main() {
  char what[32];
  while (std::scanf("%31s", what) == 1) {
    if (std::strcmp(what, "rows") == 0) {
      long long v[11];
      for (long long& x : v)
        if (std::scanf("%lld", &x) != 1) return 1;
      const int64_t lo[3] = {v[0], v[1], v[2]}, hi[3] = {v[3], v[4], v[5]}, n[3] = {v[6], v[7], v[8]};
      std::printf("%d\n", vr::rows_readable(lo, hi, n, (int32_t)v[9], v[10]) ? 1 : 0);
    } else if (std::strcmp(what, "count") == 0) {
      long long v[6];
      double step, length;
      for (long long& x : v)
        if (std::scanf("%lld", &x) != 1) return 1;
      if (std::scanf("%lf %lf", &step, &length) != 2) return 1;
      vr::Box b;
      for (int i = 0; i < 3; i++) {
        b.lo[i] = v[i];
        b.hi[i] = v[3 + i];
        b.closed[i] = 1;
      }
      vr::Camera cam;
      std::memset(&cam, 0, sizeof cam);
      cam.e3[1] = length;
      std::printf("%d\n", vr::samples_countable(cam, b, step) ? 1 : 0);
    } else {
      return 1;
    }
  }
  return 0;
}
