// wrap_add of csrc/dispatch.hpp against 64-bit arithmetic, for sides up to
// 2^31 - 1 (run under the undefined-behaviour sanitizer).
#include <cstdio>
#include <cstdlib>

#include "dispatch.hpp"

int main() {
  long checked = 0;
  for (int n : {1, 2, 3, 5, 50, 64, 100, 1000, 2147483600, 2147483647})
    for (int k = 0; k < 200; ++k) {
      const int v = k < 100 ? k % n : n - 1 - (k - 100) % n;
      for (int d = -300; d <= 4000; ++d, ++checked) {
        int64_t r = ((int64_t)v + d) % n;
        if (r < 0) r += n;
        if (oreg::detail::wrap_add(v, d, n) != r) {
          std::printf("FAIL (%d + %d) mod %d\n", v, d, n);
          return 1;
        }
      }
    }
  std::printf("checked %ld\n", checked);
  return 0;
}
