// Launches of a call of lb_step: they end in the buffer that swaps_buffers says,
// and where an even spread does not, the cheaper neighbour is taken.
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace oreg;

static void fail(const char* what, long long n, long long m, long long nodes) {
  std::printf("FAIL %s: %lld steps in %lld launches, %lld nodes\n", what, n, m, nodes);
  std::exit(1);
}

int main() {
  long long checked = 0;
  for (int64_t nodes : {300304LL, 490000LL, 1048576LL, 2890000LL, 4194304LL, 16777216LL, 1073741824LL})
    for (int64_t n = 1; n <= 400; ++n)
      for (int K : {7, 1}) {
        const bool swap = swaps_buffers(n, K == 7, 7, true);
        const int64_t m = number_launches(n, K, nodes, swap);
        if (m < (n + K - 1) / K || m > n) fail("count", n, m, nodes);
        if (((m & 1) != 0) != swap) fail("parity", n, m, nodes);
        ++checked;
      }
  // launches of one to four steps cost the same here, so few of six beat many of three
  for (int64_t n : {11, 12, 13})
    if (number_launches(n, 7, 4194304, true) < 3 || number_launches(n, 7, 4194304, false) != 2)
      fail("two launches", n, number_launches(n, 7, 4194304, false), 4194304);
  for (int64_t n : {16, 17, 18})
    if (number_launches(n, 7, 4194304, true) != 3) fail("three launches", n, 0, 4194304);
  // beyond the cache long calls take as few launches as there are
  if (number_launches(994, 7, 16777216, false) != 142) fail("sevens", 994, 0, 16777216);
  // in cache a launch of six costs more than 1.5 of four
  if (number_launches(24, 7, 1000000, false) != 6) fail("six launches", 24, 0, 1000000);
  // tile and block launches: us of a launch of L steps
  auto cheap = [](int L) { return L <= 7 ? 10.0 + L : -1.0; };
  auto dear = [](int L) { return L <= 7 ? 1.0 + 10 * L * L : -1.0; };
  auto none = [](int L) { return L <= 6 ? 10.0 + L : -1.0; };
  if (launches_for(7, 2, true, cheap) != 1) fail("one launch of seven", 7, launches_for(7, 2, true, cheap), 0);
  if (launches_for(7, 2, true, dear) != 3) fail("three launches", 7, launches_for(7, 2, true, dear), 0);
  if (launches_for(7, 2, true, none) != 3) fail("no launch of seven", 7, launches_for(7, 2, true, none), 0);
  auto even = [](int L) { return 10.0 + 2 * L; };  // one of twelve 34, three of four 54
  if (launches_for(12, 2, true, even, 0.63) != 1 || launches_for(12, 2, true, even, 0.62) != 3)
    fail("clearly cheaper", 12, 0, 0);
  if (launches_for(7, 2, true, cheap, 0) != 3 || launches_for(9, 1, false, cheap, 0) != 2 ||
      launches_for(2, 2, true, cheap, 0) != 1)
    fail("never fewer", 7, 0, 0);
  if (launches_for(12, 2, false, dear) != 2 || launches_for(2, 2, true, cheap) != 1 ||
      launches_for(9, 1, false, cheap) != 2)
    fail("ends", 0, 0, 0);
  std::printf("checked %lld\n", checked);
  return 0;
}
