// The tuner's choice with a clock that adds a disturbance to chosen
// measurements.  Ends with 0 if every case holds.
#include "../paper_2603_21869_amd/csrc/fastest.hpp"

#include <stdio.h>

#include <initializer_list>

int main() {
  const float base[5] = {0.0495f, 0.0516f, 0.0621f, 0.0618f, 0.0618f};  // (ms for three launches)
  // any one measurement of any candidate disturbed by 2 to 24 us
  for (int who = 0; who < 5; ++who)
    for (int when = 0; when < 3; ++when)
      for (float add : {0.002f, 0.006f, 0.012f, 0.024f}) {
        int count[5] = {0, 0, 0, 0, 0};
        const int got = nfvm::fastest(5, true, [&](int i) {
          return base[i] + (i == who && count[i]++ == when ? add : 0.f);
        });
        if (got != 0) {
          printf("FAILED: candidate %d chosen with candidate %d's measurement %d disturbed\n", got,
                 who, when);
          return 1;
        }
      }
  // without settling, and far from the best, a candidate is measured once
  int calls = 0;
  const float far[5] = {1.f, 2.f, 0.5f, 3.f, 4.f};
  auto once = [&](int i) {
    ++calls;
    return far[i];
  };
  if (nfvm::fastest(5, false, once) != 2 || calls != 5) return 1;
  calls = 0;
  if (nfvm::fastest(5, true, once) != 2 || calls != 7) return 1;
  return 0;
}
