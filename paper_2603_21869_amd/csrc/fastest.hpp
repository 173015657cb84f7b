// The autotuner's choice among the timed candidates of a kernel.
#pragma once

namespace nfvm {

// Index of the candidate whose time is least (n <= 8; time(i) measures i, in
// ms).  One measurement is of a few launches, and now and then something else
// on the machine adds 2 to 6 us to them.  With settle, candidates within
// FASTEST_NEAR of the best are measured twice more and the least of each
// counts: the choice is then the same in every process unless two candidates
// are equally fast.  (The dot products of a 208 x 112 x 80 grid in FP32 take
// 11.9 us with one target and 12.1 with the next: 27 of 80 processes chose the
// slower one without, none of 40 with; 128^3 in mixed precision, 16.5 / 17.2:
// 15 of 160 and none of 40.)
constexpr float FASTEST_NEAR = 0.03f;
template <class T>
int fastest(int n, bool settle, T&& time) {
  float t[8];
  int best = 0;
  for (int i = 0; i < n; ++i) {
    t[i] = time(i);
    if (t[i] < t[best]) best = i;
  }
  for (int round = 0; settle && round < 2; ++round) {
    const float near = t[best] + FASTEST_NEAR;
    for (int i = 0; i < n; ++i) {
      if (t[i] > near) continue;
      const float v = time(i);
      if (v < t[i]) t[i] = v;
    }
    for (int i = 0; i < n; ++i)
      if (t[i] < t[best]) best = i;
  }
  return best;
}

}  // namespace nfvm
