// Host program: the bounds that searches with send times, or with the two maxima apart, are asked at, for every answer that a bound
// can give.  Prints the first sequence that asks twice at a bound, asks below the least value, or does not end.
#include "../paper_2103_16063_amd/csrc/rannc_dp_attempts.h"

#include <cstdio>
#include <vector>

using namespace rannc;

static int walk(const Attempts &a, std::vector<double> asked, double U, int k) {
  for (double x : asked)
    if (x == U) { std::printf("bound %g again behind %zu attempts (least %g)\n", U, asked.size(), a.least); return 1; }
  if (U < a.least || k >= a.most()) { std::printf("bound %g, attempt %d (least %g)\n", U, k, a.least); return 1; }
  asked.push_back(U);
  if (a.next(k, U, kLevelsFound) >= 0.0) { std::printf("goes on behind a value\n"); return 1; }
  for (LevelState state : {kLevelsNone, kLevelsOpen}) {
    const double next = a.next(k, U, state);
    if (next >= 0.0 && state == kLevelsNone && next <= U) { std::printf("no value at %g, then %g\n", U, next); return 1; }
    if (next >= 0.0 && walk(a, asked, next, k + 1)) return 1;
  }
  return 0;
}

int main() {
  for (double least : {0.0, 1.0, 3.0, 100.0, 1e6, 1.7e13})
    for (bool asked : {false, true})
      for (bool apart : {false, true})
        for (bool small : {false, true})
          for (double over : {0.0, 1.0, 3.0, 1e5}) {
            const Attempts a = {least, asked, apart, small};
            if (walk(a, {}, a.first(least + over), 0)) return 1;
          }
  std::printf("ok\n");
  return 0;
}
