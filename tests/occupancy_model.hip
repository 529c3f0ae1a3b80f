// Prints how many workgroups of the sorted-merge level kernel the library expects on a compute unit:
// bits, class, recomputing form or not, workgroups.
#include "../paper_2103_16063_amd/csrc/rannc_dp_worklist.h"

#include <cstdio>

int main() {
  for (int bits : {32, 64})
    for (int DP : {8, 16, 32, 64})
      for (int recompute : {0, 1})
        std::printf("%d %d %d %d\n", bits, DP, recompute, rannc::merge_workgroups_per_cu(bits, DP, recompute != 0));
  return 0;
}
