// For each line of the input (CUs, number of tensors, their lengths): vectors per lane of the
// big tiles that the library takes for the list.  Then the calls that take big tiles.
#include <cstdio>
#include <iostream>
#include <vector>

#include "slowmo_plan.h"

using namespace slowmo;

int main() {
  int32_t cus, n;
  while (std::cin >> cus >> n) {
    std::vector<int64_t> numel(static_cast<size_t>(n));
    for (int64_t &v : numel) std::cin >> v;
    std::printf("%d\n", choose_big_vpt(n, numel.data(), cus));
  }
  for (int policy : {0, 1, 2})
    for (int32_t m : {7, 8, 15, 16, 32})
      std::printf("%d %d\n", m >= kBigFusedFromWorkers && last_takes_big(policy, false),
                  m >= kBigFusedFromWorkers && outer_takes_big(m, policy, false));
}
