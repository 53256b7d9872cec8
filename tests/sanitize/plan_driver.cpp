// Prints the launches that plan.cpp gives a pass loop: for lines of "rows cols
// beta k maps", "few lead start:passes ..." of the plain loop, then "|", the
// same (start:passes:advance) of the loop with the period-2 stop and whether
// that loop runs by them.
#include <cstdio>

#include "plan.hpp"

int main() {
  int rows, cols, beta, k, maps;
  while (std::scanf("%d %d %d %d %d", &rows, &cols, &beta, &k, &maps) == 5) {
    const phgrms_params p{rows, cols, 20, beta, k};
    const phg::LaunchPlan pl = phg::deep_plan(p, maps != 0);
    std::printf("%d %d", phg::deep_few_passes(p, maps != 0), pl.lead);
    const int launches = k > 0 ? pl.launch_of(k - 1) + 1 : 0;
    for (int j = 0; j < launches; ++j) {
      const int end = j + 1 < launches ? pl.start(j + 1) : k;
      std::printf(" %d:%d", pl.start(j), end - pl.start(j));
    }
    std::printf(" |");
    const phg::CyclePlan c = phg::cycle_plan(p);
    for (int j = 0; k > 1; ++j) {
      std::printf(" %d:%d:%d", c.start(j), c.passes(j), c.advance(j));
      if (c.last(j)) break;
    }
    std::printf(" %d\n", phg::cycle_plan_pays(p) ? 1 : 0);
  }
  return 0;
}
