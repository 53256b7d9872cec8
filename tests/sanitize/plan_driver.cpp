// Prints the launches that plan.cpp gives a pass loop: for lines of "rows cols
// beta k maps batch_px", "few lead start:passes ..." of the plain loop, then
// "|", the same (start:passes:advance) of the loop with the period-2 stop and
// whether that loop runs by them, then "|" and the loop of a batch's image.
#include <cstdio>

#include "plan.hpp"

int main() {
  int rows, cols, beta, k, maps;
  long long px;
  auto print = [&](const phg::LaunchPlan& pl) {
    std::printf(" %d", pl.lead);
    const int launches = k > 0 ? pl.launch_of(k - 1) + 1 : 0;
    for (int j = 0; j < launches; ++j)
      std::printf(" %d:%d", pl.start(j), (j + 1 < launches ? pl.start(j + 1) : k) - pl.start(j));
    std::printf(" |");
  };
  while (std::scanf("%d %d %d %d %d %lld", &rows, &cols, &beta, &k, &maps, &px) == 6) {
    const phgrms_params p{rows, cols, 20, beta, k};
    std::printf("%d", phg::deep_few_passes(p, maps != 0));
    print(phg::deep_plan(p, maps != 0));
    const phg::CyclePlan c = phg::cycle_plan(p);
    for (int j = 0; k > 1; ++j) {
      std::printf(" %d:%d:%d", c.start(j), c.passes(j), c.advance(j));
      if (c.last(j)) break;
    }
    std::printf(" %d |", phg::cycle_plan_pays(p) ? 1 : 0);
    print(phg::LaunchPlan::unpacked(phg::deep_batch_plan(beta, k, px).packed()));
    std::printf("\n");
  }
  return 0;
}
