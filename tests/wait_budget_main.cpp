// The staging loop of the single-kernel layer in miniature: `steps` waits in a row share one budget.
#include <cstdio>
#include <initializer_list>

#include "oea_wait.h"

// looks made until step s has its data (arrives[s] < 0: never); returns the steps that gave up
static int stage(oea::WaitBudget budget, const int* arrives, int steps, int* looks) {
  int gave_up = 0;
  *looks = 0;
  for (int s = 0; s < steps; ++s) {
    for (int look = 1;; ++look) {
      ++*looks;
      if (arrives[s] >= 0 && look > arrives[s]) break;
      if (!budget.again()) {
        ++gave_up;
        break;
      }
    }
  }
  return gave_up;
}

int main() {
  int looks, failures = 0;
  const int never[5] = {-1, -1, -1, -1, -1}, at_once[5] = {0, 0, 0, 0, 0}, late[5] = {3, 0, 2, 0, 1}, lost[5] = {2, -1, 4, 0, 0};
  for (uint32_t limit : {0u, 1u, 7u, 1000u, 524288u}) {
    // nothing ever arrives: the first step uses the budget up, the others look once each
    if (stage({limit}, never, 5, &looks) != 5 || looks != int(limit) + 5) ++failures;
    if (stage({limit}, at_once, 5, &looks) != 0 || looks != 5) ++failures;
  }
  if (stage({6}, late, 5, &looks) != 0 || looks != 11) ++failures;  // exactly the six repeats that are needed
  if (stage({5}, late, 5, &looks) != 1) ++failures;
  // a step that gave up leaves nothing for the ones behind it; what has already arrived is still taken
  if (stage({9}, lost, 5, &looks) != 2 || looks != 9 + 5) ++failures;
  std::printf(failures ? "wait budget: FAILED (%d)\n" : "wait budget: ok\n", failures);
  return failures ? 1 : 0;
}
