// The kernel that the projection planner (host-only header) gives a call: reads
// lines "bf16 k tok n_ex T ragged n_modules d_in d_out d_in d_out ..." and prints, for
// each, "general", "few 64" or "few 16" (tokens per workgroup).
#include <algorithm>
#include <cstdio>

#include "project_plan.h"

int main() {
  int bf16, k, tok, ragged, mods;
  long long n, T;
  while (std::scanf("%d %d %d %lld %lld %d %d", &bf16, &k, &tok, &n, &T, &ragged, &mods) == 7) {
    long long sum = 0, most = 0;
    for (int m = 0; m < mods; ++m) {
      long long a, b;
      if (std::scanf("%lld %lld", &a, &b) != 2) return 1;
      sum += a + b;
      most = std::max(most, a + b);
    }
    const attr::ProjFewPlan P = attr::plan_project_few(bf16 != 0, k / 16, tok != 0, sum, most, mods, n, T, ragged != 0);
    if (P.ct)
      std::printf("few %d\n", P.ct);
    else
      std::printf("general\n");
  }
  return 0;
}
