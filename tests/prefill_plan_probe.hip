// Host program around prefill_plan.h, for test_prefill_plan.py: answers one line
// for each line of its input.
//   plan T units d paged psaw factor sink cus   -> w ns qblock qfirst blocks
//   time T units d paged psaw factor sink cus   -> microseconds a plan takes
//   order units nqb group                       -> block of every workgroup, "unit:block"
//   group per nqb cus                           -> units worked through side by side
#include <stdio.h>
#include <string.h>

#include <chrono>

#include "prefill_plan.h"

int main() {
  char what[16];
  while (scanf("%15s", what) == 1) {
    if (!strcmp(what, "order")) {
      int units, nqb, group;
      if (scanf("%d %d %d", &units, &nqb, &group) != 3) return 1;
      for (int L = 0; L < units * nqb; ++L) {
        int bh = -1, qb = -1;
        prhs::block_of(units, nqb, group, L, &bh, &qb);
        printf("%d:%d ", bh, qb);
      }
      printf("\n");
      continue;
    }
    if (!strcmp(what, "group")) {
      int per, nqb, cus;
      if (scanf("%d %d %d", &per, &nqb, &cus) != 3) return 1;
      printf("%d\n", prhs::unit_group(per, nqb, cus));
      continue;
    }
    prhs::PrefillShape s;
    long long units;
    int cus;
    if (scanf("%d %lld %d %d %d %lf %d %d", &s.T, &units, &s.d, &s.paged, &s.psaw, &s.psaw_f, &s.sink, &cus) != 8)
      return 1;
    if (!strcmp(what, "time")) {
      double best = 1e9;
      int keep = 0;
      for (int r = 0; r < 60; ++r) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < 10; ++i) keep += prhs::plan_of(s, units, cus).qblock;
        const std::chrono::duration<double, std::micro> us = std::chrono::steady_clock::now() - t0;
        best = us.count() / 10 < best ? us.count() / 10 : best;
      }
      printf("%.4f %d\n", best, keep != 0);
      continue;
    }
    const prhs::PrefillPlan p = prhs::plan_of(s, units, cus);
    printf("%d %d %d %d %d\n", p.w, p.ns, p.qblock, p.qfirst, p.blocks(s.T));
  }
}
