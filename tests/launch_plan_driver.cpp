// Prints how a compress call's heads are spread over workgroups (csrc/fc_plan.cpp:
// plan_split, plan_fused_launches).  Built, fed and checked by test_launch_plan.py.
// Input, one case per line (all integers):
//   nl nh d mode in_place n_cu n_req, then n_req times: length method budget window
// With any argument: one line per case, whether it goes without plan_alloc (plan_one_launch), as
// a pruned call and as one that is not.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../paper_2503_08461_amd/csrc/fc_plan.h"

using namespace fc;

int main(int argc, char**) {
  PoolView pv;
  int mode, in_place, n_cu, n_req;
  while (scanf("%d %d %d %d %d %d %d", &pv.n_layers, &pv.n_heads, &pv.head_dim, &mode, &in_place,
               &n_cu, &n_req) == 7) {
    std::vector<int32_t> lens(n_req), methods(n_req), budgets(n_req), windows(n_req), widths(n_req, 7);
    for (int i = 0; i < n_req; ++i)
      if (scanf("%d %d %d %d", &lens[i], &methods[i], &budgets[i], &windows[i]) != 4) return 2;
    pv.score_mode = mode;
    pv.in_place = in_place != 0;
    pv.n_free = 1 << 30;
    CompressArgs a;
    a.n_req = n_req;
    a.max_blocks = 2048;
    a.seq_lens = lens.data();
    a.method = methods.data();
    a.budget = budgets.data();
    a.window_per_req = windows.data();
    a.pool_kernel_per_req = widths.data();
    a.q_ok = a.lse_ok = true;
    CompressPlan plan;
    if (plan_compress(pv, a, &plan) != PLAN_OK) return 3;
    const int split = plan_split(pv, n_cu, &plan);
    if (argc > 1) {
      const size_t n = split ? 0 : plan_fused_launches(pv, plan, n_cu).size();
      printf("O %d %d\n", plan_one_launch(pv, plan, n, true), plan_one_launch(pv, plan, n, false));
      continue;
    }
    printf("C %d %zu", split, plan.raw_floats);
    for (const ReqDesc& d : plan.descs) printf(" %lld", (long long)d.raw_off);
    printf("\n");
    for (const FusedLaunch& l : plan_fused_launches(pv, plan, n_cu)) {
      printf("F %d %d %d %d %d", l.wide ? 1 : 0, l.query_tiles, l.max_len, l.max_blocks, l.half_reuse ? 1 : 0);
      for (int32_t i : l.units) printf(" %d", i);
      printf("\nP");  // the lengths from which it prunes, by query tiles
      for (int32_t n : l.prune_from.tiles) printf(" %d", n);
      printf("\n");
    }
  }
  return 0;
}
