// Prints how a decode attention cuts its heads (csrc/fc_plan.cpp: plan_decode_segments).
// Built, fed and checked by test_decode_split_plan.py.
// Input, one case per line (all integers): nl nh n_cu over_kept n_req, then the lengths.
// Output, a line per case: blocks of a segment, segments of the launch, then every head's.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../paper_2503_08461_amd/csrc/fc_plan.h"

using namespace fc;

int main() {
  PoolView pv;
  pv.head_dim = 128;
  int n_cu, over_kept, n_req;
  while (scanf("%d %d %d %d %d", &pv.n_layers, &pv.n_heads, &n_cu, &over_kept, &n_req) == 5) {
    std::vector<int32_t> lens(n_req), whole(n_req, kPlanMaxSeqLen);
    for (int32_t& n : lens)
      if (scanf("%d", &n) != 1) return 2;
    DecodePlan plan;
    if (plan_decode_attention(pv, n_req, 2048, over_kept ? whole.data() : lens.data(),
                              over_kept ? lens.data() : nullptr, &plan) != PLAN_OK)
      return 3;
    plan_decode_segments(pv, n_cu, over_kept != 0, &plan);
    printf("%d %d", plan.seg_blocks, plan.n_seg);
    // every head's segments, as the kernels cut it: their number, then where each begins, then the end
    for (int len : lens) {
      const int blocks = (len + kPlanBlockSize - 1) / kPlanBlockSize;
      const int n = plan.n_seg > 1 ? decode_segments(blocks, plan.seg_blocks) : 1;
      printf(" %d", n);
      for (int seg = 0; seg <= n; ++seg) printf(" %d", decode_segment_begin(blocks, n, seg));
    }
    printf("\n");
  }
  return 0;
}
