// Host-side planning of libfastcache's batched calls (see fc_plan.h).
//
// The batch compression step of FastCache's serving loop (Algorithm 1) is
// issued once for the whole batch; what the host scheduler knows about the
// batch (lengths, methods, budgets, free blocks: "Memory-Aware Scheduling"
// paragraph) is enough to validate it, to detect that the pool cannot take
// it, and to lay out every request's share of the stage's buffers before any
// device work is queued.

#include "fc_plan.h"

#include <stdarg.h>
#include <stdio.h>

#include <algorithm>
#include <numeric>

namespace fc {

namespace {

// FusedLaunch::query_tiles of a launch whose windows need different numbers of tiles.
constexpr int kMixedQueryTiles = kPlanClasses;

// Heads shorter than this are not worth the launches of the split path, and with more
// than one head per two CUs its second read of K and its extra launches cost more than
// the idle CUs.  A call of one layer, window 32, 128 channels, fused / split in us:
//             4 heads       32            64            128           160 heads
//   SnapKV
//     1500    48.5 / 38.7   50.4 / 41.3   52.4 / 48.0   56.2 / 55.7   57.0 / 59.2
//     2048    54.8 / 41.1   57.6 / 42.8   60.3 / 50.9   64.1 / 63.2   65.7 / 71.2
//     4000    78.4 / 46.0   85.5 / 57.0   89.2 / 66.7   96.8 / 96.9   98.7 / 112
//     16000    228 / 79      247 / 115     275 / 176     301 / 314     322 / 388
//   64 channels
//     2048    43.8 / 38.0   45.1 / 40.3   46.0 / 43.6   49.4 / 48.3   50.0 / 52.1
//     16000    168 / 74      182 / 83      191 / 109     202 / 170     207 / 207
//   key-norm, 128 channels
//     2048    32.6 / 29.8   34.7 / 32.1   37.5 / 36.6   43.5 / 47.6   46.2 / 54.2
//     4000    49.2 / 33.1   53.4 / 40.2   58.8 / 49.1   68.3 / 69.0   73.6 / 78.4
//     16000    150 / 45      168 / 80      191 / 118     239 / 231     262 / 288
// (These are sums of kernels; the launches between them, two to five more, are not in them.)
constexpr int kSplitMinLen = 2048;

// Whether the `units` heads of up to 8192 tokens of a call are better off in wide workgroups.
// Of these a CU takes one at a time, of the narrow ones three or four.  So wide ones are for
// calls that one round of them can take: the heaviest head as long as it keeps their wavefronts
// busy, and all heads together, heaviest first, no more than that for every CU.  All kernels
// of a call, narrow / wide in us, each pruned or not, whichever is the faster:
//   heads                4            128          256          320          512
//   SnapKV, window 32, 128 channels
//     1000 tokens     35 / 38      39 / 43      45 / 48      54 / 75      66 / 82
//     2000            52 / 54      62 / 64      74 / 73      89 / 117    108 / 131
//     3000                                     102 / 95     121 / 154    153 / 176
//     8000                                     232 / 222    289 / 355    399 / 426
//   64 channels
//      700            25 / 26      26 / 28      28 / 29      31 / 43      35 / 47
//     1000            29 / 28      31 / 30      35 / 33      39 / 51      44 / 54
//     2000            41 / 37      48 / 43      53 / 47      61 / 73      69 / 81
//     8000                                     166 / 129    194 / 220    221 / 240
//   key-norm, 128 channels
//      256          19.0 / 18.8  19.9 / 19.6  21.0 / 20.4  22.2 / 27.8  24.8 / 32.0
//      640          24.0 / 20.8  26.6 / 23.1  29.8 / 29.1  33.9 / 40.0  40.5 / 46.1
//     2000          43.0 / 29.7  52.5 / 43.5  58.5 / 56.6  71.3 / 81.3  93.9 / 99.9
// (windows 16 and 64 cross where 32 does, streaming where key norms do).  With lengths that
// differ, 500-4000 tokens, SnapKV: 320 heads 107 / 101 and at 64 channels 81 / 66, 384 heads
// 109 / 106 and 83 / 66, 512, which are more than a round, 137 / 159 and 92 / 100.
bool wide_pays(const PoolView& pool, const CompressPlan& plan, size_t units, int n_cu) {
  if (units > 2 * (size_t)n_cu) return false;
  const ReqDesc* heaviest = nullptr;
  int64_t most = 0, all = 0;
  for (size_t i = 0; i < plan.descs.size(); ++i) {
    const ReqDesc& d = plan.descs[i];
    if (d.method != PLAN_METHOD_STREAMING && d.seq_len > kPlanFusedMaxLen) continue;  // (wide anyhow)
    all += plan.weights[i] * (int64_t)(pool.n_layers * pool.n_heads);
    if (!heaviest || plan.weights[i] > most) {
      heaviest = &d;
      most = plan.weights[i];
    }
  }
  if (!heaviest || all > most * n_cu) return false;
  return heaviest->seq_len >= (heaviest->method != PLAN_METHOD_SNAPKV ? 256 : pool.head_dim == 128 ? 2048 : 896);
}

// From what mean length of its SnapKV heads (each weighted by its own) on a launch of
// narrow workgroups leaves only half of the keys to the caches in its first pass.  All
// kernels of a pruned call, window 16 to 64, 128 channels, all / half:
//   8192 heads of  700 tokens  512-538 / 529-558 us     4096 heads of 3000  1118-1125 / 1082-1107
//   8192          1500         1082-1086 / 1105-1141    2048          4000  744-758 / 718-726
//   6144          2400         1316-1341 / 1316-1338    2048          6500  1208-1212 / 1139-1162
//   4096          2000         729-732 / 728-751         768          2500  165-172 / 157-165
// With three and more query tiles that kernel takes 3 KB more of LDS, so where a head of
// more than 7820 tokens is in the launch (kPlanHalfReuseWords) two workgroups of it fit a
// CU, not three, and the plain one is the faster.  1536 heads of 7900-8190 tokens, window
// 48 half 1200, all 1180, window 64 1210 and 1167; of 6000-8192 1065 and 1043, 1086 and
// 1052; but of 7700-7800 1052 and 1105, 1070 and 1117, and with window 32, where both fit
// alike, of 6000-8192 987 and 1036.
constexpr int kHalfReuseLen = 2304;

int blocks_for(int tokens) { return (tokens + kPlanBlockSize - 1) / kPlanBlockSize; }

template <typename Plan>
int fail(Plan* plan, int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(plan->message, sizeof(plan->message), fmt, ap);
  va_end(ap);
  plan->code = code;
  return code;
}

}  // namespace

int plan_compress(const PoolView& pool, const CompressArgs& a, CompressPlan* plan) {
  *plan = CompressPlan();
  plan->top_after = pool.n_free;
  if (a.n_req < 0) return fail(plan, PLAN_EINVAL, "n_req < 0");
  if (a.n_req == 0) return PLAN_OK;
  if (!a.seq_lens || !a.method || !a.budget) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (a.max_blocks < 1) return fail(plan, PLAN_EINVAL, "max_blocks_per_req < 1");
  const bool per_request = a.window_per_req != nullptr;
  if (per_request && !a.pool_kernel_per_req) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (!per_request &&
      (a.pool_kernel < 1 || a.pool_kernel > kPlanMaxPoolKernel || (a.pool_kernel & 1) == 0))
    return fail(plan, PLAN_EINVAL, "pool_kernel must be odd and in 1..%d", kPlanMaxPoolKernel);

  // ---- validate; lay out every request's share of the buffers ---------------
  const size_t n_lh = (size_t)pool.n_layers * pool.n_heads;
  std::vector<ReqDesc>& descs = plan->descs;
  descs.reserve(a.n_req);
  long long total_new = 0, total_old = 0, total_released = 0;
  size_t score_off = 0, kept_off = 0, q_off = 0;
  for (int r = 0; r < a.n_req; ++r) {
    const int m = a.method[r];
    // queries are packed: with per-request windows only SnapKV requests have any
    const size_t q_here = q_off;
    if (per_request) {
      if (m == PLAN_METHOD_SNAPKV)
        q_off += n_lh * (size_t)std::max(a.window_per_req[r], 0) * pool.head_dim;
    } else {
      q_off += n_lh * (size_t)std::max(a.window, 0) * pool.head_dim;
    }
    if (m == PLAN_METHOD_NONE) continue;
    const int L = a.seq_lens[r], B = a.budget[r];
    const int win = per_request ? a.window_per_req[r] : a.window;
    const int pk = per_request ? a.pool_kernel_per_req[r] : a.pool_kernel;
    if (m != PLAN_METHOD_SNAPKV && m != PLAN_METHOD_KNORM && m != PLAN_METHOD_STREAMING)
      return fail(plan, PLAN_EINVAL, "request %d: unknown method %d", r, m);
    if (L < 1 || L > kPlanMaxSeqLen)
      return fail(plan, PLAN_EINVAL, "request %d: length %d outside 1..%d", r, L, kPlanMaxSeqLen);
    if (B < 1 || B > L)
      return fail(plan, PLAN_EINVAL, "request %d: budget %d outside 1..%d", r, B, L);
    if (m == PLAN_METHOD_SNAPKV) {
      if (win < 1 || win > kPlanMaxWindow)
        return fail(plan, PLAN_EINVAL, "request %d: window %d outside 1..%d", r, win,
                    kPlanMaxWindow);
      if (pk < 1 || pk > kPlanMaxPoolKernel || (pk & 1) == 0)
        return fail(plan, PLAN_EINVAL, "request %d: pool_kernel must be odd and in 1..%d", r,
                    kPlanMaxPoolKernel);
      if (L < win || B < win)
        return fail(plan, PLAN_EINVAL, "request %d: SnapKV needs length and budget >= window", r);
      if (!a.q_ok)
        return fail(plan, PLAN_EINVAL, "dev_q_window must be a 16-byte aligned device pointer");
      if (a.need_lse && !a.lse_ok)
        return fail(plan, PLAN_EINVAL, "dev_lse_window must be a 4-byte aligned device pointer");
      plan->window_hi = std::max(plan->window_hi, win);
    }
    ReqDesc d = {};
    d.window = m == PLAN_METHOD_SNAPKV ? win : 0;
    d.pool_kernel = m == PLAN_METHOD_SNAPKV ? pk : 1;
    d.seq_len = L;
    d.budget = B;
    d.method = m;
    d.table_row = r;
    d.n_old = blocks_for(L);
    d.n_new = blocks_for(B);
    if (d.n_old > a.max_blocks)
      return fail(plan, PLAN_EINVAL, "request %d: %d blocks exceed max_blocks_per_req %d", r,
                  d.n_old, a.max_blocks);
    d.old_off = (int32_t)total_old;
    d.new_off = (int32_t)(pool.in_place ? total_released : total_new);
    d.score_off = (int64_t)score_off;
    d.raw_off = 0;
    d.kept_off = (int64_t)kept_off;
    d.q_off = (int64_t)q_here;
    total_old += d.n_old;
    total_new += pool.in_place ? 0 : d.n_new;
    total_released += d.n_old - d.n_new;
    score_off += n_lh * (size_t)L;
    kept_off += n_lh * (size_t)B;
    descs.push_back(d);
  }
  const int n_comp = (int)descs.size();
  if (n_comp == 0) return PLAN_OK;
  if (total_old > 0x7fffffffLL || total_new > 0x7fffffffLL)
    return fail(plan, PLAN_EINVAL, "batch too large");
  if (total_new > pool.n_free)
    return fail(plan, PLAN_ENOMEM, "batch needs %lld new blocks, %d free", total_new, pool.n_free);
  plan->total_new = (int)total_new;
  plan->total_old = (int)total_old;
  plan->total_released = (int)total_released;
  plan->kept_entries = kept_off;
  plan->score_entries = score_off;
  plan->top_after = pool.in_place ? pool.n_free + (int)total_released
                                  : pool.n_free - (int)total_new + (int)total_old;

  // ---- work lists ------------------------------------------------------------------
  // Descriptor indices, heaviest first so that the tail of each launch is made
  // of light units, per window class (class c: SnapKV with ceil(window/16) == c,
  // the number of 16-row query tiles the kernels are compiled for; class 0: no
  // queries at all).  Heads that narrow workgroups of the fused kernels (score ->
  // select -> gather in one workgroup) can take are in the fused lists; the rest
  // in those of the separate kernels: SnapKV per class, key-norm, and one list of
  // all of them for select and gather.  In the default scheduling the rest are the
  // longer heads, which plan_fused_launches puts into wide workgroups, and the
  // separate kernels run only with PLAN_SCORE_TWO_PASS.
  std::vector<int> sorted(n_comp);
  std::iota(sorted.begin(), sorted.end(), 0);
  // bytes a unit moves (K once or twice, kept K/V read and written)
  auto weight = [&](int i) {
    const ReqDesc& d = descs[i];
    const int passes = d.method == PLAN_METHOD_SNAPKV ? (a.need_lse ? 1 : 2)
                                                      : d.method == PLAN_METHOD_KNORM ? 1 : 0;
    return (int64_t)d.seq_len * passes + (int64_t)d.budget * 4;
  };
  for (int i = 0; i < n_comp; ++i) plan->weights.push_back(weight(i));
  std::stable_sort(sorted.begin(), sorted.end(),
                   [&](int x, int y) { return plan->weights[x] > plan->weights[y]; });
  const bool allow_fused = pool.score_mode == PLAN_SCORE_AUTO;
  auto fused = [&](int i) {
    const ReqDesc& d = descs[i];
    // (streaming: no score, no LDS, so the fused kernel whatever the length)
    return d.method == PLAN_METHOD_STREAMING ||
           (allow_fused && d.seq_len <= kPlanFusedMaxLen);
  };
  size_t raw_need = 0;
  for (int di : sorted) {
    ReqDesc& d = descs[di];
    const bool snap = d.method == PLAN_METHOD_SNAPKV;
    const int cls = snap ? (d.window + 15) / 16 : 0;
    int li;
    if (fused(di)) {
      li = LIST_FUSED + cls;
    } else {
      // (the separate kernels keep these units' scores in the library's scratch)
      d.raw_off = (int64_t)raw_need;
      raw_need += n_lh * (size_t)d.seq_len;
      li = snap ? LIST_SNAP + cls : LIST_KNORM;
      plan->lists[LIST_ALL].push_back(di);
      plan->max_len[LIST_ALL] = std::max(plan->max_len[LIST_ALL], d.seq_len);
    }
    plan->lists[li].push_back(di);
    // (sizes the score buffer in LDS, which streaming units do not use)
    if (d.method != PLAN_METHOD_STREAMING) plan->max_len[li] = std::max(plan->max_len[li], d.seq_len);
  }
  plan->raw_floats = raw_need;
  return PLAN_OK;
}

// Shorter heads take the two passes: the tokens of the first step have no bounds, and a step of
// a wide workgroup is three to four times as many tokens; bounding costs the same next to rows
// of 128 bytes as next to rows of 256, and more with more query tiles; and where a CU has less
// than its narrow workgroups to do, it waits for the longer chain of phases and not for K.  All
// kernels of a call, two passes / pruned in us:
//   narrow, 128 channels     window 32                     window 64
//     256 heads     1400 tokens  58 / 60  2000  77 / 74    1400  62 / 64  2000   81 / 79
//     512            512         41 / 45   700  53 / 53     700  53 / 55  1000   72 / 68
//     1024           450       60.5 / 59  512   66 / 62     512  76 / 83   640   91 / 95
//     4096           450        193 / 191  512 218 / 210    580 262 / 262  640  283 / 280
//     16384          450        756 / 733  512 850 / 810    450 787 / 782  580 1000 / 966
//   64 channels
//     256           8000        167 / 166                  5000 126 / 123
//     512           1400         57 / 57  2000  73 / 69    3000 107 / 105
//     2048           800         97 / 101  900 108 / 107   1024 126 / 124 1200  148 / 144
//     4096           800        172 / 173 1024 220 / 214   1200 275 / 280 1400  320 / 312
//     16384          700        566 / 558  900 738 / 701    900 798 / 817 1200 1040 / 1032
//   wide, 256 heads
//     128 channels  1600         66 / 67  2000  78 / 73    1600  68 / 69  2000   80 / 77
//      64           4500         85 / 85  5500 100 / 97    5500 105 / 105 7000  129 / 127
//   window 16, wide: 128 channels 1400 57 / 57, 64 channels 3000 61 / 61; window 48 as 64, at
//   64 channels earlier: narrow, 2048 heads, 900 114 / 113, wide 5500 101 / 100
// (192 heads of 64 channels cross later, 5000 tokens 83 / 88, 8000 122 / 120.)
PruneFrom plan_prune_from(int head_dim, bool wide, size_t heads, int n_cu) {
  if (wide) return head_dim == 128 ? PruneFrom{{1408, 1664, 1664, 1664}} : PruneFrom{{3584, 5120, 5632, 7168}};
  if (heads > 2 * (size_t)n_cu)
    return head_dim == 128 ? PruneFrom{{512, 512, 576, 576}} : PruneFrom{{864, 864, 1024, 1152}};
  if (heads > (size_t)n_cu)
    return head_dim == 128 ? PruneFrom{{768, 768, 896, 896}} : PruneFrom{{2048, 2048, 2048, 3072}};
  return head_dim == 128 ? PruneFrom{{1664, 1664, 2048, 2048}} : PruneFrom{{4096, 4096, 4096, 4096}};
}

std::vector<FusedLaunch> plan_fused_launches(const PoolView& pool, const CompressPlan& plan, int n_cu) {
  const size_t n_lh = (size_t)pool.n_layers * pool.n_heads;
  // Narrow workgroups (three or four to a CU) take heads of up to 8192 tokens; wide
  // ones (one to a CU, three to four times the wavefronts) take the longer heads,
  // whose scores fill the LDS of a CU, and calls with so few units that narrow
  // workgroups would leave most of the chip's wavefronts idle.  One launch per
  // shape, whatever windows its requests have: a launch per window class ends in a
  // tail of its own (24 requests with windows 1..64, 2 layers of 32 heads: 776 us
  // as four launches, 661-715 as one, by box).
  FusedLaunch wide, narrow;
  auto add = [](FusedLaunch& to, const std::vector<int32_t>& list) {
    to.units.insert(to.units.end(), list.begin(), list.end());
  };
  size_t short_units = 0;
  for (int c = 0; c < kPlanClasses; ++c) short_units += plan.lists[LIST_FUSED + c].size() * n_lh;
  const bool few = wide_pays(pool, plan, short_units, n_cu);
  for (int c = 0; c < kPlanClasses; ++c) {
    add(few ? wide : narrow, plan.lists[LIST_FUSED + c]);
    if (pool.score_mode == PLAN_SCORE_AUTO) add(wide, plan.lists[LIST_SNAP + c]);
  }
  if (pool.score_mode == PLAN_SCORE_AUTO) add(wide, plan.lists[LIST_KNORM]);
  wide.wide = true;
  std::vector<FusedLaunch> launches;
  for (FusedLaunch* l : {&wide, &narrow}) {
    if (l->units.empty()) continue;
    std::stable_sort(l->units.begin(), l->units.end(),
                     [&](int x, int y) { return plan.weights[x] > plan.weights[y]; });
    int64_t tokens = 0, weighted = 0;
    for (int i : l->units) {
      const ReqDesc& d = plan.descs[i];
      if (d.method != PLAN_METHOD_STREAMING) l->max_len = std::max(l->max_len, d.seq_len);
      l->max_blocks = std::max(l->max_blocks, d.n_old);
      if (d.method != PLAN_METHOD_SNAPKV) continue;
      const int tiles = (d.window + 15) / 16;
      l->query_tiles = l->query_tiles == 0 || l->query_tiles == tiles ? tiles : kMixedQueryTiles;
      tokens += d.seq_len;
      weighted += (int64_t)d.seq_len * d.seq_len;
    }
    l->half_reuse = pool.head_dim == 128 && !l->wide && tokens > 0 && weighted >= kHalfReuseLen * tokens &&
                    (l->query_tiles <= 2 || fused_lds(l->max_len, l->max_blocks, false).words <= kPlanHalfReuseWords);
    l->prune_from = plan_prune_from(pool.head_dim, l->wide, l->units.size() * n_lh, n_cu);
    launches.push_back(std::move(*l));
  }
  return launches;
}

// All kernels of a call, with plan_alloc / without in us (32 heads and fewer: a launch less is
// 2 to 4.5 of the host's).  Without it every workgroup counts itself out before its copy, one
// after the other (some 6 ns each); where there are many short heads they all come at once:
//   128 channels, tokens   128          256          400          700          1000
//    256 heads  SnapKV   21.7 / 19.0  22.0 / 21.6  27.3 / 26.7  38.7 / 38.3  48.7 / 47.6
//    512        SnapKV   22.1 / 23.0  28.8 / 29.2  37.0 / 36.5  67.2 / 66.4  86.9 / 84.7
//               key-norm 20.4 / 20.2  23.7 / 25.4  31.1 / 31.3  43.6 / 41.5  63.4 / 61.4
//    1024       SnapKV   29.1 / 33.3  38.7 / 39.7  56.7 / 55.0  79.8 / 77.9  105.0 / 102.8
//    2048       key-norm 35.2 / 44.5  52.8 / 57.5  83.6 / 83.7
//   64 channels
//    512        key-norm 20.4 / 19.3  20.4 / 19.7  21.8 / 23.0  28.7 / 30.2  34.0 / 32.6
//    1024       SnapKV   22.2 / 28.4  27.5 / 32.5  34.6 / 37.9  51.3 / 50.9  66.2 / 64.4
//               key-norm 20.1 / 24.8  22.8 / 29.9  30.5 / 34.9  42.7 / 43.6  55.4 / 54.4
// From a million tokens of all heads on the taking back at the very end shows and the launch
// at the beginning does not (1024 heads of 2000 tokens 228.7 / 231.6, of 7000 697 / 699).
// Streaming requests all come to their copy at once (25.2 / 25.9); calls with scores,
// log-sum-exps or without pruning gain as little and have no kernels for it.
bool plan_one_launch(const PoolView& pool, const CompressPlan& plan, size_t n_launches, bool pruned) {
  if (pool.score_mode != PLAN_SCORE_AUTO || plan.descs.size() != 1 || n_launches != 1) return false;
  const ReqDesc& d = plan.descs[0];
  if (d.method != PLAN_METHOD_KNORM && !(d.method == PLAN_METHOD_SNAPKV && pruned)) return false;
  if (plan.total_old + plan.total_new > kPlanOnlyMaxIds) return false;
  const long long heads = (long long)pool.n_layers * pool.n_heads;
  if (heads * d.seq_len > 1 << 20) return false;
  return heads <= 256 || d.seq_len * pool.head_dim >= 400 * 128;
}

int plan_split(const PoolView& pool, int n_cu, CompressPlan* plan) {
  if (pool.score_mode != PLAN_SCORE_AUTO || pool.in_place || plan->descs.empty()) return 0;
  const size_t units = (size_t)pool.n_layers * pool.n_heads * plan->descs.size();
  int longest = 0;
  for (const ReqDesc& d : plan->descs)
    if (d.method != PLAN_METHOD_STREAMING) longest = std::max(longest, d.seq_len);
  if (units > (size_t)n_cu / 2 || longest < kSplitMinLen) return 0;
  size_t raw = 0;
  for (ReqDesc& d : plan->descs) {
    d.raw_off = (int64_t)raw;
    raw += (size_t)pool.n_layers * pool.n_heads * d.seq_len;
  }
  plan->raw_floats = raw;
  // two workgroups per CU, segments of at least 256 tokens of the longest head
  return (int)std::min<size_t>(std::max<size_t>(2 * (size_t)n_cu / units, 2), longest / 256);
}

// All kernels of a key-norm call with the separate kernels, 4 / 16 wavefronts in us:
// 256 heads of 300, 700, 1500 and 4000 tokens 41.9 / 42.4, 60.5 / 61.5, 96.6 / 94.4
// and 209 / 203; 512 heads 50.4 / 54.8, 72.6 / 77.6, 119 / 123 and 300 / 300; 4096
// heads of 300 and 700 tokens 160 / 224 and 369 / 434.
bool select_is_wide(int max_len, size_t units, int n_cu) {
  return max_len > kPlanFusedMaxLen || (units <= (size_t)n_cu && max_len >= 1024);
}

int plan_window_lse(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                    const int32_t* method, int window, LsePlan* plan) {
  *plan = LsePlan();
  if (n_req < 0) return fail(plan, PLAN_EINVAL, "n_req < 0");
  if (n_req == 0) return PLAN_OK;
  if (!seq_lens) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (max_blocks < 1) return fail(plan, PLAN_EINVAL, "max_blocks_per_req < 1");
  if (window < 1 || window > kPlanMaxWindow)
    return fail(plan, PLAN_EINVAL, "window %d outside 1..%d", window, kPlanMaxWindow);
  const size_t n_lh = (size_t)pool.n_layers * pool.n_heads;
  for (int r = 0; r < n_req; ++r) {
    if (method && method[r] != PLAN_METHOD_SNAPKV) continue;
    const int L = seq_lens[r];
    if (L < window || L > kPlanMaxSeqLen)
      return fail(plan, PLAN_EINVAL, "request %d: length %d outside %d..%d", r, L, window,
                  kPlanMaxSeqLen);
    ReqDesc d = {};
    d.window = window;
    d.pool_kernel = 1;
    d.seq_len = L;
    d.budget = L;
    d.method = PLAN_METHOD_SNAPKV;
    d.table_row = r;
    d.n_old = blocks_for(L);
    if (d.n_old > max_blocks)
      return fail(plan, PLAN_EINVAL, "request %d: %d blocks exceed max_blocks_per_req %d", r,
                  d.n_old, max_blocks);
    d.q_off = (int64_t)((size_t)r * n_lh * window * pool.head_dim);
    plan->descs.push_back(d);
  }
  // longest first, so that the tail of the launch is made of short units
  std::stable_sort(plan->descs.begin(), plan->descs.end(),
                   [](const ReqDesc& x, const ReqDesc& y) { return x.seq_len > y.seq_len; });
  return PLAN_OK;
}

int plan_mlp(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
             const int32_t* img_begin, const int32_t* img_end, const int32_t* enable, int k,
             int tile_rows, MlpPlan* plan) {
  *plan = MlpPlan();
  plan->top_after = pool.n_free;
  if (n_req < 0) return fail(plan, PLAN_EINVAL, "n_req < 0");
  if (n_req == 0) return PLAN_OK;
  if (!seq_lens || !img_begin || !img_end) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (max_blocks < 1) return fail(plan, PLAN_EINVAL, "max_blocks_per_req < 1");
  if (k < 1 || tile_rows < 1) return fail(plan, PLAN_EINVAL, "bad chunk size or tile size");
  const long long n_units = (long long)pool.n_layers * pool.n_heads * 2;
  long long total_new = 0, total_old = 0;
  for (int r = 0; r < n_req; ++r) {
    if (enable && !enable[r]) continue;
    const int L = seq_lens[r], ib = img_begin[r], ie = img_end[r];
    if (L < 1 || L > kPlanMaxSeqLen)
      return fail(plan, PLAN_EINVAL, "request %d: length %d outside 1..%d", r, L, kPlanMaxSeqLen);
    if (ib < 0 || ib > ie || ie > L)
      return fail(plan, PLAN_EINVAL, "request %d: image span [%d, %d) outside [0, %d]", r, ib, ie,
                  L);
    ReqDesc d = {};
    d.seq_len = L;
    d.img_begin = ib;
    d.img_end = ie;
    d.chunks_text0 = (ib + k - 1) / k;
    d.chunks_image = (ie - ib + k - 1) / k;
    d.chunks_text1 = (L - ie + k - 1) / k;
    d.budget = d.chunks_text0 + d.chunks_image + d.chunks_text1;
    d.method = PLAN_METHOD_NONE;
    d.table_row = r;
    d.n_old = blocks_for(L);
    d.n_new = blocks_for(d.budget);
    if (d.n_old > max_blocks)
      return fail(plan, PLAN_EINVAL, "request %d: %d blocks exceed max_blocks_per_req %d", r,
                  d.n_old, max_blocks);
    d.old_off = (int32_t)total_old;
    d.new_off = (int32_t)total_new;
    total_old += d.n_old;
    total_new += d.n_new;
    const int di = (int)plan->descs.size();
    const int per_modality[2] = {d.chunks_text0 + d.chunks_text1, d.chunks_image};
    for (int m = 0; m < 2; ++m) {
      if (per_modality[m] == 0) continue;
      MlpJob j;
      j.desc = di;
      j.modality = m;
      j.chunks = per_modality[m];
      j.tile_start = (int)plan->n_tiles;
      plan->n_tiles += (n_units * per_modality[m] + tile_rows - 1) / tile_rows;
      if (plan->n_tiles > 0x7fffffffLL)
        return fail(plan, PLAN_EINVAL, "batch too large for one launch");
      plan->jobs.push_back(j);
    }
    plan->descs.push_back(d);
  }
  if (plan->descs.empty()) return PLAN_OK;
  if (total_old > 0x7fffffffLL) return fail(plan, PLAN_EINVAL, "batch too large");
  if (total_new > pool.n_free)
    return fail(plan, PLAN_ENOMEM, "batch needs %lld new blocks, %d free", total_new, pool.n_free);
  plan->total_new = (int)total_new;
  plan->total_old = (int)total_old;
  plan->top_after = pool.n_free - (int)total_new + (int)total_old;
  return PLAN_OK;
}

int plan_append(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                const int32_t* enable, DecodePlan* plan) {
  *plan = DecodePlan();
  if (n_req < 0) return fail(plan, PLAN_EINVAL, "n_req < 0");
  if (n_req == 0) return PLAN_OK;
  if (!seq_lens) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (max_blocks < 1) return fail(plan, PLAN_EINVAL, "max_blocks_per_req < 1");
  for (int r = 0; r < n_req; ++r) {
    if (enable && !enable[r]) continue;
    const int L = seq_lens[r];
    if (L < 0 || L >= kPlanMaxSeqLen)
      return fail(plan, PLAN_EINVAL, "request %d: length %d outside 0..%d", r, L,
                  kPlanMaxSeqLen - 1);
    if (L / kPlanBlockSize >= max_blocks)
      return fail(plan, PLAN_EINVAL, "request %d: its table row is full", r);
    DecodeReq q = {r, L, (L % kPlanBlockSize == 0) ? plan->n_pop++ : -1, 0, 0};
    plan->reqs.push_back(q);
  }
  if (plan->n_pop > pool.n_free)
    return fail(plan, PLAN_ENOMEM, "append needs %d new blocks, %d free", plan->n_pop,
                pool.n_free);
  return PLAN_OK;
}

int plan_decode_attention(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                          const int32_t* budget, DecodePlan* plan) {
  *plan = DecodePlan();
  if (n_req < 0) return fail(plan, PLAN_EINVAL, "n_req < 0");
  if (n_req == 0) return PLAN_OK;
  if (!seq_lens) return fail(plan, PLAN_EINVAL, "NULL argument");
  if (max_blocks < 1) return fail(plan, PLAN_EINVAL, "max_blocks_per_req < 1");
  const size_t n_lh = (size_t)pool.n_layers * pool.n_heads;
  plan->reqs.resize(n_req);
  for (int r = 0; r < n_req; ++r) {
    const int L = seq_lens[r];
    if (L < 0 || L > kPlanMaxSeqLen)
      return fail(plan, PLAN_EINVAL, "request %d: length %d outside 0..%d", r, L, kPlanMaxSeqLen);
    if (blocks_for(L) > max_blocks)
      return fail(plan, PLAN_EINVAL, "request %d: %d tokens exceed max_blocks_per_req", r, L);
    DecodeReq q = {r, L, -1, 0, 0};
    if (budget) {
      const int B = budget[r];
      if (B < 0 || B > L)
        return fail(plan, PLAN_EINVAL, "request %d: budget %d outside 0..%d", r, B, L);
      q.pop_index = B;
      q.kept_off = (int64_t)plan->kept_entries;
      plan->kept_entries += n_lh * (size_t)B;
    }
    plan->reqs[r] = q;
  }
  // longest first, so that the tail of the launch is made of short units
  std::stable_sort(plan->reqs.begin(), plan->reqs.end(),
                   [&](const DecodeReq& x, const DecodeReq& y) {
                     return budget ? x.pop_index > y.pop_index : x.seq_len > y.seq_len;
                   });
  return PLAN_OK;
}

// Heads are cut when whole ones would leave the CUs unevenly loaded: into segments of
// an eighth of a CU's share, at least 16 blocks (four for each wavefront), if that is
// at most half of the longest head, or two fifths of it where it is the share that sets
// the size: then a CU has more than three heads anyhow, and two segments a head gain less
// than their states cost (59 caches of 249-747 tokens, 24 heads of 64 channels, 31.7 us
// cut, 29.8 whole; 36 of 358-1074, 40 heads, 87.9 and 83.9; 44 of 496-744, 24 heads, 56.6
// and 57.2).  The attention alone, 32 heads, us:
//   segments at least of     8      16      24      whole
//   8 caches of 256-1408    23.7    22.8    22.9    32.6
//   1 of 4000               17.0    14.7    15.9    80.8
//   a share's            quarter  eighth  sixteenth
//   16 of 130-16384        365     353     357      417
//   12 of 4000-16000 (2 layers)  661  637  641      663
//   48 of 1280-7040 (2 layers)   957  956  973      954
// (a ninth, a tenth and a twelfth are equal to an eighth over 60 calls of 1 to 48 caches
// of 600-32000 tokens, 3 % either way in single ones).
void plan_decode_segments(const PoolView& pool, int n_cu, bool over_kept, DecodePlan* plan, int max_segments) {
  if (plan->reqs.empty()) return;
  auto blocks = [&](const DecodeReq& q) { return blocks_for(over_kept ? q.pop_index : q.seq_len); };
  const int64_t n_lh = (int64_t)pool.n_layers * pool.n_heads;
  const int64_t units = (int64_t)plan->reqs.size() * n_lh;
  int64_t total = 0;
  for (const DecodeReq& q : plan->reqs) total += blocks(q) * n_lh;
  const int longest = blocks(plan->reqs.front());  // (longest first)
  plan->seg_blocks = std::max(longest, 1);
  plan->n_seg = 1;
  const int64_t room = max_segments / units;  // segments per head
  if (room < 2) return;
  const int64_t eighth = total / (8 * (int64_t)std::max(n_cu, 1));
  const int64_t seg = std::max<int64_t>({eighth, 16, (longest + room - 1) / room});
  if (2 * seg > longest || (seg == eighth && 5 * seg > 2 * (int64_t)longest)) return;
  plan->seg_blocks = (int)seg;
  plan->n_seg = decode_segments(longest, plan->seg_blocks);
}

}  // namespace fc
