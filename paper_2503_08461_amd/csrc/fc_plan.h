// Host-side planning of libfastcache's batched calls: validation with what the
// host scheduler knows (lengths, methods, budgets, free-block count), prefix
// sums of block counts, request descriptors and work lists.  Plain C++ with no
// HIP in it: fc_api.hip turns a plan into launches, and the CPU tests build
// this file with the host sanitizers and drive it on its own.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "fc_types.h"

namespace fc {

// Result codes and limits, numerically those of include/fastcache.h (the
// translation unit that includes both checks it).
enum { PLAN_OK = 0, PLAN_EINVAL = -1, PLAN_ENOMEM = -2 };
enum { PLAN_METHOD_NONE = 0, PLAN_METHOD_SNAPKV = 1, PLAN_METHOD_KNORM = 2, PLAN_METHOD_STREAMING = 3 };
enum { PLAN_SCORE_AUTO = 0, PLAN_SCORE_TWO_PASS = 1 };
static constexpr int kPlanBlockSize = 16;
static constexpr int kPlanMaxWindow = 64;
static constexpr int kPlanMaxSeqLen = 32768;
static constexpr int kPlanMaxPoolKernel = 63;
static constexpr int kPlanFusedMaxLen = 8192;   // longest head of narrow workgroups of the fused kernels
static constexpr int kPlanClasses = 5;          // query-tile counts 0..4 (0: no queries)

// LDS of a head's per-token words: stage[0 .. n) plus room in front and behind
// that the four-token reads of the pooling may touch (filled with what changes no
// result), then one bit per token.
static constexpr int kChunk = 256;  // tokens a wavefront takes at a time (4 per lane)
static constexpr int kStageFront = 4;
constexpr int stage_words(int len) { return kStageFront + ((len + 3) & ~3) + 8; }
constexpr int need_words(int len) { return (len + kChunk - 1) / kChunk * (kChunk / 32); }

// LDS words of a fused launch: scores, then one bit per token, then the block ids.
struct FusedLds {
  int ids_at, ids_room, words;
};
constexpr FusedLds fused_lds(int max_len, int max_blocks, bool wide) {
  FusedLds f = {};
  f.ids_at = stage_words(max_len) + need_words(max_len);
  const int most = (wide ? kPlanMaxSeqLen : kPlanFusedMaxLen) / kPlanBlockSize;
  f.ids_room = max_blocks < most ? max_blocks : most;
  f.words = f.ids_at + ((f.ids_room + 3) & ~3);
  return f;
}
// Of narrow workgroups, three and more query tiles: the words up to which a CU takes as
// many of the kernel that leaves half of the keys to the caches as of the plain one.
static constexpr int kPlanHalfReuseWords = 8572;

// What the pool contributes to a plan.
struct PoolView {
  int n_layers = 0, n_heads = 0, head_dim = 0;
  int n_free = 0;                       // free blocks on entry
  int score_mode = PLAN_SCORE_AUTO;
  bool in_place = false;
};

// The caller's arguments of fc_compress_batch / _var / _lse, pointers reduced
// to what validation needs.
struct CompressArgs {
  int n_req = 0, max_blocks = 0;
  const int32_t* seq_lens = nullptr;    // [n_req]
  const int32_t* method = nullptr;      // [n_req]
  const int32_t* budget = nullptr;      // [n_req]
  const int32_t* window_per_req = nullptr;       // [n_req] or NULL: `window` for all
  const int32_t* pool_kernel_per_req = nullptr;  // [n_req] or NULL: `pool_kernel` for all
  int window = 0, pool_kernel = 0;
  bool need_lse = false;
  bool q_ok = false;                    // dev_q_window non-NULL and 16-byte aligned
  bool lse_ok = false;                  // dev_lse_window non-NULL and 4-byte aligned
};

// Work lists of a compress call (descriptor indices, heaviest first).
enum {
  // (in the default scheduling the lists after the first hold the heads that only wide
  // workgroups of the fused kernels take, see plan_fused_launches)
  LIST_FUSED = 0,                  // + class: units of the fused kernels, per query-tile count
  LIST_SNAP = kPlanClasses,        // + class: separate two-pass score kernel
  LIST_KNORM = 2 * kPlanClasses,   // separate key-norm score kernel
  LIST_ALL,                        // select and gather of the separate path
  N_LISTS
};

struct CompressPlan {
  int code = PLAN_OK;
  char message[256] = "";
  std::vector<ReqDesc> descs;                 // compressed requests, batch order
  std::vector<int64_t> weights;               // per descriptor: what its units move, in rows
  std::vector<int32_t> lists[N_LISTS];
  int max_len[N_LISTS] = {};
  int total_new = 0, total_old = 0, total_released = 0;
  int window_hi = 0;                          // largest window of a SnapKV request
  size_t kept_entries = 0;                    // ints of the kept buffer
  size_t score_entries = 0;                   // floats of a packed scores_out
  size_t raw_floats = 0;                      // floats of un-pooled score scratch (separate or split kernels)
  int top_after = 0;                          // free blocks after the call
};

// Fills `plan`; returns plan->code.  On an error nothing else in the plan is
// meaningful.  A batch with nothing to compress gives PLAN_OK and no descs.
int plan_compress(const PoolView& pool, const CompressArgs& args, CompressPlan* plan);

// Lengths from which a fused launch of `heads` heads prunes the second pass of its SnapKV
// heads, by the query tiles of their windows (fc_plan.cpp has the times of both sides).
struct PruneFrom {
  int32_t tiles[kPlanClasses - 1];  // of 1..4
};
PruneFrom plan_prune_from(int head_dim, bool wide, size_t heads, int n_cu);

// The launches of the fused kernels (score -> select -> gather in one workgroup
// per unit) of a planned call, heaviest unit first in each.
struct FusedLaunch {
  std::vector<int32_t> units;  // descriptor indices
  int query_tiles = 0;         // 16-row query tiles of its SnapKV units (0: it holds none, 5: they differ)
  bool wide = false;           // wide workgroups, one per CU
  int max_len = 0;             // longest head that is scored
  int max_blocks = 0;          // most blocks of a unit
  bool half_reuse = false;     // long heads: a pruned first pass leaves only half of the keys to the caches
  PruneFrom prune_from = {};
};
std::vector<FusedLaunch> plan_fused_launches(const PoolView& pool, const CompressPlan& plan, int n_cu);

// Whether a call in the default scheduling that is not split needs no plan_alloc: one request
// in one launch whose kernels read the table and the stack themselves (pruned: the call asks
// for no scores and gives no log-sum-exps).
bool plan_one_launch(const PoolView& pool, const CompressPlan& plan, size_t n_launches, bool pruned);
// Most block ids, old and new, of such a request: the wavefront that takes its old blocks
// back keeps them in LDS.
static constexpr int kPlanOnlyMaxIds = 512;

// A call with so few heads that they are better split over workgroups: segments
// per head, or 0 (not split).  Otherwise all requests of the call run that way;
// plan->descs get their offsets in the score scratch, plan->raw_floats its size.
int plan_split(const PoolView& pool, int n_cu, CompressPlan* plan);

// Whether the select kernel of `units` heads of at most max_len tokens takes 16 wavefronts a head.
bool select_is_wide(int max_len, size_t units, int n_cu);

// fc_window_lse: one descriptor per SnapKV request (all if method is NULL),
// longest first, queries packed as [n_req][...][window].
struct LsePlan {
  int code = PLAN_OK;
  char message[256] = "";
  std::vector<ReqDesc> descs;
};
int plan_window_lse(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                    const int32_t* method, int window, LsePlan* plan);

// fc_compress_batch_mlp.
struct MlpPlan {
  int code = PLAN_OK;
  char message[256] = "";
  std::vector<ReqDesc> descs;
  std::vector<MlpJob> jobs;
  int total_new = 0, total_old = 0;
  long long n_tiles = 0;
  int top_after = 0;
};
int plan_mlp(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
             const int32_t* img_begin, const int32_t* img_end, const int32_t* enable, int k,
             int tile_rows, MlpPlan* plan);

// fc_append_batch and the decode attentions.
struct DecodePlan {
  int code = PLAN_OK;
  char message[256] = "";
  std::vector<DecodeReq> reqs;
  int n_pop = 0;
  size_t kept_entries = 0;
  // attention: blocks per segment of a head, segments of the longest one (no head has more)
  int seg_blocks = 0, n_seg = 1;
};
// Attention: most segments of all heads of a call that is split (heads x n_seg), which
// is what the pool's buffers for their states hold (10.5 MB at 128 channels).
static constexpr int kMaxDecodeSegments = 16384;
// Segments of a head of `blocks` blocks in a call that cuts its heads: as many of
// seg_blocks as come nearest (1 for a short or empty head), all alike in size; segment s
// begins at block decode_segment_begin(blocks, n, s) and ends where the next one does.
constexpr int decode_segments(int blocks, int seg_blocks) {
  const int n = (blocks + seg_blocks / 2) / seg_blocks;
  return n > 1 ? n : 1;
}
constexpr int decode_segment_begin(int blocks, int n, int s) { return blocks * s / n; }
int plan_append(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                const int32_t* enable, DecodePlan* plan);
int plan_decode_attention(const PoolView& pool, int n_req, int max_blocks, const int32_t* seq_lens,
                          const int32_t* budget /* NULL: whole cache */, DecodePlan* plan);
// Sets seg_blocks and n_seg of a planned attention (over_kept: of the kept lists);
// max_segments: of all heads, kMaxDecodeSegments or 0 (a pool without the buffers).
void plan_decode_segments(const PoolView& pool, int n_cu, bool over_kept, DecodePlan* plan,
                          int max_segments = kMaxDecodeSegments);

}  // namespace fc
