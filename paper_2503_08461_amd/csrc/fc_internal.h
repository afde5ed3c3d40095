// Internal declarations shared by the host API and the kernel launchers of
// libfastcache.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fc_plan.h"

namespace fc {

struct MlpParams {
  const MlpJob* jobs;
  int32_t n_jobs, n_tiles;
  int32_t max_grid;    // workgroups to launch at most (as many as are resident)
  int32_t k, hidden;
  int32_t activation;  // FC_ACT_*
  // weights in operand order, index 0 text / 1 image; w2p[m] starts where w1p[m] ends
  const _Float16* w1p[2];
  const _Float16* w2p[2];
  const float* b1[2];
  const float* b2[2];
};

// Requests of a decode step that travel as kernel arguments, up to kInline of them:
// a copy through pinned memory costs the stream a copy kernel and 10 to 20 us of
// idle time on either side, and the host has to wait until the last one is through.
struct DecodeReqs {
  static constexpr int kInline = 3584 / sizeof(DecodeReq);  // 149
  DecodeReq req[kInline];
};
struct DecodeReqList {  // requests on the device
  const DecodeReq* req;
};
static_assert(sizeof(DecodeReq) == 24, "tests count on the sizes of descriptors and argument blocks");
static constexpr size_t kMaxArgumentBytes = 4096;  // what the arguments of a kernel may take

struct DecodeParams {
  _Float16* kv;
  int32_t n_blocks, n_layers, n_heads, head_dim;
  const int32_t* stack;  // free stack (append: new blocks are stack[top_before - 1 - pop_index])
  int32_t top_before;
  int32_t* block_tables;
  int32_t max_blocks;
  const DecodeReq* reqs;  // NULL: the requests are in the DecodeReqs argument
  int32_t n_req;
  const _Float16* new_kv;  // append: [row][layer][2][head][d]
  const _Float16* q;       // attention: [row][layer][head][d]
  float* out;              // attention: [row][layer][head][d]
  const int32_t* kept;     // attention over kept lists of an uncompacted cache, else NULL
  float scale_log2e;
  // attention: blocks per segment of a head, segments of the longest one (1: no head is cut)
  int32_t seg_blocks, n_seg;
  float* partial;          // [n_req * layers * heads][n_seg][state_words] states of the segments
  int32_t* owner;          // ownership checks (debug mode), else NULL
  int32_t* error_flag;
  // (whole cache lines: the states of one head's last segment and the next one's first come
  // from different XCDs.  8 caches of 560-620 tokens, two segments each: 16.9 us with head_dim
  // + 4 words, where they share a line, 16.2 so)
  static constexpr int state_words(int head_dim) { return head_dim + 32; }
};
static_assert(sizeof(DecodeParams) + sizeof(DecodeReqs) <= kMaxArgumentBytes, "decode kernels");

// Everything a kernel of the stage needs.  Passed by value.
struct BatchParams {
  // pool geometry
  _Float16* kv;        // kv[layer][block][2][head][16][d]
  int32_t n_blocks, n_layers, n_heads, head_dim;
  // free stack
  int32_t* stack;
  int32_t top_before;  // top on entry to the call
  int32_t total_new;   // sum of n_new
  int32_t total_old;   // sum of n_old
  // batch
  const ReqDesc* descs;        // [n_comp] in batch order
  const int32_t* order_all;    // [n_comp] desc indices, longest first
  const int32_t* order_snap;   // [n_snap]
  const int32_t* order_knorm;  // [n_knorm]
  const int32_t* order_fused;  // [n_fused] units handled by the fused kernel (both methods)
  int32_t n_comp, n_snap, n_knorm, n_unfused, n_fused;
  int32_t* block_tables;       // caller's [n_req][max_blocks]
  int32_t max_blocks;
  int32_t* old_ids;            // [total_old] saved pre-compression ids
  int32_t* new_ids;            // [total_new]
  const _Float16* q_window;
  const float* lse_window;     // nullable: natural log-sum-exp of every window row, packed like
                               // q_window without the channel axis; pass 1 is skipped
  float* lse_out;              // nullable: write that quantity (from pass 1) and stop
  int32_t window;              // a bound on the windows of this launch's SnapKV units (picks the
                               // number of 16-row query tiles); the unit's own is in its descriptor
  int32_t n_sink;              // leading tokens kept by streaming requests
  int32_t in_place;            // 1: compact inside the request's own blocks
  float scale_log2e;           // scale * log2(e)
  float* raw_scores;           // un-pooled scores of the units that take the separate kernels
  float* scores_out;           // nullable
  int32_t* kept;               // kept indices, packed, of the units that take the separate kernels
  int32_t* kept_out;           // nullable: the caller's copy of them, written by the fused kernels
  int32_t* error_flag;         // set if a kernel finds something wrong (an ownership check that fails)
  int32_t n_split;             // heads split over workgroups: segments per head (1: gather of the
                               // separate kernels)
  float* split_part;           // ... [unit][segment][2][64]: the segments' row (max, sum) pairs
  int32_t ids_at, ids_room;    // fused kernels: where the block ids lie in LDS (words), room for how many
  int32_t main_reclaims;       // 1: the last kernel of the stage does what reclaim_kernel would
  int32_t bounded;             // 1: the fused kernel prunes the second pass of its SnapKV units
  int32_t half_reuse;          // ... and leaves only half of the keys that it reads first to the caches
  PruneFrom prune_from;        // ... and prunes heads of these lengths and more
  int32_t* owner;              // ownership checks (debug mode): [n_blocks] 0 free, 1 handed out,
                               // 2 being released; NULL when the checks are off
  // A call of one request whose only launch is a fused one (plan_one_launch): its descriptor;
  // `arrivals` counts the workgroups that are done with the table and the stack, and is
  // zero between calls.  NULL: plan_alloc has run, descriptors and ids are in the buffers above.
  int32_t* arrivals;
  int32_t new_ids_at;          // ... and where the new block ids lie in LDS (words)
  struct Only {  // (of a ReqDesc what isn't zero then)
    int32_t seq_len, budget, method, table_row, n_old, n_new, window, pool_kernel;
    int64_t q_off;
  } only;
};
static constexpr int kOnlyMaxIds = kPlanOnlyMaxIds;

// Descriptor bytes that travel as a kernel argument.
struct MetaChunk {
  alignas(16) char bytes[3584];
};
static_assert(sizeof(BatchParams) + sizeof(MetaChunk) + 32 <= kMaxArgumentBytes, "plan_alloc_inline_kernel");

enum KernelSlot {
  K_PLAN_ALLOC = 0,
  K_SNAPKV_SCORE = 1,
  K_KNORM_SCORE = 2,
  K_SELECT = 3,
  K_GATHER = 4,
  K_RECLAIM = 5,
  K_FUSED = 6,
  K_MLP = 7,
  K_APPEND = 8,
  K_DECODE_ATTENTION = 9,
  K_WINDOW_LSE = 10,
  K_COUNT = 11
};

// Launchers (fc_kernels.hip).  Each returns the hipError_t of the launch.
hipError_t launch_stack_init(int32_t* stack, int n_blocks, hipStream_t s);
// owner / flag: ownership checks (debug mode), NULL when off
hipError_t launch_pool_pop(const int32_t* stack, int top, int n, int32_t* out, int32_t* owner,
                           int n_blocks, int32_t* flag, hipStream_t s);
hipError_t launch_pool_push(int32_t* stack, int top, int n, const int32_t* ids, int32_t* owner,
                            int n_blocks, hipStream_t s);
// owner[b] = 1, then 0 for the blocks on the free stack
hipError_t launch_owner_init(int32_t* owner, const int32_t* stack, int top, int n_blocks,
                             hipStream_t s);
// claim (or, revert: give back) the ids of a release; *word collects what was wrong
hipError_t launch_owner_check_ids(const int32_t* ids, int n, int n_blocks, int32_t* owner,
                                  int32_t* word, bool revert, hipStream_t s);
hipError_t launch_owner_check_tables(const BatchParams& p, int32_t* word, bool revert,
                                     hipStream_t s);
// inline_meta (nullable): the n_bytes of descriptors and lists that the kernel writes
// to p.descs before anything else reads them
hipError_t launch_plan_alloc(const BatchParams& p, const MetaChunk* inline_meta, int n_bytes, hipStream_t s);
hipError_t launch_snapkv_score(const BatchParams& p, hipStream_t s);
// a fill kernel (not a memset: calls may be captured into a graph)
hipError_t launch_zero_ints(int32_t* p, int n, hipStream_t s);
hipError_t launch_knorm_score(const BatchParams& p, hipStream_t s);
// scores of heads split over workgroups (order_all; select and gather follow)
hipError_t launch_split_scores(const BatchParams& p, hipStream_t s);
// wide: workgroups for heads of more than kFusedMaxLen tokens and for few heads
hipError_t launch_select(const BatchParams& p, int max_seq_len, bool wide, hipStream_t s);
hipError_t launch_gather(const BatchParams& p, hipStream_t s);
// score -> select -> gather of every unit of order_fused in one launch.
// max_seq_len: longest head that is scored, at most kFusedMaxLen (kFusedWideMaxLen
// with wide workgroups); max_blocks: most blocks of any of the units; query_tiles:
// 16-row tiles of its SnapKV units (0: none, 5: of several classes)
hipError_t launch_fused(BatchParams p, int query_tiles, int max_seq_len, int max_blocks, bool wide,
                        hipStream_t s);
// (per head size and workgroup shape; lds: dynamic LDS bytes)
hipError_t launch_fused_narrow_64(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s);
hipError_t launch_fused_narrow_128(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s);
hipError_t launch_fused_wide_64(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s);
hipError_t launch_fused_wide_128(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s);
hipError_t fused_wide_setup_64();
hipError_t fused_wide_setup_128();
static constexpr int kFusedMaxLen = 8192;
static constexpr int kFusedWideMaxLen = 32768;
hipError_t launch_reclaim(const BatchParams& p, hipStream_t s);
hipError_t launch_meta_upload(const MetaChunk& c, char* dst, int n_bytes, hipStream_t s);
hipError_t kernels_one_time_setup();
// decode-side pool traffic (fc_decode.hip)
hipError_t launch_append(const DecodeParams& p, const DecodeReqs& inline_reqs, hipStream_t s);
hipError_t launch_decode_attention(const DecodeParams& p, const DecodeReqs& inline_reqs, hipStream_t s);
// chunk-MLP compressor (fc_mlp.hip)
hipError_t mlp_one_time_setup();
size_t mlp_w1p_elems(int head_dim, int hidden, int k);
size_t mlp_w2p_elems(int head_dim, int hidden);
int mlp_rows_per_tile(int head_dim, int hidden);  // rows (units x chunks) one workgroup takes at a time
int mlp_workgroups_per_cu(int head_dim, int hidden);
hipError_t launch_mlp_permute_weights(const _Float16* w1, const _Float16* w2, _Float16* w1p,
                                      _Float16* w2p, int head_dim, int hidden, int k,
                                      hipStream_t s);
hipError_t launch_mlp_compress(const BatchParams& p, const MlpParams& mp, hipStream_t s);

}  // namespace fc
