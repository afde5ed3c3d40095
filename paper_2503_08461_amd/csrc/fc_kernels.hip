// HIP kernels of the batched KV-cache compression stage, written for gfx950
// (CDNA4: 64-wide wavefronts, MFMA, 160 KB LDS per CU).
//
// Pool layout (fixed by the public ABI):
//   kv[layer][block][0=K,1=V][head][slot 0..15][d]   fp16
// so one (layer, block, kv, head) chunk is 16*d contiguous halves (4 KiB at
// d = 128) and one token row is d contiguous halves.

#include "fc_unit.h"

namespace fc {

// ---------------------------------------------------------------------------
// free stack
// ---------------------------------------------------------------------------

__global__ void stack_init_kernel(int32_t* stack, int n_blocks) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_blocks) stack[i] = n_blocks - 1 - i;
}

// ---------------------------------------------------------------------------
// ownership checks (debug mode)
// ---------------------------------------------------------------------------
//
// owner[b]: 0 = block b is on the free stack, 1 = handed out, 2 = named by a
// release that is being checked.  A release (fc_pool_free, or the reclaim of a
// compression) is checked before it is carried out: every id must be in range
// and handed out, and no id may come twice; the check claims each id with a
// compare-and-swap 1 -> 2, so a second occurrence finds 2.  The host reads the
// verdict and either lets the release go ahead (2 -> 0 as the ids are pushed)
// or takes the claims back (2 -> 1) and refuses the call.
enum { kOwnBadRange = 1, kOwnNotOwned = 2, kOwnNotFree = 4 };

__device__ __forceinline__ void owner_claim(int32_t* owner, int id, int n_blocks, int32_t* word) {
  if ((unsigned)id >= (unsigned)n_blocks) {
    atomicOr(word, kOwnBadRange);
  } else if (atomicCAS(&owner[id], 1, 2) != 1) {
    atomicOr(word, kOwnNotOwned);
  }
}

__device__ __forceinline__ void owner_unclaim(int32_t* owner, int id, int n_blocks) {
  if ((unsigned)id < (unsigned)n_blocks) atomicCAS(&owner[id], 2, 1);
}

__global__ void owner_fill_kernel(int32_t* owner, int n_blocks, int value) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_blocks) owner[i] = value;
}

__global__ void owner_mark_free_kernel(int32_t* owner, const int32_t* stack, int top, int n_blocks) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < top && (unsigned)stack[i] < (unsigned)n_blocks) owner[stack[i]] = 0;
}

__global__ void owner_check_ids_kernel(const int32_t* ids, int n, int n_blocks, int32_t* owner,
                                       int32_t* word, int revert) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (revert)
    owner_unclaim(owner, ids[i], n_blocks);
  else
    owner_claim(owner, ids[i], n_blocks, word);
}

// the table rows of the requests a compression is about to release
__global__ __launch_bounds__(kThreads) void owner_check_tables_kernel(BatchParams p, int32_t* word,
                                                                    int revert) {
  const ReqDesc rd = p.descs[blockIdx.x];
  const int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  for (int i = threadIdx.x; i < rd.n_old; i += kThreads) {
    if (revert)
      owner_unclaim(p.owner, row[i], p.n_blocks);
    else
      owner_claim(p.owner, row[i], p.n_blocks, word);
  }
}

// a popped id must have been free
__device__ __forceinline__ void owner_take(int32_t* owner, int id, int n_blocks, int32_t* flag) {
  if (!owner) return;
  if ((unsigned)id >= (unsigned)n_blocks || atomicExch(&owner[id], 1) != 0) atomicOr(flag, kOwnNotFree << 8);
}

__global__ void pool_pop_kernel(const int32_t* stack, int top, int n, int32_t* out, int32_t* owner,
                                int n_blocks, int32_t* flag) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const int id = stack[top - 1 - i];
    out[i] = id;
    owner_take(owner, id, n_blocks, flag);
  }
}

__global__ void pool_push_kernel(int32_t* stack, int top, int n, const int32_t* ids, int32_t* owner,
                                 int n_blocks) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    stack[top + i] = ids[i];
    if (owner && (unsigned)ids[i] < (unsigned)n_blocks) owner[ids[i]] = 0;  // checked before
  }
}

// Writes descriptor bytes that came as a kernel argument to device memory.
__global__ void meta_upload_kernel(MetaChunk c, char* dst, int n_bytes) {
  for (int i = threadIdx.x; i < n_bytes; i += blockDim.x) dst[i] = c.bytes[i];
}

// Pops the new blocks of every compressed request (batch order) and saves the
// pre-compression ids.  One workgroup per request; offsets are exclusive
// prefix sums computed by the host, which knows every count.
__global__ __launch_bounds__(kThreads) void plan_alloc_kernel(BatchParams p) {
  const ReqDesc rd = p.descs[blockIdx.x];
  const int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  for (int i = threadIdx.x; i < rd.n_old; i += kThreads)
    p.old_ids[rd.old_off + i] = row[i];
  if (!p.in_place)
    for (int i = threadIdx.x; i < rd.n_new; i += kThreads) {
      const int id = p.stack[p.top_before - 1 - rd.new_off - i];
      p.new_ids[rd.new_off + i] = id;
      owner_take(p.owner, id, p.n_blocks, p.error_flag);
    }
}

// Zombie reclaim: pushes the pre-compression blocks (batch order, table
// order) above the stack top left by plan_alloc and rewrites the table rows.
__global__ __launch_bounds__(kThreads) void reclaim_kernel(BatchParams p) {
  const ReqDesc rd = p.descs[blockIdx.x];
  int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  if (p.in_place) {
    // the request keeps its first n_new blocks; the rest are released
    for (int i = threadIdx.x; i < rd.n_old - rd.n_new; i += kThreads)
      p.stack[p.top_before + rd.new_off + i] = p.old_ids[rd.old_off + rd.n_new + i];
    for (int i = rd.n_new + threadIdx.x; i < p.max_blocks; i += kThreads) row[i] = -1;
    if (p.owner)  // (ids checked before the stage: in range, claimed)
      for (int i = threadIdx.x; i < rd.n_old; i += kThreads)
        p.owner[p.old_ids[rd.old_off + i]] = i < rd.n_new ? 1 : 0;
    return;
  }
  const int base = p.top_before - p.total_new;
  for (int i = threadIdx.x; i < rd.n_old; i += kThreads) {
    p.stack[base + rd.old_off + i] = p.old_ids[rd.old_off + i];
    if (p.owner) p.owner[p.old_ids[rd.old_off + i]] = 0;  // (checked before the stage)
  }
  for (int i = threadIdx.x; i < p.max_blocks; i += kThreads)
    row[i] = (i < rd.n_new) ? p.new_ids[rd.new_off + i] : -1;
}

// ---------------------------------------------------------------------------
// separate kernels (FC_SCORE_TWO_PASS, fc_window_lse): scores through HBM
// ---------------------------------------------------------------------------

template <int D, int NT>
__global__ __launch_bounds__(kThreads) void snapkv_score_kernel(BatchParams p) {
  __shared__ ScoreShared<kWaves> sh;
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_snap[slot]];
  float* raw = p.raw_scores + rd.raw_off + (size_t)lh * rd.seq_len;
  // the denominators-only call runs outside a compression: no saved ids, the table row itself
  const int32_t* ids = p.lse_out != nullptr ? p.block_tables + (size_t)rd.table_row * p.max_blocks
                                            : p.old_ids + rd.old_off;
  snapkv_unit<D, NT, kWaves>(p, rd, lh, ids, sh, [&](int j, float v) { raw[j] = v; });
}

template <int D>
__global__ __launch_bounds__(kThreads) void knorm_score_kernel(BatchParams p) {
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_knorm[slot]];
  float* raw = p.raw_scores + rd.raw_off + (size_t)lh * rd.seq_len;
  knorm_unit<D, kWaves>(p, rd, lh, p.old_ids + rd.old_off, [&](int j, float v) { raw[j] = v; });
}

// Heads of up to 32768 tokens whose scores come from a kernel of their own: 16
// wavefronts, so that a lane's share of the keys is that of a short head.
static constexpr int kSelectWaves = 16;
__global__ __launch_bounds__(64 * kSelectWaves) void select_kernel(BatchParams p) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ SelectShared<kSelectWaves> sh;
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_all[slot]];
  uint32_t* stage = lds + kStageFront;
  const float* raw = p.raw_scores + rd.raw_off + (size_t)lh * rd.seq_len;
  const int n_sel = rd.method == 1 /* FC_METHOD_SNAPKV */ ? rd.seq_len - rd.window : rd.seq_len;
  for (int j = threadIdx.x; j < n_sel; j += 64 * kSelectWaves) stage[j] = __float_as_uint(raw[j]);
  __syncthreads();
  select_unit<kSelectWaves>(p, rd, lh, stage, lds + stage_words(rd.seq_len), p.kept + rd.kept_off + (size_t)lh * rd.budget, sh);
}

template <int D>
__global__ __launch_bounds__(kThreads) void gather_kernel(BatchParams p) {
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_all[slot]];
  const int32_t* kept = p.kept + rd.kept_off + (size_t)lh * rd.budget;
  gather_unit<D, kWaves>(p, rd, lh, [&](int i) { return p.old_ids[rd.old_off + i]; },
                         [&](int t) { return kept[t]; });
}

// a fill kernel for small device arrays (flags, verdict words): calls may be
// captured into a graph, where a memset node is not wanted
__global__ void zero_ints_kernel(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t kernels_one_time_setup() {
  // kernels that may need more than the default 64 KiB of dynamic LDS
  // (the narrow fused kernels never do)
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(select_kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (stage_words(32768) + need_words(32768)) * 4);
  if (e == hipSuccess) e = fused_wide_setup_64();
  if (e == hipSuccess) e = fused_wide_setup_128();
  return e;
}

hipError_t launch_stack_init(int32_t* stack, int n_blocks, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  stack_init_kernel<<<(n_blocks + 255) / 256, 256, 0, s>>>(stack, n_blocks);
  return hipGetLastError();
}

hipError_t launch_pool_pop(const int32_t* stack, int top, int n, int32_t* out, int32_t* owner,
                           int n_blocks, int32_t* flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  pool_pop_kernel<<<(n + 255) / 256, 256, 0, s>>>(stack, top, n, out, owner, n_blocks, flag);
  return hipGetLastError();
}

hipError_t launch_pool_push(int32_t* stack, int top, int n, const int32_t* ids, int32_t* owner,
                            int n_blocks, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  pool_push_kernel<<<(n + 255) / 256, 256, 0, s>>>(stack, top, n, ids, owner, n_blocks);
  return hipGetLastError();
}

hipError_t launch_owner_init(int32_t* owner, const int32_t* stack, int top, int n_blocks,
                             hipStream_t s) {
  owner_fill_kernel<<<(n_blocks + 255) / 256, 256, 0, s>>>(owner, n_blocks, 1);
  if (top > 0) owner_mark_free_kernel<<<(top + 255) / 256, 256, 0, s>>>(owner, stack, top, n_blocks);
  return hipGetLastError();
}

hipError_t launch_owner_check_ids(const int32_t* ids, int n, int n_blocks, int32_t* owner,
                                  int32_t* word, bool revert, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  owner_check_ids_kernel<<<(n + 255) / 256, 256, 0, s>>>(ids, n, n_blocks, owner, word,
                                                         revert ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_owner_check_tables(const BatchParams& p, int32_t* word, bool revert,
                                     hipStream_t s) {
  if (p.n_comp <= 0) return hipSuccess;
  owner_check_tables_kernel<<<p.n_comp, kThreads, 0, s>>>(p, word, revert ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_meta_upload(const MetaChunk& c, char* dst, int n_bytes, hipStream_t s) {
  if (n_bytes <= 0) return hipSuccess;
  if (n_bytes > (int)sizeof(MetaChunk)) return hipErrorInvalidValue;
  meta_upload_kernel<<<1, 256, 0, s>>>(c, dst, n_bytes);
  return hipGetLastError();
}

hipError_t launch_plan_alloc(const BatchParams& p, hipStream_t s) {
  plan_alloc_kernel<<<p.n_comp, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_reclaim(const BatchParams& p, hipStream_t s) {
  reclaim_kernel<<<p.n_comp, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_snapkv_d(const BatchParams& p, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_snap * p.n_layers * p.n_heads;
  const int nt = (p.window + 15) / 16;
  switch (nt) {
    case 1: snapkv_score_kernel<D, 1><<<grid, kThreads, 0, s>>>(p); break;
    case 2: snapkv_score_kernel<D, 2><<<grid, kThreads, 0, s>>>(p); break;
    case 3: snapkv_score_kernel<D, 3><<<grid, kThreads, 0, s>>>(p); break;
    case 4: snapkv_score_kernel<D, 4><<<grid, kThreads, 0, s>>>(p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_snapkv_score(const BatchParams& p, hipStream_t s) {
  if (p.n_snap == 0) return hipSuccess;
  if (p.head_dim == 128) return launch_snapkv_d<128>(p, s);
  if (p.head_dim == 64) return launch_snapkv_d<64>(p, s);
  return hipErrorInvalidValue;
}

hipError_t launch_knorm_score(const BatchParams& p, hipStream_t s) {
  if (p.n_knorm == 0) return hipSuccess;
  const unsigned grid = (unsigned)p.n_knorm * p.n_layers * p.n_heads;
  if (p.head_dim == 128)
    knorm_score_kernel<128><<<grid, kThreads, 0, s>>>(p);
  else if (p.head_dim == 64)
    knorm_score_kernel<64><<<grid, kThreads, 0, s>>>(p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_select(const BatchParams& p, int max_seq_len, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_unfused * p.n_layers * p.n_heads;
  const size_t lds = (size_t)(stage_words(max_seq_len) + need_words(max_seq_len)) * sizeof(uint32_t);
  select_kernel<<<grid, 64 * kSelectWaves, lds, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_fused(BatchParams p, bool any_snap, int max_seq_len, int max_blocks, bool wide,
                        hipStream_t s) {
  if (p.n_fused == 0) return hipSuccess;
  if (max_seq_len > (wide ? kFusedWideMaxLen : kFusedMaxLen)) return hipErrorInvalidValue;
  const FusedLds f = fused_lds(max_seq_len, max_blocks, wide);
  p.ids_at = f.ids_at;
  p.ids_room = f.ids_room;
  const size_t lds = (size_t)f.words * sizeof(uint32_t);
  const int tiles = any_snap ? (p.window + 15) / 16 : 0;
  if (p.head_dim == 128)
    return wide ? launch_fused_wide_128(p, tiles, lds, s) : launch_fused_narrow_128(p, tiles, lds, s);
  if (p.head_dim == 64)
    return wide ? launch_fused_wide_64(p, tiles, lds, s) : launch_fused_narrow_64(p, tiles, lds, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gather(const BatchParams& p, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_unfused * p.n_layers * p.n_heads;
  if (p.head_dim == 128)
    gather_kernel<128><<<grid, kThreads, 0, s>>>(p);
  else if (p.head_dim == 64)
    gather_kernel<64><<<grid, kThreads, 0, s>>>(p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_zero_ints(int32_t* p, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  zero_ints_kernel<<<(n + 255) / 256, 256, 0, s>>>(p, n);
  return hipGetLastError();
}

}  // namespace fc
