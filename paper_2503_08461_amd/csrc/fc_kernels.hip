// HIP kernels of the batched KV-cache compression stage, written for gfx950
// (CDNA4: 64-wide wavefronts, MFMA, 160 KB LDS per CU).
//
// Pool layout (fixed by the public ABI):
//   kv[layer][block][0=K,1=V][head][slot 0..15][d]   fp16
// so one (layer, block, kv, head) chunk is 16*d contiguous halves (4 KiB at
// d = 128) and one token row is d contiguous halves.

#include <algorithm>

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
__device__ __forceinline__ void write_meta(const MetaChunk& c, char* dst, int n_bytes) {
  // (dst and n_bytes are multiples of 16)
  for (int i = threadIdx.x; i < n_bytes / 16; i += blockDim.x)
    reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(c.bytes)[i];
}
__global__ void meta_upload_kernel(MetaChunk c, char* dst, int n_bytes) {
  write_meta(c, dst, n_bytes);
}

// Pops the new blocks of every compressed request (batch order) and saves the
// pre-compression ids.  One workgroup per request; offsets are exclusive
// prefix sums computed by the host, which knows every count.
__device__ __forceinline__ void plan_alloc_request(const BatchParams& p, const ReqDesc& rd) {
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
__global__ __launch_bounds__(kThreads) void plan_alloc_kernel(BatchParams p) {
  plan_alloc_request(p, p.descs[blockIdx.x]);
}
// The same with the descriptors in its arguments, from where they go to device
// memory for the kernels that follow: a small call has no copy of its own in the
// stream (a copy through pinned memory left the GPU idle for 20 to 40 us, most of
// it the host's wait for the staging buffer; a launch costs about 4.5 us).
__global__ __launch_bounds__(kThreads) void plan_alloc_inline_kernel(BatchParams p, MetaChunk c, char* meta,
                                                                     int n_bytes) {
  plan_alloc_request(p, reinterpret_cast<const ReqDesc*>(c.bytes)[blockIdx.x]);
  if (blockIdx.x == 0) write_meta(c, meta, n_bytes);
}

__global__ __launch_bounds__(kThreads) void reclaim_kernel(BatchParams p) { reclaim_request(p, p.descs[blockIdx.x]); }

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
  snapkv_unit<D, NT, kWaves, false>(p, rd, lh, ids, sh, [&](int j, float v) { raw[j] = v; });
}

template <int D>
__global__ __launch_bounds__(kThreads) void knorm_score_kernel(BatchParams p) {
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_knorm[slot]];
  float* raw = p.raw_scores + rd.raw_off + (size_t)lh * rd.seq_len;
  knorm_unit<D, kWaves>(p, rd, lh, p.old_ids + rd.old_off, 0, rd.n_old, [&](int j, float v) { raw[j] = v; });
}

// ---------------------------------------------------------------------------
// heads split over workgroups
// ---------------------------------------------------------------------------
//
// A call with few heads (one layer, one or two requests) leaves most CUs idle in
// the fused kernels, and one CU gets no more than about 27 GB/s out of HBM
// whatever its wavefronts have in flight (16 wavefronts: 64 KB per 5600 cycles).
// So the heads of such a call are cut into p.n_split segments of whole blocks, one
// workgroup each:
//   split_rows    row (max, sum) pairs of the segment -> p.split_part; key norms
//   split_scores  the rows' denominators from all segments' pairs, then the
//                 segment's column sums (K again, by then mostly from the
//                 memory-side cache)
//   select        one workgroup per head
//   gather        the kept blocks, cut into p.n_split segments as well
static constexpr int kSplitIds = 2048;  // blocks of the longest head

struct SplitUnit {
  int unit, seg, lh;
  ReqDesc rd;
};
__device__ __forceinline__ SplitUnit split_unit(const BatchParams& p) {
  SplitUnit u;
  const int n_lh = p.n_layers * p.n_heads;
  u.unit = blockIdx.x / p.n_split;
  u.seg = blockIdx.x - u.unit * p.n_split;
  const int slot = u.unit / n_lh;
  u.lh = u.unit - slot * n_lh;
  u.rd = p.descs[p.order_all[slot]];
  return u;
}
// segment of [0, n): [first, last)
__device__ __forceinline__ void split_range(const BatchParams& p, int seg, int n, int& first, int& last) {
  const int per = (n + p.n_split - 1) / p.n_split;
  first = min(n, seg * per);
  last = min(n, first + per);
}

template <int D, int NT>
__global__ __launch_bounds__(kThreads) void split_rows_kernel(BatchParams p) {
  __shared__ ScoreShared<kWaves> sh;
  __shared__ int32_t sm_ids[kSplitIds];
  const SplitUnit u = split_unit(p);
  int b0, b1;
  split_range(p, u.seg, u.rd.n_old, b0, b1);
  const bool snap = u.rd.method == 1 /* FC_METHOD_SNAPKV */;
  if (u.rd.method == 3 /* FC_METHOD_STREAMING */ || (snap && p.lse_window != nullptr)) return;  // uniform
  for (int i = b0 + threadIdx.x; i < b1; i += kThreads) sm_ids[i] = p.old_ids[u.rd.old_off + i];
  __syncthreads();
  if (snap) {
    if constexpr (NT > 0) {
      half8 qreg[NT][D / 32];
      load_window_queries<D, NT>(p, u.rd, u.lh, qreg);
      snapkv_rows<D, NT, kWaves, false>(p, u.rd, u.lh, sm_ids, b0, b1, sh, qreg);
      __syncthreads();
      if (threadIdx.x < 16 * NT) {
        float mm, zz;
        merged_row<kWaves>(sh, threadIdx.x, mm, zz);
        float* part = p.split_part + ((size_t)u.unit * p.n_split + u.seg) * 128;
        part[threadIdx.x] = mm;
        part[64 + threadIdx.x] = zz;
      }
    }
  } else {
    float* raw = p.raw_scores + u.rd.raw_off + (size_t)u.lh * u.rd.seq_len;
    knorm_unit<D, kWaves>(p, u.rd, u.lh, sm_ids, b0, b1, [&](int j, float v) { raw[j] = v; });
  }
}

template <int D, int NT>
__global__ __launch_bounds__(kThreads) void split_scores_kernel(BatchParams p) {
  __shared__ float fin[64];
  __shared__ KeyTiles<kWaves> tiles;
  __shared__ int32_t sm_ids[kSplitIds];
  const SplitUnit u = split_unit(p);
  if (u.rd.method != 1 /* FC_METHOD_SNAPKV */) return;  // uniform
  int b0, b1;
  split_range(p, u.seg, (u.rd.seq_len - u.rd.window + 15) >> 4, b0, b1);
  for (int i = b0 + threadIdx.x; i < b1; i += kThreads) sm_ids[i] = p.old_ids[u.rd.old_off + i];
  const int row = threadIdx.x;
  if (row < 64) {
    float out = INFINITY;  // padded rows contribute exp2(-inf) = 0
    if (row < u.rd.window) {
      if (p.lse_window != nullptr) {
        out = p.lse_window[lse_offset<D>(u.rd, u.lh) + row] * 1.44269504088896340736f;
      } else {
        const float* part = p.split_part + (size_t)u.unit * p.n_split * 128 + row;
        float mm = -3.0e38f, zz = 0.f;
        for (int g = 0; g < p.n_split; ++g) mm = fmaxf(mm, part[g * 128]);
        for (int g = 0; g < p.n_split; ++g) zz += part[g * 128 + 64] * __builtin_amdgcn_exp2f(part[g * 128] - mm);
        out = mm + log2f(zz);
      }
    }
    fin[row] = out;
  }
  half8 qreg[NT][D / 32];
  load_window_queries<D, NT>(p, u.rd, u.lh, qreg);
  __syncthreads();
  float* raw = p.raw_scores + u.rd.raw_off + (size_t)u.lh * u.rd.seq_len;
  snapkv_columns<D, NT, kWaves, false>(p, u.rd, u.lh, sm_ids, b0, b1, fin, tiles, qreg,
                                       [&](int j, float v) { raw[j] = v; });
}

// Heads whose scores come from a kernel of their own.  16 wavefronts for heads of up
// to 32768 tokens and for launches with few heads, so that a lane's share of the keys
// is that of a short head; 4, of which a CU holds several workgroups, for the rest.
static constexpr int kSelectWaves = 16;
template <int WV>
__global__ __launch_bounds__(64 * WV) void select_kernel(BatchParams p) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ SelectShared<WV> sh;
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = p.descs[p.order_all[slot]];
  uint32_t* stage = lds + kStageFront;
  int32_t* kept = p.kept + rd.kept_off + (size_t)lh * rd.budget;
  if (rd.method == 3 /* FC_METHOD_STREAMING */) {  // uniform (heads split over workgroups only)
    streaming_unit<WV>(p, rd, lh, kept);
    return;
  }
  const float* raw = p.raw_scores + rd.raw_off + (size_t)lh * rd.seq_len;
  const int n_sel = rd.method == 1 /* FC_METHOD_SNAPKV */ ? rd.seq_len - rd.window : rd.seq_len;
  for (int j = threadIdx.x; j < n_sel; j += 64 * WV) stage[j] = __float_as_uint(raw[j]);
  __syncthreads();
  select_unit<WV>(p, rd, lh, stage, lds + stage_words(rd.seq_len), kept, sh);
}

// The copy of heads whose selection was a kernel of its own.  A wavefront takes its blocks
// four at a time, a lane for each of their rows: what goes there, then where that lies; of
// the next four both are on their way before the rows of these are asked for, and no load
// stands between the rows asked for and those that are stored.  (Each id and kept token
// loaded where it was used, 18 loads a block, all of them waited for with the rows: 64 heads
// of 4000 tokens 58.5 -> 57.0 us, the whole call; the split kernels' loops alone 58.3; 64
// channels 45.4 -> 44.0; 3072 heads whole, 1000-3000 tokens, 923 -> 917 and 459 -> 464.)
template <int D>
__global__ __launch_bounds__(kThreads) void gather_kernel(BatchParams p) {
  const SplitUnit u = split_unit(p);
  if (p.main_reclaims && u.lh == 0 && u.seg == 0) reclaim_request(p, u.rd);
  const int32_t* kept = p.kept + u.rd.kept_off + (size_t)u.lh * u.rd.budget;
  const int32_t* old_ids = p.old_ids + u.rd.old_off;
  const int32_t* new_ids = p.new_ids + u.rd.new_off;
  if (p.in_place) {  // (a head is not split then)
    gather_unit<D, kWaves, false>(
        p, u.rd, u.lh, [&](int i) { return old_ids[i]; }, [&](int i) { return new_ids[i]; }, [&](int t) { return kept[t]; });
    return;
  }
  int nb0, nb1;
  split_range(p, u.seg, u.rd.n_new, nb0, nb1);
  const RowCopy<D, kWaves> c(p, u.rd, u.lh, nb0);
  typedef typename RowCopy<D, kWaves>::Rows Rows;
  const int n = own_tiles(nb1 - nb0, c.wave, kWaves);
  if (n <= 0) return;
  const int lane = threadIdx.x & 63;
  auto target_of = [&](int i) { return new_ids[min(c.block(i + lane), nb1 - 1)]; };  // lane l: of block i + l
  auto kept_of = [&](int i) { return kept[min(c.block(i + (lane >> 4)) * 16 + (lane & 15), u.rd.budget - 1)]; };
  auto row_of = [&](int token) {
    const int idx = min(max(token, 0), u.rd.seq_len - 1);
    return clamp_block(old_ids[idx >> 4], p.n_blocks) * 16 + (idx & 15);
  };
  int targets = target_of(0);
  int from = row_of(kept_of(0)), token = kept_of(4);
  for (int i0 = 0; i0 < n; i0 += 4) {  // uniform over the wavefront
    if (i0 > 0 && (i0 & 63) == 0) targets = target_of(i0);
    const int rows = made_here(from);
    targets = made_here(targets);
    if (i0 + 4 < n) {
      from = row_of(token);
      token = kept_of(i0 + 8);
    }
    stream_tiles<Rows>(
        min(n - i0, 4),
        [&](int i, Rows& kv) {
          c.template load<false>(kv, [&](int row) {
            const int at = __shfl(rows, 16 * i + row);
            return int2{at >> 4, at & 15};
          });
        },
        [&](int i, const Rows& kv) { c.store(c.block(i0 + i), __builtin_amdgcn_readlane(targets, (i0 + i) & 63), kv); });
  }
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
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(select_kernel<kSelectWaves>),
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

hipError_t launch_plan_alloc(const BatchParams& p, const MetaChunk* inline_meta, int n_bytes, hipStream_t s) {
  if (inline_meta) {
    if (n_bytes > (int)sizeof(MetaChunk)) return hipErrorInvalidValue;
    plan_alloc_inline_kernel<<<p.n_comp, kThreads, 0, s>>>(
        p, *inline_meta, const_cast<char*>(reinterpret_cast<const char*>(p.descs)), n_bytes);
  } else {
    plan_alloc_kernel<<<p.n_comp, kThreads, 0, s>>>(p);
  }
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

template <int D, int NT>
static void launch_split_one(const BatchParams& p, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_unfused * p.n_layers * p.n_heads * p.n_split;
  split_rows_kernel<D, NT><<<grid, kThreads, 0, s>>>(p);
  if constexpr (NT > 0) split_scores_kernel<D, NT><<<grid, kThreads, 0, s>>>(p);
}

template <int D>
static hipError_t launch_split_d(const BatchParams& p, hipStream_t s) {
  switch ((p.window + 15) / 16) {
    case 0: launch_split_one<D, 0>(p, s); break;
    case 1: launch_split_one<D, 1>(p, s); break;
    case 2: launch_split_one<D, 2>(p, s); break;
    case 3: launch_split_one<D, 3>(p, s); break;
    case 4: launch_split_one<D, 4>(p, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_split_scores(const BatchParams& p, hipStream_t s) {
  if (p.head_dim == 128) return launch_split_d<128>(p, s);
  if (p.head_dim == 64) return launch_split_d<64>(p, s);
  return hipErrorInvalidValue;
}

hipError_t launch_select(const BatchParams& p, int max_seq_len, bool wide, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_unfused * p.n_layers * p.n_heads;
  const size_t lds = (size_t)(stage_words(max_seq_len) + need_words(max_seq_len)) * sizeof(uint32_t);
  if (wide)
    select_kernel<kSelectWaves><<<grid, 64 * kSelectWaves, lds, s>>>(p);
  else if (max_seq_len <= kFusedMaxLen)
    select_kernel<kNarrow><<<grid, 64 * kNarrow, lds, s>>>(p);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_fused(BatchParams p, int query_tiles, int max_seq_len, int max_blocks, bool wide,
                        hipStream_t s) {
  if (p.n_fused == 0) return hipSuccess;
  if (max_seq_len > (wide ? kFusedWideMaxLen : kFusedMaxLen)) return hipErrorInvalidValue;
  const FusedLds f = fused_lds(max_seq_len, max_blocks, wide);
  p.ids_at = f.ids_at;
  p.ids_room = f.ids_room;
  p.new_ids_at = f.words;  // (a call of one request without plan_alloc)
  size_t lds = (size_t)(f.words + (p.arrivals ? (p.only.n_new + 3) & ~3 : 0)) * sizeof(uint32_t);
  // A launch of nothing but copies is faster with fewer of them at a time: it asks for LDS that
  // it doesn't use.  64 channels, one wide workgroup a CU, not two: 512 heads of 3000-6000
  // tokens 83.0 -> 77.3 us; two narrow ones, not eight, from eight heads a CU on: 3840 heads of
  // 1400-4300 341 -> 328, in place 357 -> 329 (128 channels 835 -> 817, 832 -> 820); but 1024
  // of 640 tokens 25.8 -> 27.8, and 2048 of 200-300, 64 channels, 32.3 -> 34.2 (in place 32.4 ->
  // 34.4; of 640-960 82.0 -> 79.9).
  const bool copies = query_tiles == 0 && max_seq_len == 0;  // (LDS for no score)
  if (copies && wide && p.head_dim == 64) lds = std::max<size_t>(lds, 68 * 1024);
  if (copies && !wide && p.n_fused * p.n_layers * p.n_heads >= 8 * 256 && (p.head_dim == 128 || max_blocks > 32))
    lds = std::max<size_t>(lds, 39 * 1024);
  if (p.head_dim == 128)
    return wide ? launch_fused_wide_128(p, query_tiles, lds, s) : launch_fused_narrow_128(p, query_tiles, lds, s);
  if (p.head_dim == 64)
    return wide ? launch_fused_wide_64(p, query_tiles, lds, s) : launch_fused_narrow_64(p, query_tiles, lds, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gather(const BatchParams& p, hipStream_t s) {
  const unsigned grid = (unsigned)p.n_unfused * p.n_layers * p.n_heads * p.n_split;
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
