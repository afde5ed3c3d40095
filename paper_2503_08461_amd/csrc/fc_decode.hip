// Decode-side pool traffic (Algorithm 1, ExecuteDecoding: every step reads the
// compressed cache of each request of the batch and appends the new token's
// K and V): a batched one-token append and the single-query attention of one
// decode step over the paged cache.  Both are HBM-bound: the append moves
// 4*d bytes per (request, layer, head), the attention reads every cached K and
// V row once, 4*d bytes per token of a (layer, head).

#include <type_traits>

#include "fc_device.h"

namespace fc {

// ---------------------------------------------------------------------------
// append: workgroup = (request, layer); the 2 * n_heads new rows of that layer
// go to slot L % 16 of the request's last block.  A request on a block
// boundary takes the block that the host assigned it from the top of the free
// stack (pops in batch order) and the layer-0 workgroup records it in the table.
// ---------------------------------------------------------------------------
//
// Reqs (here and below): DecodeReqs, the requests in the arguments, or DecodeReqList,
// on the device.  Kernels of their own: 3.6 KB of arguments that nobody reads cost a
// launch of small caches several us.
template <int D, typename Reqs>
__global__ __launch_bounds__(kThreads) void append_kernel(DecodeParams p, Reqs reqs) {
  const int r = blockIdx.x / p.n_layers;
  const int layer = blockIdx.x - r * p.n_layers;
  const DecodeReq rq = reqs.req[r];
  const int L = rq.seq_len;
  int32_t* row = p.block_tables + (size_t)rq.table_row * p.max_blocks;
  int blk;
  if (rq.pop_index >= 0) {
    const int id = p.stack[p.top_before - 1 - rq.pop_index];
    blk = clamp_block(id, p.n_blocks);
    if (layer == 0 && threadIdx.x == 0) {
      row[L >> 4] = blk;
      // ownership checks (debug mode): a popped block must have been free
      if (p.owner && ((unsigned)id >= (unsigned)p.n_blocks || atomicExch(&p.owner[id], 1) != 0))
        atomicOr(p.error_flag, 4 << 8);
    }
  } else {
    blk = clamp_block(row[L >> 4], p.n_blocks);
  }
  constexpr int PPR = D / 8;  // 16-byte pieces of a row
  const size_t blk_stride = (size_t)2 * p.n_heads * 16 * D;
  _Float16* dst = p.kv + ((size_t)layer * p.n_blocks + blk) * blk_stride + (size_t)(L & 15) * D;
  const _Float16* src = p.new_kv + ((size_t)rq.table_row * p.n_layers + layer) * 2 * p.n_heads * D;
  for (int i = threadIdx.x; i < 2 * p.n_heads * PPR; i += kThreads) {
    const int rh = i / PPR, piece = i - rh * PPR;  // rh = kv * n_heads + head
    store_half8(dst + (size_t)rh * 16 * D + piece * 8, load_half8(src + (size_t)rh * D + piece * 8));
  }
}

// f(the requests of p, wherever they are)
template <typename F>
static void with_reqs(const DecodeParams& p, const DecodeReqs& inline_reqs, F f) {
  if (p.reqs)
    f(DecodeReqList{p.reqs});
  else
    f(inline_reqs);
}

hipError_t launch_append(const DecodeParams& p, const DecodeReqs& inline_reqs, hipStream_t s) {
  if (p.n_req == 0) return hipSuccess;
  if (p.head_dim != 64 && p.head_dim != 128) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)p.n_req * p.n_layers;
  with_reqs(p, inline_reqs, [&](const auto& reqs) {
    using Reqs = std::decay_t<decltype(reqs)>;
    if (p.head_dim == 128)
      append_kernel<128, Reqs><<<grid, kThreads, 0, s>>>(p, reqs);
    else
      append_kernel<64, Reqs><<<grid, kThreads, 0, s>>>(p, reqs);
  });
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// attention of one decode step: workgroup = (request, layer, head) or a segment of
// one, requests in the order the host lists them (longest first).  A 16-token block
// of one head is 32*D contiguous bytes for K and for V; a wavefront reads it with
// D/8 neighbouring lanes on one row (fully coalesced 16-byte loads), forms
// q.k by a DPP reduction inside that lane group, and keeps one online-softmax state
// (running max, sum, and this lane's 8 output channels) per lane group.  The
// 4 * (512 / D) states of the workgroup are merged through LDS at the end.
//
// What bounds it is HBM where the call has many heads to offer.  With few of them
// the chip waits for the CU that has the longest one (one CU draws about 27 GB/s
// whatever its wavefronts request), so such a call cuts every head into segments of
// about p.seg_blocks blocks, all of one head alike: each leaves its state in p.partial, and
// a second launch merges them.  A wavefront has only about four blocks of a segment, so
// there its loads' latency shows: it asks for the next block before it works on this one
// (kCut).  8 caches of 256-1408 tokens, 32 heads: 26.5 us with segments of exactly
// p.seg_blocks and one block in flight, 25.3 with even segments, 24.2 with both; 4 of
// 1080-1120: 18.8, 18.0, 16.2.  Whole heads keep one block in flight and more wavefronts (58
// registers against 94): 957 us against 964 (48 caches of 1280-7040 tokens, 2 layers).
// (Merged by the workgroup that finishes a head last, the release and acquire fences of
// all segments cost 170 to 300 us, against the 5 us of a launch.)
// ---------------------------------------------------------------------------
//
// kIndexed: the counterfactual of a cache that was pruned WITHOUT compaction:
// the unit attends over the budget_r tokens of its kept list, read where they
// lie in the uncompacted cache (every row its own 2*D contiguous bytes).

// sum over the LPR neighbouring lanes of a row, in every one of them
template <int LPR>
__device__ __forceinline__ float row_lanes_sum(float s) {
  s += from_lane<0xB1>(s);   // the other lane of the pair,
  s += from_lane<0x4E>(s);   // the other pair of the quad,
  s += from_lane<0x141>(s);  // the other quad of the eight,
  if constexpr (LPR == 16) s += from_lane<0x140>(s);  // the other eight of the sixteen
  return s;
}

template <int D, bool kIndexed, bool kCut, typename Reqs>
__global__ __launch_bounds__(kThreads) void decode_attention_kernel(DecodeParams p, Reqs reqs) {
  constexpr int LPR = D / 8;        // lanes per row
  constexpr int RPI = 64 / LPR;     // rows per wavefront load instruction
  constexpr int IPB = 16 / RPI;     // load instructions per 16-token block
  constexpr int NG = kWaves * RPI;  // softmax states per workgroup
  const int n_lh = p.n_layers * p.n_heads;
  // (segment, request, layer and head): the workgroups of segments that a shorter request
  // does not have come last (16 caches of 1000-3000 tokens, 4 layers of 12 heads: 131.6 us
  // with them between the others, 128.0 so)
  const int unit = kCut ? blockIdx.x % (p.n_req * n_lh) : blockIdx.x;
  const int seg = kCut ? blockIdx.x / (p.n_req * n_lh) : 0;
  const int slot = unit / n_lh;
  const int lh = unit - slot * n_lh;
  const DecodeReq rq = reqs.req[slot];
  const int L = kIndexed ? rq.pop_index : rq.seq_len;  // indexed: pop_index holds the budget
  const int nb = (L + 15) >> 4;
  const int n_seg = kCut ? decode_segments(nb, p.seg_blocks) : 1;
  if (seg >= n_seg) return;  // uniform: this request has fewer segments
  const int b0 = kCut ? decode_segment_begin(nb, n_seg, seg) : 0;
  const int b1 = kCut ? decode_segment_begin(nb, n_seg, seg + 1) : nb;
  const int layer = lh / p.n_heads;
  const int head = lh - layer * p.n_heads;
  const int32_t* kept =
      kIndexed ? p.kept + rq.kept_off + (size_t)lh * L : nullptr;  // ascending token indices
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane / LPR;    // which row of a load instruction
  const int piece = lane % LPR;  // which 8 channels
  float* out = p.out + ((size_t)rq.table_row * n_lh + lh) * D;

  const _Float16* qp = p.q + ((size_t)rq.table_row * n_lh + lh) * D + piece * 8;
  float qf[8];
  {
    const half8 qh = load_half8(qp);
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[e] = (float)qh[e] * p.scale_log2e;
  }
  const int32_t* row = p.block_tables + (size_t)rq.table_row * p.max_blocks;
  const size_t blk_stride = (size_t)2 * p.n_heads * 16 * D;
  const size_t v_off = (size_t)p.n_heads * 16 * D;
  const _Float16* base = p.kv + (size_t)layer * p.n_blocks * blk_stride + (size_t)head * 16 * D +
                         (kIndexed ? 0 : (size_t)grp * D) + piece * 8;

  float m = -INFINITY, z = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  struct Rows {
    half8 k[IPB], v[IPB];
  };
  auto fetch = [&](int b, Rows& x) {
    if (kIndexed) {
      // 16 kept tokens at a time, each fetched from its own block and slot
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        const int j = b * 16 + i * RPI + grp;
        const int tok = min(max(kept[min(j, L - 1)], 0), rq.seq_len - 1);
        const _Float16* kp = base + (size_t)clamp_block(row[tok >> 4], p.n_blocks) * blk_stride +
                             (size_t)(tok & 15) * D;
        x.k[i] = load_half8_nt(kp);
        x.v[i] = load_half8_nt(kp + v_off);
      }
    } else {
      const _Float16* kp = base + (size_t)clamp_block(row[b], p.n_blocks) * blk_stride;
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        x.k[i] = load_half8_nt(kp + (size_t)i * RPI * D);
        x.v[i] = load_half8_nt(kp + v_off + (size_t)i * RPI * D);
      }
    }
  };
  auto attend = [&](int b, const Rows& x) {
#pragma unroll
    for (int i = 0; i < IPB; ++i) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) s += qf[e] * (float)x.k[i][e];
      s = row_lanes_sum<LPR>(s);
      const int tok = b * 16 + i * RPI + grp;
      if (tok < L) {  // the whole lane group takes the same branch
        const float mn = fmaxf(m, s);
        const float a = __builtin_amdgcn_exp2f(m - mn);  // 0 for the first token (m = -inf)
        const float w = __builtin_amdgcn_exp2f(s - mn);
        z = z * a + w;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = acc[e] * a + w * (float)x.v[i][e];
        m = mn;
      }
    }
  };
  if constexpr (kCut) {
    stream_tiles<Rows>(
        own_tiles(b1 - b0, wave, kWaves), [&](int i, Rows& x) { fetch(b0 + wave + kWaves * i, x); },
        [&](int i, const Rows& x) { attend(b0 + wave + kWaves * i, x); });
  } else {
    for (int b = wave; b < nb; b += kWaves) {
      Rows x;
      fetch(b, x);
      attend(b, x);
    }
  }

  // merge the NG states: each has its own max, so rescale to the common one
  __shared__ float sm_m[NG], sm_z[NG];
  __shared__ float sm_acc[NG][D];
  const int g = wave * RPI + grp;
  if (piece == 0) {
    sm_m[g] = m;
    sm_z[g] = z;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) sm_acc[g][piece * 8 + e] = acc[e];
  __syncthreads();
  float mm = -INFINITY, zz = 0.f, o = 0.f;
  if (threadIdx.x < D) {
    for (int i = 0; i < NG; ++i) mm = fmaxf(mm, sm_m[i]);
    for (int i = 0; i < NG; ++i) {
      // (a sum of zero: no token; not a number stays not a number)
      const float f = sm_z[i] == 0.f ? 0.f : __builtin_amdgcn_exp2f(sm_m[i] - mm);
      zz += sm_z[i] * f;
      o += sm_acc[i][threadIdx.x] * f;
    }
  }
  if (n_seg == 1) {  // uniform
    if (threadIdx.x < D) out[threadIdx.x] = L > 0 ? o / zz : 0.f;
    return;
  }

  // a segment's state: channel sums, max, sum
  float* mine = p.partial + (((size_t)slot * n_lh + lh) * p.n_seg + seg) * DecodeParams::state_words(D);
  if (threadIdx.x < D) mine[threadIdx.x] = o;
  if (threadIdx.x == 0) {
    mine[D] = mm;
    mine[D + 1] = zz;
  }
}

// segments of at least 16 blocks, of a head of at most 32768 tokens
static constexpr int kMaxHeadSegments = kPlanMaxSeqLen / kPlanBlockSize / 16;

// Heads that were cut: the output from the segments' states.  workgroup =
// (request, layer, head), one thread per channel.
template <int D, bool kIndexed, typename Reqs>
__global__ __launch_bounds__(D) void decode_merge_kernel(DecodeParams p, Reqs reqs) {
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const DecodeReq rq = reqs.req[slot];
  const int L = kIndexed ? rq.pop_index : rq.seq_len;
  const int n_seg = decode_segments((L + 15) >> 4, p.seg_blocks);
  if (n_seg <= 1) return;  // written by the kernel above
  constexpr int kWords = DecodeParams::state_words(D);
  const float* states = p.partial + (size_t)blockIdx.x * p.n_seg * kWords;
  __shared__ float sm_m[kMaxHeadSegments], sm_z[kMaxHeadSegments];
  for (int i = threadIdx.x; i < n_seg; i += D) {  // (kMaxHeadSegments at most: checked by the launcher)
    sm_m[i] = states[(size_t)i * kWords + D];
    sm_z[i] = states[(size_t)i * kWords + D + 1];
  }
  __syncthreads();
  float mm = -INFINITY, zz = 0.f, o = 0.f;
  for (int i = 0; i < n_seg; ++i) mm = fmaxf(mm, sm_m[i]);
#pragma unroll 8
  for (int i = 0; i < n_seg; ++i) {
    const float f = sm_z[i] == 0.f ? 0.f : __builtin_amdgcn_exp2f(sm_m[i] - mm);
    zz += sm_z[i] * f;
    o += states[(size_t)i * kWords + threadIdx.x] * f;
  }
  p.out[((size_t)rq.table_row * n_lh + lh) * D + threadIdx.x] = o / zz;
}

template <int D, bool kIndexed>
static void launch_decode_one(const DecodeParams& p, const DecodeReqs& inline_reqs, hipStream_t s) {
  const unsigned heads = (unsigned)p.n_req * p.n_layers * p.n_heads;
  with_reqs(p, inline_reqs, [&](const auto& reqs) {
    using Reqs = std::decay_t<decltype(reqs)>;
    if (p.n_seg == 1) {
      decode_attention_kernel<D, kIndexed, false, Reqs><<<heads, kThreads, 0, s>>>(p, reqs);
      return;
    }
    decode_attention_kernel<D, kIndexed, true, Reqs><<<heads * p.n_seg, kThreads, 0, s>>>(p, reqs);
    decode_merge_kernel<D, kIndexed, Reqs><<<heads, D, 0, s>>>(p, reqs);
  });
}

hipError_t launch_decode_attention(const DecodeParams& p, const DecodeReqs& inline_reqs, hipStream_t s) {
  if (p.n_req == 0) return hipSuccess;
  if (p.n_seg < 1 || p.n_seg > kMaxHeadSegments || p.seg_blocks < 1) return hipErrorInvalidValue;
  const bool indexed = p.kept != nullptr;
  if (p.head_dim == 128 && !indexed)
    launch_decode_one<128, false>(p, inline_reqs, s);
  else if (p.head_dim == 128)
    launch_decode_one<128, true>(p, inline_reqs, s);
  else if (p.head_dim == 64 && !indexed)
    launch_decode_one<64, false>(p, inline_reqs, s);
  else if (p.head_dim == 64)
    launch_decode_one<64, true>(p, inline_reqs, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace fc
