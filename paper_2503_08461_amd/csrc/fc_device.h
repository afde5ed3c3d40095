// Device-side helpers shared by the kernel translation units.
#pragma once

#include "fc_internal.h"

namespace fc {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#ifndef FC_WAVES
#define FC_WAVES 4
#endif
static constexpr int kWaves = FC_WAVES;  // wavefronts per workgroup
static constexpr int kThreads = 64 * kWaves;

__device__ __forceinline__ int clamp_block(int blk, int n_blocks) {
  // Block ids come from caller-owned device memory; an id outside the pool
  // must not turn into an out-of-bounds access.
  return ((unsigned)blk < (unsigned)n_blocks) ? blk : 0;
}

// Zombie reclaim of one request: pushes the pre-compression blocks (batch order, table
// order) above the stack top that the new blocks leave and rewrites the table row; old_ids
// and new_ids: copies of what table and stack held.  With copies that plan_alloc made
// nobody reads the table or the stack any more, so one workgroup of a request may do this
// at any time after it.
__device__ __forceinline__ void reclaim_request(const BatchParams& p, const ReqDesc& rd, const int32_t* old_ids,
                                                const int32_t* new_ids, int tid, int n_threads) {
  int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  if (p.in_place) {
    // the request keeps its first n_new blocks; the rest are released
    for (int i = tid; i < rd.n_old - rd.n_new; i += n_threads)
      p.stack[p.top_before + rd.new_off + i] = old_ids[rd.n_new + i];
    for (int i = rd.n_new + tid; i < p.max_blocks; i += n_threads) row[i] = -1;
    if (p.owner)  // (ids checked before the stage: in range, claimed)
      for (int i = tid; i < rd.n_old; i += n_threads) p.owner[old_ids[i]] = i < rd.n_new ? 1 : 0;
    return;
  }
  const int base = p.top_before - p.total_new;
  for (int i = tid; i < rd.n_old; i += n_threads) {
    p.stack[base + rd.old_off + i] = old_ids[i];
    if (p.owner) p.owner[old_ids[i]] = 0;  // (checked before the stage)
  }
  for (int i = tid; i < p.max_blocks; i += n_threads) row[i] = (i < rd.n_new) ? new_ids[i] : -1;
}
__device__ __forceinline__ void reclaim_request(const BatchParams& p, const ReqDesc& rd) {
  reclaim_request(p, rd, p.old_ids + rd.old_off, p.new_ids + rd.new_off, threadIdx.x, blockDim.x);
}

// Loads of what no lane of the launch writes, from a uniform address: scalar loads.
// (Next to the kernel's own stores the compiler takes vector loads, and whatever
// waits for one of those waits for all pool rows in flight.)
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  typedef const __attribute__((address_space(4))) int32_t* ConstWords;
  static_assert(sizeof(T) % 4 == 0, "whole words");
  union {
    T value;
    int32_t words[sizeof(T) / 4];
  } u;
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) u.words[i] = ((ConstWords)(uintptr_t)p)[i];
  return u.value;
}

// LDS accesses of a wavefront's lanes before and after this point stay in that order
// across its lanes (the hardware executes them in program order; this binds the
// compiler, and costs no instruction)
__device__ __forceinline__ void wave_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same value, made at this point: what is computed from it isn't kept from before a loop.
__device__ __forceinline__ int made_here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A thread's lane.  kAnew: made at this point.  The phases of the fused kernels each take it
// anew: what they compute from it (a token's number in a block, a row's, a mask's limit) was
// else computed once, for all phases and all numbers of query tiles, kept while the registers
// hold four tiles of queries, that is, spilled, and read back in the loops.  (In the kernels of
// one phase there is nothing to keep, and 600-1300 tokens, 64 channels, window 32, take 47.6 us
// for their log-sum-exps with it and 43.2 without.)
template <bool kAnew>
__device__ __forceinline__ int lane_number() {
  const int lane = threadIdx.x & 63;
  if constexpr (kAnew) return made_here(lane);
  return lane;
}

// What stands before this point is issued before what follows (binds the compiler, which
// would put requests for what comes next behind the wait for what is used now)
__device__ __forceinline__ void requests_first() { __builtin_amdgcn_sched_barrier(0); }

// the same register of another lane of the 16-lane row, by DPP control
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ uint32_t from_lane_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
// Scan and reductions over a wavefront by DPP (row_shr 1, 2, 4, 8, then
// row_bcast:15 and :31): a handful of vector instructions each, where the same
// steps by __shfl are six LDS round trips one after the other.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or(uint32_t identity, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROWS, 0xF, false);
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, uint32_t identity, Op op) {  // inclusive
  v = op(v, dpp_or<0x111, 0xF>(identity, v));
  v = op(v, dpp_or<0x112, 0xF>(identity, v));
  v = op(v, dpp_or<0x114, 0xF>(identity, v));
  v = op(v, dpp_or<0x118, 0xF>(identity, v));
  v = op(v, dpp_or<0x142, 0xA>(identity, v));
  return op(v, dpp_or<0x143, 0xC>(identity, v));
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, uint32_t identity, Op op) {  // uniform
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(v, identity, op), 63);
}
__device__ __forceinline__ int wave_scan_add(int v) {
  return (int)wave_scan((uint32_t)v, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ int wave_sum(int v) {
  return (int)wave_reduce((uint32_t)v, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  return wave_reduce(v, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  return wave_reduce(v, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ float wave_sum(float v) {
  return __uint_as_float(wave_reduce(__float_as_uint(v), 0u, [](uint32_t a, uint32_t b) {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  }));
}

// sum over the four lanes that share lane % 16, left in every one of them:
// neighbouring rows of 16 change places, then the halves of the wavefront
__device__ __forceinline__ float quarter_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ half8 load_half8(const _Float16* p) {
  return *reinterpret_cast<const half8*>(p);
}

// The same accesses with the non-temporal hint, for data that this kernel will
// not touch again: the line is the first to leave the caches, which keeps what
// IS read again (K between the two passes of the SnapKV score, the rows that
// the compaction re-reads) in L2 and in the memory-side cache for longer.
__device__ __forceinline__ half8 load_half8_nt(const _Float16* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const half8*>(p));
}

__device__ __forceinline__ void store_half8_nt(_Float16* p, half8 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<half8*>(p));
}

__device__ __forceinline__ void store_half8(_Float16* p, half8 v) {
  *reinterpret_cast<half8*>(p) = v;
}

// Walks n tiles: load(i, tile) requests the i-th, use(i, tile) works on it
// with the next one on its way.  The loop has no branch around a load and no copy between
// the two buffers: after a branch the compiler waits for as few loads as either side left
// in flight, and a copy waits for what it copies, so that with either of them a wavefront
// waited for the tile that it had just asked for before it worked on the one it had.
// The whole of a call, with that wait and without: one prompt of 640 tokens, 32 layers of 32
// heads, 79.5 -> 70 us (5.9 us a head less in the first pass, 7 in the copy); 1024 heads of
// 7000 tokens 813 -> 700; 2048 of 1500, 64 channels, 184 -> 155; 24 prompts of 500-6000
// tokens with scores, 2 layers, 671 -> 635; 32 of 600-1200, 8 layers, 1037 -> 1009.
template <typename Tile, typename Load, typename Use>
__device__ __forceinline__ void stream_tiles(int n, Load load, Use use) {
  if (n <= 0) return;  // uniform over the wavefront, as all conditions here
  Tile a, b;
  auto request = [&](int i, Tile& tile) {
    load(i, tile);
    requests_first();
  };
  load(0, a);
  int i = 0;
  for (; i + 2 < n; i += 2) {
    request(i + 1, b);
    use(i, a);
    request(i + 2, a);
    use(i + 1, b);
  }
  const bool two = i + 1 < n;
  if (two) request(i + 1, b);
  use(i, a);
  if (two) use(i + 1, b);
}
// how many of n tiles a wavefront has, every `step`-th from its own on
__device__ __forceinline__ int own_tiles(int n, int wave, int step) { return (n - wave + step - 1) / step; }

}  // namespace fc
