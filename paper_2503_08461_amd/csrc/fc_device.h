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
// order) above the stack top left by plan_alloc and rewrites the table row.  From
// plan_alloc on all kernels of the stage read the saved copies of the ids, nobody the
// table or the stack, so one workgroup of a request may do this at any time after it.
__device__ __forceinline__ void reclaim_request(const BatchParams& p, const ReqDesc& rd) {
  const int tid = threadIdx.x, n_threads = blockDim.x;
  int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  if (p.in_place) {
    // the request keeps its first n_new blocks; the rest are released
    for (int i = tid; i < rd.n_old - rd.n_new; i += n_threads)
      p.stack[p.top_before + rd.new_off + i] = p.old_ids[rd.old_off + rd.n_new + i];
    for (int i = rd.n_new + tid; i < p.max_blocks; i += n_threads) row[i] = -1;
    if (p.owner)  // (ids checked before the stage: in range, claimed)
      for (int i = tid; i < rd.n_old; i += n_threads) p.owner[p.old_ids[rd.old_off + i]] = i < rd.n_new ? 1 : 0;
    return;
  }
  const int base = p.top_before - p.total_new;
  for (int i = tid; i < rd.n_old; i += n_threads) {
    p.stack[base + rd.old_off + i] = p.old_ids[rd.old_off + i];
    if (p.owner) p.owner[p.old_ids[rd.old_off + i]] = 0;  // (checked before the stage)
  }
  for (int i = tid; i < p.max_blocks; i += n_threads) row[i] = (i < rd.n_new) ? p.new_ids[rd.new_off + i] : -1;
}

// LDS accesses of a wavefront's lanes before and after this point stay in that order
// across its lanes (the hardware executes them in program order; this binds the
// compiler, and costs no instruction)
__device__ __forceinline__ void wave_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

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

}  // namespace fc
