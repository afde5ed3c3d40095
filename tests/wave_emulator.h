// One workgroup of device code on the CPU: every lane is a coroutine, lanes meet
// only where the code makes them (a wavefront operation, a wavefront barrier, a
// workgroup barrier), and between those the caller picks who runs first.  What the
// device code owes to lock step or to luck shows as a wrong result under some order;
// lanes of a workgroup at different barriers, and lanes that wait for each other,
// are reported.
//
// Include this instead of hip_runtime.h and before any header with device code
// (compiled with -x hip --offload-host-only); only the operations that the tests
// need are here.
#pragma once

#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>

namespace emu {

enum State { READY, AT_WAVE, AT_BLOCK, DONE };

struct Lane {
  ucontext_t ctx;
  std::vector<char> stack;
  State state = READY;
  int line = 0;       // where it waits
  unsigned n_ops = 0;  // wavefront operations so far
};

struct Block {
  std::vector<Lane> lanes;
  std::vector<uint64_t> post[2];  // operands of the wavefront operation before and after the running one
  ucontext_t home;
  int self = 0;
  std::function<void()> body;
};
inline Block* g_block = nullptr;

inline void yield(State s, int line) {
  Lane& l = g_block->lanes[g_block->self];
  l.state = s;
  l.line = line;
  swapcontext(&l.ctx, &g_block->home);
}

inline void lane_main() {
  g_block->body();
  yield(DONE, 0);
}

// Runs body() as a workgroup of n_waves wavefronts.  waves_down: the highest
// wavefront runs first, as far as it can, else the lowest; lanes_down: the same for
// the lanes of a wavefront.
inline void run_block(int n_waves, bool waves_down, bool lanes_down, std::function<void()> body) {
  Block b;
  g_block = &b;
  b.body = std::move(body);
  const int n = 64 * n_waves;
  b.lanes.resize(n);
  for (auto& p : b.post) p.assign(n, 0);
  for (Lane& l : b.lanes) {
    l.stack.resize(64 << 10);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.data();
    l.ctx.uc_stack.ss_size = l.stack.size();
    l.ctx.uc_link = nullptr;
    makecontext(&l.ctx, lane_main, 0);
  }
  // one round of a wavefront: every lane that may, up to where it waits; false: none could
  auto step_wave = [&](int w) {
    bool ran = false;
    int at_wave = 0, done = 0, line = 0;
    for (int i = 0; i < 64; ++i) {
      const int t = 64 * w + (lanes_down ? 63 - i : i);
      Lane& l = b.lanes[t];
      if (l.state == READY) {
        b.self = t;
        swapcontext(&b.home, &l.ctx);
        ran = true;
      }
      done += l.state == DONE;
      if (l.state == AT_WAVE) {
        ++at_wave;
        if (line && l.line != line) {
          printf("lanes of a wavefront at different operations (lines %d and %d)\n", line, l.line);
          exit(4);
        }
        line = l.line;
      }
    }
    if (at_wave == 64) {
      for (int i = 0; i < 64; ++i) b.lanes[64 * w + i].state = READY;
      ran = true;
    }
    return ran;
  };
  for (;;) {
    for (int i = 0; i < n_waves; ++i)
      while (step_wave(waves_down ? n_waves - 1 - i : i)) {
      }
    int done = 0, at_block = 0, line = 0;
    for (Lane& l : b.lanes) {
      done += l.state == DONE;
      if (l.state != AT_BLOCK) continue;
      ++at_block;
      if (line && l.line != line) {
        printf("wavefronts at different barriers (lines %d and %d)\n", line, l.line);
        exit(5);
      }
      line = l.line;
    }
    if (done == n) break;
    if (at_block != n) {
      printf("lanes that wait for ever: %d ended, %d at a barrier, %d lanes\n", done, at_block, n);
      exit(6);
    }
    for (Lane& l : b.lanes) l.state = READY;
  }
  g_block = nullptr;
}

struct ThreadIdx {
  unsigned x;
};
inline ThreadIdx thread_idx() { return {(unsigned)g_block->self}; }
inline void block_barrier(int line) { yield(AT_BLOCK, line); }

// all lanes of the wavefront post a value and meet; the returned array holds all 64
inline const uint64_t* exchange(uint64_t v, int line) {
  const int self = g_block->self;
  std::vector<uint64_t>& post = g_block->post[g_block->lanes[self].n_ops++ & 1];
  post[self] = v;
  yield(AT_WAVE, line);
  return post.data() + (self & ~63);
}
inline void wave_barrier(int line) { exchange(0, line); }
inline uint64_t ballot(bool b, int line) {
  const uint64_t* v = exchange(b, line);
  uint64_t m = 0;
  for (int i = 0; i < 64; ++i) m |= v[i] << i;
  return m;
}
inline int readlane(int v, int lane, int line) { return (int)exchange((uint32_t)v, line)[lane]; }
// data parallel primitives: quad_perm, row_shr, mirrors and broadcasts
inline int dpp(int old, int src, int ctrl, int row_mask, int line) {
  const uint64_t* v = exchange((uint32_t)src, line);
  const int lane = g_block->self & 63, row = lane >> 4, at = lane & 15;
  int from = -1;
  if (ctrl <= 0xFF) {
    from = (lane & ~3) | ((ctrl >> (2 * (lane & 3))) & 3);
  } else if (ctrl > 0x110 && ctrl <= 0x11F) {
    if (at >= ctrl - 0x110) from = lane - (ctrl - 0x110);
  } else if (ctrl == 0x140) {
    from = 16 * row + 15 - at;
  } else if (ctrl == 0x141) {
    from = (lane & ~7) + 7 - (lane & 7);
  } else if (ctrl == 0x142) {
    if (row > 0) from = 16 * row - 1;
  } else if (ctrl == 0x143) {
    if (row > 1) from = 31;
  } else {
    printf("DPP control %x\n", ctrl);
    exit(7);
  }
  return ((row_mask >> row) & 1) && from >= 0 ? (int)v[from] : old;
}
template <typename T, typename U>
inline T atomic_add(T* p, U v) {
  const T old = *p;
  *p += v;
  return old;
}

}  // namespace emu

// the device vocabulary of the included headers
#undef __device__
#define __device__ __attribute__((host, device))
#define threadIdx emu::thread_idx()
#define __syncthreads() emu::block_barrier(__LINE__)
#define __ballot(b) emu::ballot(b, __LINE__)
#define atomicAdd(p, v) emu::atomic_add(p, v)
#define __builtin_amdgcn_wave_barrier() emu::wave_barrier(__LINE__)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_readlane(v, lane) emu::readlane(v, lane, __LINE__)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_update_dpp(old, src, ctrl, rows, banks, bound) emu::dpp(old, src, ctrl, rows, __LINE__)
#define __popcll(x) __builtin_popcountll(x)
#define __clz(x) ((x) ? __builtin_clz((uint32_t)(x)) : 32)
#define __float_as_uint(x) __builtin_bit_cast(uint32_t, (float)(x))
#define __uint_as_float(x) __builtin_bit_cast(float, (uint32_t)(x))

// (hip_runtime.h has host versions of min and max for int only)
namespace fc {
inline __device__ int min(int a, int b) { return a < b ? a : b; }
inline __device__ int max(int a, int b) { return a > b ? a : b; }
inline __device__ uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
inline __device__ uint32_t max(uint32_t a, uint32_t b) { return a > b ? a : b; }
}  // namespace fc
