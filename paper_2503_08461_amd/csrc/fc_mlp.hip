// Chunk-MLP compressor kernel for gfx950: every run of k consecutive tokens
// of one modality becomes one row, y = W2 . act(W1 . x + b1) + b2 (GELU, erf or tanh form).
//
// This is the one dense contraction of the library that is MFMA-bound
// (about 390 kflop per 1.3 KB chunk at k = 5, d = 128, hidden = 256), so it is
// laid out around v_mfma_f32_16x16x32_f16 in the TRANSPOSED form
//     H^T [hidden x chunks] = W1 [hidden x k*d] . X^T [k*d x chunks]
//     Y^T [d x chunks]      = W2 [d x hidden]   . H^T
// with chunks on the MFMA column (lane) axis:
//   * the B operand of the first product (lane = chunk, 8 consecutive channels
//     of one token row) comes from the scattered pool blocks through registers and
//     a small LDS tile of the wavefront's own;
//   * the A operands (weights) are pre-permuted once into operand order; a token's
//     slabs of W1 and all of W2 are equally large, contiguous pieces, and the workgroup
//     pulls them through one ring in LDS, straight from memory;
//   * the result tiles of the first product already have the chunk on the
//     lane, which is what the B operand of the second product needs; only the
//     order of the contraction index differs, and that is folded into the
//     pre-permutation of W2.  The hidden activations therefore never leave
//     registers.
// A workgroup handles tiles of 128 or 256 rows (row = (layer, head, K|V) x chunk of
// one request and one modality), two column tiles of 16 rows per wavefront; the kernel
// is persistent (one to three workgroups per CU walk the tile list).
//
// What bounds it: at d = 128, hidden 256 the instructions of a tile at the clock that the
// card's power allows.  The clock falls to 1.7 GHz, and with rows of zeros the same
// instructions take two thirds of the time, every phase alike.  That is no ceiling: the
// matrix pipes are busy for 46 % of those cycles, and next to a product stand 0.68 LDS
// instructions (an operand of W1 serves two products) and 2.5 vector instructions, most of
// them the activation's, which take cycles and power alike.  A loop of nothing but MFMAs
// on random values: 32x32x16 1.56-1.65 PFLOP/s, 16x16x32 1.92; with an operand read from
// LDS every 32 cycles 1.43 and 1.62.  So the smaller tiles are used although both need as
// many operands (24 prompts of 1280-7040 tokens, 2 layers of 32 heads, k = 5: 1383 -> 1294 us;
// with weights from memory to LDS past the registers, rows read 64 bytes at a time and
// target rows looked up by one lane each 1403 -> 1383).  Loads complete in order, so any
// load that is waited for waits for all rows requested before it: weights are requested
// seven groups ahead, waits count what may still be on its way, and the tile list and
// the requests are read by scalar loads.

#include "fc_device.h"

#include <math.h>

#include <type_traits>

namespace fc {

static constexpr uint32_t kNoRow = 0xffffffffu;  // "no such token" in the table of pool rows

// Wavefronts of a workgroup (32 rows of a tile each) and workgroups per CU.  Eight
// wavefronts of up to 256 registers are what the accumulators and the operands in
// flight allow; at 64 channels and 128 hidden units a wavefront needs 150 registers
// and a workgroup 46 KB of LDS, so three workgroups of four fit, whose phases (first
// product, activation, second product, store) then run side by side instead of in
// step (24 prompts of 1280-7040 tokens, 2 layers of 32 heads, k = 5, an earlier form of
// the kernel: 743 -> 595 us).
template <int D, int HID>
struct MlpShape {
  static constexpr int kWaves = D == 64 && HID == 128 ? 4 : 8;
  static constexpr int kPerCu = D == 64 && HID == 128 ? 3 : 1;
  static constexpr int kRows = 32 * kWaves, kThreads = 64 * kWaves;
  static constexpr int kWavesPerSimd = kWaves * kPerCu / 4;
};

template <typename F>
static auto with_mlp_shape(int head_dim, int hidden, F f) {
  if (head_dim == 128) return hidden == 256 ? f(MlpShape<128, 256>()) : f(MlpShape<128, 128>());
  return hidden == 256 ? f(MlpShape<64, 256>()) : f(MlpShape<64, 128>());
}
int mlp_rows_per_tile(int head_dim, int hidden) {
  return with_mlp_shape(head_dim, hidden, [](auto s) -> int { return s.kRows; });
}
int mlp_workgroups_per_cu(int head_dim, int hidden) {
  return with_mlp_shape(head_dim, hidden, [](auto s) -> int { return s.kPerCu; });
}

// hidden unit that sits at contraction position (slab sl of 32, lane quarter q4,
// element e) of the second product, given how the first product leaves its result in
// registers (16x16 tile: register r of lane quarter q4 holds row 4 q4 + r; a slab is
// two tiles)
__host__ __device__ constexpr int mlp_hidden_unit(int sl, int q4, int e) {
  return 32 * sl + 16 * (e / 4) + 4 * q4 + e % 4;
}

// Output channel that sits on row rho of tile ot of the second product's A operand:
// the registers of a pair of tiles are then 8 consecutive channels of a lane, one
// 16-byte store, and the four quarters of the wavefront store 64 bytes of a row.
__host__ __device__ constexpr int mlp_out_channel(int ot, int rho) {
  return 32 * (ot / 2) + 8 * (rho / 4) + 4 * (ot % 2) + rho % 4;
}

size_t mlp_w1p_elems(int head_dim, int hidden, int k) { return (size_t)hidden * k * head_dim; }
size_t mlp_w2p_elems(int head_dim, int hidden) { return (size_t)hidden * head_dim; }

// Contraction position (slab s, lane quarter q4, element e) of the first product is
// channel 32 j + 8 q4 + e of token t of the chunk, s = t * (d / 32) + j.
// w1p[s][mt][lane][e] = w1[mt*16 + lane%16][t*D + 32*j + 8*(lane/16) + e]
// w2p[sl][ot][lane][e] = w2[mlp_out_channel(ot, lane%16)][mlp_hidden_unit(sl, lane/16, e)]
__global__ void mlp_permute_kernel(const _Float16* w1, const _Float16* w2, _Float16* w1p,
                                   _Float16* w2p, int head_dim, int hidden, int k) {
  const int kd = k * head_dim;
  const size_t n1 = (size_t)hidden * kd, n2 = (size_t)hidden * head_dim;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n1) {
    const int e = i & 7, lane = (i >> 3) & 63;
    const size_t rest = i >> 9;
    const int mt1 = hidden / 16;
    const int mt = rest % mt1, s = rest / mt1;
    const int spt = head_dim / 32;
    const int t = s / spt, j = s - t * spt;
    w1p[i] = w1[(size_t)(mt * 16 + (lane & 15)) * kd + t * head_dim + 32 * j + 8 * (lane >> 4) + e];
  }
  if (i < n2) {
    const int e = i & 7, lane = (i >> 3) & 63;
    const size_t rest = i >> 9;
    const int mt2 = head_dim / 16;
    const int ot = rest % mt2, sl = rest / mt2;
    w2p[i] = w2[(size_t)mlp_out_channel(ot, lane & 15) * hidden + mlp_hidden_unit(sl, lane >> 4, e)];
  }
}

hipError_t launch_mlp_permute_weights(const _Float16* w1, const _Float16* w2, _Float16* w1p,
                                      _Float16* w2p, int head_dim, int hidden, int k,
                                      hipStream_t s) {
  const size_t n = std::max(mlp_w1p_elems(head_dim, hidden, k), mlp_w2p_elems(head_dim, hidden));
  mlp_permute_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(w1, w2, w1p, w2p, head_dim,
                                                                 hidden, k);
  return hipGetLastError();
}

// tanh form of GELU, v/2 * (1 + tanh(u)) with u = sqrt(2/pi) * (v + 0.044715 v^3),
// written as v / (1 + exp(-2u)) = v / (1 + exp2(v * (A + B v^2))) with the
// constants folded (A = -2 log2(e) sqrt(2/pi), B = 0.044715 A): one exp2, one
// reciprocal and five other operations per value
__device__ __forceinline__ float gelu_tanh(float v) {
  const float e = __builtin_amdgcn_exp2f(v * fmaf(v * v, -0.10294324f, -2.3022082f));
  return v * __builtin_amdgcn_rcpf(1.0f + e);
}

// GELU by its definition, v * Phi(v), Phi the standard normal distribution
// function.  Phi(-|v|) = exp2(P(|v|)) with P a polynomial of degree 6: log2 of
// the normal tail is smooth (about -x^2 / 2 ln 2 - log2 x for large x), and a
// fit of P that minimises the largest error of v * Phi(v) over |v| <= 9 leaves
// 1.4e-7 absolute in exact arithmetic, 3e-7 evaluated in fp32 (as accurate as
// the usual five-term rational approximation of erfc, at one transcendental
// instead of two and no division).  Past |v| = 8.5 nothing is left of the tail
// (Phi(-8.5) = 1e-17) and the polynomial is not followed further.
// GELU(v) = v Phi(-|v|) for v < 0, v - v Phi(-|v|) otherwise, i.e. max(v, 0) - |v| Phi(-|v|).
#define FC_GELU_TAIL_P0 -9.999973123e-01f
#define FC_GELU_TAIL_P1 -1.151156811e+00f
#define FC_GELU_TAIL_P2 -4.588952346e-01f
#define FC_GELU_TAIL_P3 -5.326704516e-02f
#define FC_GELU_TAIL_P4 7.999533677e-03f
#define FC_GELU_TAIL_P5 -7.477810617e-04f
#define FC_GELU_TAIL_P6 3.095778387e-05f
#define FC_GELU_TAIL_CLAMP 8.5f
__device__ __forceinline__ float gelu_erf(float v) {
  const float a = fminf(fabsf(v), FC_GELU_TAIL_CLAMP);
  float p = fmaf(a, FC_GELU_TAIL_P6, FC_GELU_TAIL_P5);
  p = fmaf(a, p, FC_GELU_TAIL_P4);
  p = fmaf(a, p, FC_GELU_TAIL_P3);
  p = fmaf(a, p, FC_GELU_TAIL_P2);
  p = fmaf(a, p, FC_GELU_TAIL_P1);
  p = fmaf(a, p, FC_GELU_TAIL_P0);
  // max(v, 0) - |v| Phi(-|v|): v - v Phi(-|v|) for v >= 0, v Phi(-|v|) below
  return fmaf(-fabsf(v), __builtin_amdgcn_exp2f(p), fmaxf(v, 0.f));
}

template <int ACT>
__device__ __forceinline__ float mlp_activation(float v) {
  return ACT == 0 ? gelu_erf(v) : gelu_tanh(v);
}

// 16 bytes a lane from memory to LDS: `to` is the wavefront's, lane l's piece goes to
// to[l].  (A buffer load: of a global one the compiler assumes that it may touch LDS
// out of order, and waits for everything at the next use of any load.)
typedef __amdgpu_buffer_rsrc_t BufferPtr;
__device__ __forceinline__ BufferPtr buffer_of(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void load_to_lds(BufferPtr from, int lane_offset, int offset, half8* to) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void*)to, 16, lane_offset, offset,
                                           0, 0);
}
// Waits until at most N of the wavefront's vector memory accesses are on their way
// (they complete in order).
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N < 64, "six bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

// A barrier that leaves vector memory accesses on their way (__syncthreads waits for all
// of them where some write to LDS).
__device__ __forceinline__ void ring_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// what the lanes of a chunk read for the tokens its segment does not have
__device__ __align__(256) _Float16 g_zero_row[128];

template <int D, int HID, int ACT>
__global__ __launch_bounds__((MlpShape<D, HID>::kThreads), (MlpShape<D, HID>::kWavesPerSimd))
void mlp_compress_kernel(BatchParams p, MlpParams mp) {
  constexpr int kMlpRowsPerTile = MlpShape<D, HID>::kRows;
  constexpr int MT1 = HID / 16;               // 16-row tiles of hidden units
  constexpr int MT2 = D / 16;                 // 16-row tiles of output channels
  constexpr int S2 = HID / 32;                // K slabs of the second product
  constexpr int SPT = D / 32;                 // K slabs of the first product per token
  constexpr int GPT = 4;                      // groups of W1 per token, and of W2
  constexpr int GO = SPT * MT1 / GPT;         // A operands (W1 tiles) per group: a slab of them or half of one
  constexpr int kMlpThreads = MlpShape<D, HID>::kThreads;
  constexpr int PPG = GO * 64 / kMlpThreads;  // 16-byte pieces of a group per thread
  constexpr int QUAD = GPT * GO * 64;         // pieces of four groups
  constexpr int AR = 4;                       // A operands in flight from LDS
  // tokens of B operands held in registers (at 128 channels and 256 hidden units there
  // are none for a second one: with two the loop spills)
  constexpr int XR = D == 128 && HID == 256 ? 1 : 2;
  constexpr int RT = 8 + XR;                  // tokens in the table of pool rows
  static_assert(GO % AR == 0 && PPG >= 1, "tiling");
  extern __shared__ __align__(16) unsigned char smem[];
  half8* sm_w = reinterpret_cast<half8*>(smem);                      // [2 GPT groups][GO][64]
  float* sm_b1 = reinterpret_cast<float*>(sm_w + 2 * QUAD);          // [HID]
  float* sm_b2 = sm_b1 + HID;                                        // [D]
  half8* sm_x = reinterpret_cast<half8*>(sm_b2 + D);                 // [wavefronts][32 rows][4]
  uint32_t* sm_rows = reinterpret_cast<uint32_t*>(sm_x + MlpShape<D, HID>::kWaves * 128);  // [wavefronts][RT + 1][32]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31;  // the chunk that the lane looks things up for
  const int c16 = lane & 15;  // chunk within a 16-wide column tile
  const int q4 = lane >> 4;   // which 8 of the slab's 32 contraction positions
  const int k = mp.k;
  const int n_units = p.n_layers * p.n_heads * 2;
  const int blk_rows = 2 * p.n_heads * 16;  // a block's rows of D elements

  // Persistent: a workgroup walks tiles blockIdx.x, blockIdx.x + gridDim.x, ...
  // The walk is software-pipelined over tiles, because what a tile needs before
  // its first MFMA (which job it belongs to, where its chunks start, the block
  // ids of its rows, its first pool rows) is a chain of dependent memory
  // accesses of several microseconds: while tile T runs its GELU, second
  // product and store, in which nothing else is loaded, the chain of tile
  // T + gridDim.x is walked, so that its first rows are on their way when it
  // starts.
  struct Lane {            // what a lane knows about its chunk of a tile
    int s0, n_valid;       // first token of the chunk, tokens it has (< k at a segment's end)
    uint32_t base_row;     // pool row (units of D elements) of slot 0 of block 0 of its (layer, head, K|V)
  };
  auto find_job = [&](int tile, int& ji) {  // jobs are sorted by tile_start; ji only moves up
    while (ji + 1 < mp.n_jobs && load_uniform(&mp.jobs[ji + 1].tile_start) <= tile) ++ji;
  };
  auto lane_of = [&](int tile, const MlpJob& job, const ReqDesc& rd) -> Lane {
    Lane ln;
    const long long n_rows = (long long)n_units * job.chunks;
    const long long row = (long long)(tile - job.tile_start) * kMlpRowsPerTile +
                          wave * 32 + col;
    int unit = 0;
    ln.s0 = 0;
    ln.n_valid = 0;
    if (row < n_rows) {
      unit = (int)(row / job.chunks);
      const int cl = (int)(row - (long long)unit * job.chunks);
      int seg_end;
      if (job.modality == 1) {
        ln.s0 = rd.img_begin + cl * k;
        seg_end = rd.img_end;
      } else if (cl < rd.chunks_text0) {
        ln.s0 = cl * k;
        seg_end = rd.img_begin;
      } else {
        ln.s0 = rd.img_end + (cl - rd.chunks_text0) * k;
        seg_end = rd.seq_len;
      }
      ln.n_valid = min(k, seg_end - ln.s0);
    }
    const int lh = unit >> 1;
    const int layer = lh / p.n_heads;
    // (the pool has fewer than 2^32 - 1 rows: checked by the launcher)
    ln.base_row = (uint32_t)(layer * p.n_blocks) * (uint32_t)blk_rows +
                  (uint32_t)((unit & 1) * (p.n_heads * 16) + (lh - layer * p.n_heads) * 16);
    return ln;
  };
  // The pool rows of a chunk's tokens (absolute, in units of D elements,
  // kNoRow = no such token) go to a table in LDS, the wavefront's own: registers
  // are needed for data in flight, and a lookup inside the pipelined loop would
  // make every iteration wait for all loads in flight.  A chunk has at most 8
  // tokens, so it lies in at most two blocks: bid[0], bid[1].  The last line of the
  // table is where the tile's results go.
  uint32_t* const my_rows = sm_rows + wave * (RT + 1) * 32;
  auto write_rows = [&](const Lane& ln, const int (&bid)[2]) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int tok = ln.s0 + t;
      const int blk = (tok >> 4) == (ln.s0 >> 4) ? bid[0] : bid[1];
      my_rows[t * 32 + col] =
          t < ln.n_valid ? ln.base_row + (uint32_t)clamp_block(blk, p.n_blocks) * (uint32_t)blk_rows +
                               (uint32_t)(tok & 15)
                         : kNoRow;
    }
    wave_lds_barrier();  // (lanes read what others wrote)
  };

  // Every load of the pipelined loop is unconditional (a load under a branch
  // makes the compiler wait for ALL loads in flight at the next use): a token
  // that does not exist (past the end of a chunk's segment, or a lane without
  // a chunk) reads a row of zeros instead.
  // A token's rows are fetched 64 bytes (a slab) at a time, four neighbouring lanes a
  // row (rows lane / 4 and 16 + lane / 4 of the tile's 32), and go through 2 KB of LDS of
  // the wavefront's own into operand order: lane (q4, c16) gets channels [32 j + 8 q4, +8)
  // of rows c16 and 16 + c16.  Loaded in operand order, every 16 bytes are an access of
  // their own to the L1.
  struct RowPair {
    const _Float16* at[2];
  };
  auto rows_of = [&](int t) -> RowPair {
    RowPair r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t ri = my_rows[t * 32 + 16 * i + (lane >> 2)];
      r.at[i] = (ri != kNoRow ? p.kv + (size_t)ri * D : g_zero_row) + (lane & 3) * 8;
    }
    return r;
  };
  half8* const tile_x = sm_x + wave * 128;  // a piece of row r lies at its index ^ (r / 2 % 4)
  half8* const put_x = tile_x + (lane >> 2) * 4 + ((lane & 3) ^ ((lane >> 3) & 3));
  const half8* const got_x = tile_x + c16 * 4 + (q4 ^ ((c16 >> 1) & 3));
  auto load_x = [&](const RowPair& r, int j, half8 (&x)[SPT][2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) x[j][i] = load_half8(r.at[i] + j * 32);
  };
  auto arrange_x = [&](half8 (&x)[2]) {
    put_x[0] = x[0];
    put_x[64] = x[1];
    wave_lds_barrier();
    x[0] = got_x[0];
    x[1] = got_x[64];
    wave_lds_barrier();
  };
  // vector memory accesses that the rows add to n groups in a row, at least
  constexpr auto row_loads = [](int n) { return GO == MT1 ? 2 * n : 2 * (n / 2); };

  // Group g of four (a quad: a token's slabs of W1, or all of W2) to its place in the
  // ring, straight from memory.
  auto fetch = [&](const _Float16* w, int quad, int half, int g) {
    const BufferPtr buffer = buffer_of(w, (k + 1) * QUAD * 16);
#pragma unroll
    for (int i = 0; i < PPG; ++i) {
      const int at = g * GO * 64 + i * kMlpThreads;
      load_to_lds(buffer, tid * 16, (quad * QUAD + at) * 16, sm_w + half * QUAD + at + wave * 64);
    }
  };

  int cur_m = -1;
  int ji = 0;
  find_job(blockIdx.x, ji);
  MlpJob job = load_uniform(mp.jobs + ji);
  ReqDesc rd = load_uniform(p.descs + job.desc);
  half8 xq[XR][SPT][2];
  // the first tile's chain, not overlapped with anything
  {
    const Lane ln = lane_of(blockIdx.x, job, rd);
    const int32_t* ids = p.old_ids + rd.old_off;
    const int last = ln.s0 + max(ln.n_valid, 1) - 1;
    const int bid[2] = {ids[ln.s0 >> 4], ids[last >> 4]};
    write_rows(ln, bid);
  }
  int half = 0;  // of the ring: where the quad lies that comes next
#pragma unroll
  for (int g = 0; g < GPT; ++g) fetch(mp.w1p[job.modality], 0, half, g);
  wait_loads<0>();
  auto load_first_tokens = [&] {
#pragma unroll
    for (int u = 0; u < XR; ++u) {
      const RowPair r = rows_of(u);
#pragma unroll
      for (int j = 0; j < SPT; ++j) load_x(r, j, xq[u]);
    }
  };
  load_first_tokens();

  for (int tile = blockIdx.x; tile < mp.n_tiles; tile += gridDim.x) {
    // the tile after this one (the last tile prefetches itself again: loads in
    // bounds that nobody uses, so that nothing here sits under a branch)
    const int tile_n = tile + (int)gridDim.x < mp.n_tiles ? tile + (int)gridDim.x : tile;
    int ji_n = ji;
    find_job(tile_n, ji_n);
    const MlpJob job_n = load_uniform(mp.jobs + ji_n);
    const ReqDesc rd_n = load_uniform(p.descs + job_n.desc);

    const int m = job.modality;
    // k quads of W1, then one of W2, then the next tile's
    const _Float16 *const w = mp.w1p[m], *const w_n = mp.w1p[job_n.modality];
    auto fetch_ahead = [&](int q, int half_, int g) {
      fetch(q <= k ? w : w_n, q <= k ? q : q - k - 1, half_, g);
    };
    ring_barrier();  // the first quad is in LDS; nobody reads W2 or the biases of the previous tile any more
    if (m != cur_m) {  // uniform (the next barrier makes them visible)
      for (int i = tid; i < HID; i += kMlpThreads) sm_b1[i] = mp.b1[m][i];
      for (int i = tid; i < D; i += kMlpThreads) sm_b2[i] = mp.b2[m][i];
      cur_m = m;
    }

    // ---- first product: H^T tile [HID x 32] per wavefront -----------------
    // The weights are a stream of quads of four groups: k quads of W1, W2, the next
    // tile's.  The ring holds two quads; the place of a group is filled again as soon as
    // all wavefronts are done with it, one barrier per group, and a group is visible one
    // barrier before its turn, so A operands are read AR ahead of their use, across group
    // boundaries.  A scattered pool row takes microseconds to arrive (address translation,
    // HBM): the B operands of XR tokens are held, and those of a finished slab are
    // replaced at once by the same slab XR tokens on.
    floatx4 acc[MT1][2];
#pragma unroll
    for (int mt = 0; mt < MT1; ++mt) acc[mt][0] = acc[mt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    half8 ar[AR];
#pragma unroll
    for (int g = 0; g < GPT - 1; ++g) fetch_ahead(1, half ^ 1, g);
#pragma unroll
    for (int n = 0; n < AR; ++n) ar[n] = sm_w[half * QUAD + n * 64 + lane];
    wait_loads<3 * PPG>();  // the first tokens' rows
    arrange_x(xq[0][0]);
    int t = 0;
    auto token = [&](auto slot) {
      constexpr int u = decltype(slot)::value;
      const RowPair new_rows = rows_of(t + XR);
      const half8* const mine = sm_w + half * QUAD + lane;
      const half8* const next = sm_w + (half ^ 1) * QUAD + lane;
#pragma unroll
      for (int jj = 0; jj < GPT; ++jj) {
        // the place of the group before this one is free: the group seven on
        if (jj == 0)
          fetch_ahead(t + 1, half ^ 1, GPT - 1);
        else
          fetch_ahead(t + 2, half, jj - 1);
        const int slab = jj * GO / MT1;
        const bool last_of_slab = (jj + 1) * GO % MT1 == 0;
        if (last_of_slab) {  // the rows of the next slab
          if (slab + 1 < SPT)
            arrange_x(xq[u][slab + 1]);
          else
            arrange_x(xq[(u + 1) % XR][0]);
        }
        const half8* w1s = mine + jj * GO * 64;
        const half8* w1f = jj + 1 < GPT ? mine + (jj + 1) * GO * 64 : next;  // visible since the last barrier
#pragma unroll
        for (int n = 0; n < GO; ++n) {
          const half8 a = ar[n % AR];
          const int nn = n + AR;
          ar[n % AR] = (nn < GO) ? w1s[nn * 64] : w1f[(nn - GO) * 64];
          const int mt = (jj * GO + n) % MT1;
#pragma unroll
          for (int ct = 0; ct < 2; ++ct)
            acc[mt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, xq[u][slab][ct], acc[mt][ct], 0, 0, 0);
          // pin the issue order "one LDS read, two MFMAs": left alone, the
          // scheduler sinks each read to just before its use
          __builtin_amdgcn_sched_barrier(0);
        }
        // this slab's operands are done: fetch the same channels XR tokens on
        if (last_of_slab) load_x(new_rows, slab, xq[u]);
        // in LDS at the next barrier: the group after the next one (requested five groups
        // ago, or together with two others at the beginning of the tile), or all of W2
        // (the last of it three groups ago).  What has been requested since may be on its way.
        if (jj == 2 && t == 0) {
          wait_loads<5 * PPG + row_loads(3)>();
        } else if (jj == 0) {
          wait_loads<5 * PPG + row_loads(5)>();
        } else if (jj + 1 < GPT) {
          wait_loads<5 * PPG + row_loads(6)>();
        } else if (t + 1 < k) {
          wait_loads<5 * PPG + row_loads(4)>();
        } else {
          wait_loads<3 * PPG + row_loads(4)>();
        }
        ring_barrier();  // and nobody reads this group any more
      }
      half ^= 1;
      ++t;
      asm volatile("" : "+s"(t));  // (not known to be 0 in a first copy of the loop)
    };
    // (two exits and no test at the top: a path that leaves after the first token and
    // meets the other one before it does would make the compiler wait for loads in
    // flight at the top)
    for (;;) {
      token(std::integral_constant<int, 0>{});
      if (t >= k) break;  // uniform
      if constexpr (XR == 2) {
        token(std::integral_constant<int, 1>{});
        if (t >= k) break;
      }
    }
    fetch_ahead(k + 1, half ^ 1, GPT - 1);

    // ---- the next tile's chain, first half: where its chunks are, their block ids
    const Lane ln_n = lane_of(tile_n, job_n, rd_n);
    const int32_t* ids_n = p.old_ids + rd_n.old_off;
    const int bid_n[2] = {ids_n[ln_n.s0 >> 4], ids_n[(ln_n.s0 + max(ln_n.n_valid, 1) - 1) >> 4]};
    // ---- where this tile's rows go: looked up here, behind the next tile's rows the block
    // id would arrive only after all of them
    const long long row = (long long)(tile - job.tile_start) * kMlpRowsPerTile + wave * 32 + col;
    const bool has_row = row < (long long)n_units * job.chunks;
    const int unit = has_row ? (int)row / job.chunks : 0;
    const int cl = has_row ? (int)row - unit * job.chunks : 0;
    const int o = (m == 1) ? rd.chunks_text0 + cl : (cl < rd.chunks_text0 ? cl : rd.chunks_image + cl);
    const int out_blk = p.new_ids[rd.new_off + (o >> 4)];

    // ---- bias, gelu, fp16: each pair of result tiles becomes a B operand of
    // the second product and stays in registers.  Half-way through, when half
    // of the accumulators are gone, the next tile's row table is written (this
    // tile's is no longer read) and its first XR tokens are requested: they travel while the rest of the
    // GELU, the second product and the store keep the other units busy.
    half8 hb[S2][2];
    auto gelu_slab = [&](int sl) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const floatx4 b1 = *reinterpret_cast<const floatx4*>(sm_b1 + mlp_hidden_unit(sl, q4, 4 * h));
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            hb[sl][ct][4 * h + r] = (_Float16)mlp_activation<ACT>(acc[2 * sl + h][ct][r] + b1[r]);
      }
    };
#pragma unroll
    for (int sl = 0; sl < S2 / 2; ++sl) gelu_slab(sl);
    {
      const int lh = unit >> 1;
      const int layer = lh / p.n_heads;
      my_rows[RT * 32 + col] =
          has_row ? (uint32_t)(layer * p.n_blocks + clamp_block(out_blk, p.n_blocks)) * (uint32_t)blk_rows +
                        (uint32_t)((unit & 1) * (p.n_heads * 16) + (lh - layer * p.n_heads) * 16 + (o & 15))
                  : kNoRow;
    }
    write_rows(ln_n, bid_n);
    wait_loads<0>();  // the next tile's first quad (the block ids, requested after it, have arrived)
    load_first_tokens();
    __builtin_amdgcn_sched_barrier(0);  // (left alone, the scheduler sinks the loads to the end)
#pragma unroll
    for (int sl = S2 / 2; sl < S2; ++sl) gelu_slab(sl);

    // ---- second product, Y^T tile [D x 32]
    floatx4 acc2[MT2][2];
#pragma unroll
    for (int ot = 0; ot < MT2; ++ot) acc2[ot][0] = acc2[ot][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sl = 0; sl < S2; ++sl)
#pragma unroll
      for (int ot = 0; ot < MT2; ++ot) {
        const half8 w = sm_w[half * QUAD + (sl * MT2 + ot) * 64 + lane];
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
          acc2[ot][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, hb[sl][ct], acc2[ot][ct], 0, 0, 0);
      }

    // ---- bias, fp16, store the rows into the request's new blocks -------------
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const uint32_t to = my_rows[RT * 32 + ct * 16 + c16];
      if (to != kNoRow) {
        _Float16* const dst = p.kv + (size_t)to * D + 8 * q4;
#pragma unroll
        for (int g = 0; g < MT2 / 2; ++g) {
          half8 y;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const floatx4 b2 = *reinterpret_cast<const floatx4*>(sm_b2 + 32 * g + 8 * q4 + 4 * h);
#pragma unroll
            for (int r = 0; r < 4; ++r) y[4 * h + r] = (_Float16)(acc2[2 * g + h][ct][r] + b2[r]);
          }
          store_half8(dst + 32 * g, y);
        }
      }
    }
    half ^= 1;
    job = job_n;
    rd = rd_n;
    ji = ji_n;
  }
  // (the last workgroups: they have a tile less, if any have)
  if (p.main_reclaims)
    for (int r = (int)gridDim.x - 1 - (int)blockIdx.x; r < p.n_comp; r += gridDim.x) reclaim_request(p, p.descs[r]);
  wait_loads<0>();  // nothing may arrive in the LDS of a workgroup that has ended
}

template <int D, int HID>
static constexpr size_t mlp_lds_bytes() {
  return 2 * (size_t)(D / 16) * (HID / 32) * 64 * 16 +
         (size_t)(HID + D) * sizeof(float) + MlpShape<D, HID>::kWaves * (size_t)(2048 + (8 + 2 + 1) * 32 * sizeof(int));
}

template <int D, int HID>
static hipError_t mlp_setup_one() {
  static_assert(mlp_lds_bytes<D, HID>() * MlpShape<D, HID>::kPerCu <= 160 * 1024, "LDS of a CU");
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_compress_kernel<D, HID, 0>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)mlp_lds_bytes<D, HID>());
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_compress_kernel<D, HID, 1>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)mlp_lds_bytes<D, HID>());
  return e;
}

hipError_t mlp_one_time_setup() {
  hipError_t e = mlp_setup_one<128, 256>();
  if (e == hipSuccess) e = mlp_setup_one<128, 128>();
  if (e == hipSuccess) e = mlp_setup_one<64, 256>();
  if (e == hipSuccess) e = mlp_setup_one<64, 128>();
  return e;
}

template <int D, int HID>
static hipError_t mlp_launch_one(const BatchParams& p, const MlpParams& mp, hipStream_t s) {
  constexpr int threads = MlpShape<D, HID>::kThreads;
  const unsigned grid = (unsigned)std::min(mp.n_tiles, mp.max_grid);
  if (mp.activation == 0)
    mlp_compress_kernel<D, HID, 0><<<grid, threads, mlp_lds_bytes<D, HID>(), s>>>(p, mp);
  else
    mlp_compress_kernel<D, HID, 1><<<grid, threads, mlp_lds_bytes<D, HID>(), s>>>(p, mp);
  return hipGetLastError();
}

hipError_t launch_mlp_compress(const BatchParams& p, const MlpParams& mp, hipStream_t s) {
  if (mp.n_tiles <= 0) return hipSuccess;
  // the kernel addresses pool rows (head_dim elements each) with 32 bits
  if ((unsigned long long)p.n_layers * p.n_blocks * 2 * p.n_heads * 16 >= kNoRow)
    return hipErrorInvalidValue;
  if (p.head_dim == 128 && mp.hidden == 256) return mlp_launch_one<128, 256>(p, mp, s);
  if (p.head_dim == 128 && mp.hidden == 128) return mlp_launch_one<128, 128>(p, mp, s);
  if (p.head_dim == 64 && mp.hidden == 256) return mlp_launch_one<64, 256>(p, mp, s);
  if (p.head_dim == 64 && mp.hidden == 128) return mlp_launch_one<64, 128>(p, mp, s);
  return hipErrorInvalidValue;
}

}  // namespace fc
