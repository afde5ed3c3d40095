// Device code of one (request, layer, head): scores, selection, copy, and the
// fused kernels made of them.  Included by the translation units that
// instantiate the kernels (one per head size and workgroup shape, so that they
// compile side by side).
#pragma once

#include <type_traits>

#include "fc_device.h"

namespace fc {

// ---------------------------------------------------------------------------
// SnapKV-style observation-window score
// ---------------------------------------------------------------------------
//
// One workgroup per (request, layer, head).  A wavefront takes pool blocks
// (16 tokens) round-robin and feeds them to v_mfma_f32_16x16x32_f16: lane l holds
// 8 consecutive channels [32*ks + 8*(l/16), +8) of token l%16, which is both the
// A-operand layout (rows = tokens) and the B-operand layout (columns = tokens) of
// that instruction (KeyBlocks: how they get there).
//
// Pass 1 (A = keys, B = queries): the 16x16 result has the window query on the
// lane (l%16) and 4 tokens in the lane's registers, so every lane keeps an
// online (max, sum-of-exp) pair for its query with no cross-lane traffic.
// Pass 2 (A = queries, B = keys): the result has the token on the lane and 4
// queries in registers, so the sum over window queries is an in-lane add plus
// two cross-lane adds.  Softmax uses exp2 with scale*log2(e) folded in.
//
// The un-pooled column sums of the prefix go to store(): LDS in the fused kernels,
// raw_scores in the others; pooling and the forced window are the selection's.

// Wavefronts of a workgroup of the fused kernels.  Four, so that three or four
// workgroups share a CU and the selection of one overlaps the streaming of the
// others; or as many as one workgroup can have (a "wide" workgroup, at most one
// per CU), for heads whose scores take most of the LDS and for launches with too
// few heads to fill the chip.  16 where the registers allow four wavefronts per
// SIMD (128 each), else 12 (168 each).
static constexpr int kNarrow = kWaves;
template <int D, int NT>
static constexpr int kWide = NT <= 2 ? 16 : 12;
// longest head a workgroup of WV wavefronts takes
template <int WV>
static constexpr int kMaxLen = WV == kNarrow ? kFusedMaxLen : kFusedWideMaxLen;

// Epochs of the bound-keeping first pass: wavefront w takes blocks w, w + WV,
// ...; its t-th block (step t) belongs to epoch 0 (t = 0), 1 (t = 1), then 2, and
// to a new one at every multiple of seg: the references are renewed before t = 1,
// 2 and every multiple of seg, by all wavefronts together.  Every 256 tokens with
// four wavefronts, every 512 to 576 with wide workgroups (1024 to 1152 for their
// longest heads, whose per-epoch numbers must fit next to 32768 scores in LDS).
template <int WV>
__host__ __device__ constexpr int bound_seg(int len) {
  return WV == kNarrow ? 4 : (WV == 16 ? 2 : 3) * (len > kFusedWideMaxLen / 2 ? 2 : 1);
}
__host__ __device__ constexpr int bound_epoch_of_step(int t, int seg) {
  return t < 2 ? t : t / seg + (seg > 2 ? 2 : 1);
}
__host__ __device__ constexpr bool bound_renews_before(int t, int seg) {
  return t == 1 || t == 2 || (t >= seg && t % seg == 0);
}
template <int WV>
__host__ __device__ constexpr int bound_max_epochs() {
  const int half = kMaxLen<WV> / (WV == kNarrow ? 1 : 2), full = kMaxLen<WV>;
  const int a = 1 + bound_epoch_of_step((half / 16 + WV - 1) / WV, bound_seg<WV>(half));
  const int b = 1 + bound_epoch_of_step((full / 16 + WV - 1) / WV, bound_seg<WV>(full));
  return a > b ? a : b;
}
// (the first step lies before the window)
template <int WV>
static constexpr int kBoundMinLen = 16 * WV + 64;

// A block's keys of one (layer, head), from memory to the operand layout of the
// products: k[ks] of lane (q4, c16) = channels [32 ks + 8 q4, +8) of token c16.
// Loaded straight into that layout, 16 rows of 64 bytes an instruction, or (kLines)
// eight rows of 128 bytes, whole cache lines, which arrange() then hands to the lanes
// through 2 KB of LDS of the wavefront's own, 64 channels at a time.  Only with whole
// lines does the non-temporal hint give anything: a plain pass over 2 GB of K blocks
// reads 5.95 TB/s without it in either layout, with it 6.0 straight and 6.6 in lines.
// So lines are for keys that are not wanted again (second pass of a call with scores,
// 4096 heads of 3000 tokens, window 64: 1638 -> 1494 us; the single pass of a call with
// the log-sum-exps), and passes that leave the keys to the caches load straight.  Wide
// workgroups do in any case: their wavefronts wait longer for the LDS than lines save
// (pruned heads of 10000 tokens, 1024 of them, 64 channels: 603 us straight, 653 in lines).
static constexpr int kTilePieces = 128;  // 16-byte pieces of a wavefront's tile
template <int WV, bool kUsed = true>
struct KeyTiles {
  half8 piece[kUsed && WV == kNarrow ? WV * kTilePieces : 1];
};
template <int D, int WV, bool kWanted>
struct KeyBlocks {
  static constexpr bool kLines = kWanted && WV == kNarrow;
  const _Float16* base;      // this lane's channels of token 0 of block 0
  const _Float16* row_base;  // of the first token it loads of a block
  size_t stride;
  int n_blocks;
  half8* put;         // where this lane's piece of rows 0 .. 7 goes (a piece of row r lies at its index ^ (r & 7))
  const half8* got0;  // its operand of the first 32 of 64 channels,
  const half8* got1;  // of the second
  // tiles: of the workgroup (nullptr: no lines)
  __device__ __forceinline__ KeyBlocks(const BatchParams& p, int lh, half8* tiles) : n_blocks(p.n_blocks) {
    const int layer = lh / p.n_heads, head = lh - layer * p.n_heads;
    const int lane = threadIdx.x & 63;
    const int row = lane >> 3, c16 = lane & 15, q4 = lane >> 4;
    stride = (size_t)2 * p.n_heads * 16 * D;
    base = p.kv + (size_t)layer * p.n_blocks * stride + (size_t)head * 16 * D + (kLines ? (lane & 7) * 8 : q4 * 8);
    row_base = base + (kLines ? row : c16) * D;
    if constexpr (kLines) {
      half8* const mine = tiles + (threadIdx.x >> 6) * kTilePieces;
      put = mine + row * 8 + ((lane & 7) ^ row);
      got0 = mine + c16 * 8 + (q4 ^ (c16 & 7));
      got1 = mine + c16 * 8 + ((4 + q4) ^ (c16 & 7));
    }
  }
  __device__ __forceinline__ size_t block(int id) const { return (size_t)clamp_block(id, n_blocks) * stride; }
  template <bool kNonTemporal>
  static __device__ __forceinline__ half8 piece(const _Float16* at) {
    return kNonTemporal ? load_half8_nt(at) : load_half8(at);
  }
  template <bool kNonTemporal>
  __device__ __forceinline__ void load(int id, half8 (&k)[D / 32]) const {
    // (the block is the wavefront's: scalar address arithmetic)
    const _Float16* kp = row_base + block(__builtin_amdgcn_readfirstlane(id));
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
      k[i] = piece<kNonTemporal>(kLines ? kp + (i & 1) * 8 * D + (i >> 1) * 64 : kp + i * 32);
  }
  // The same of sixteen tokens from anywhere in the head: lane % 16 names one in tok.
  __device__ __forceinline__ void load_rows(int tok, const int32_t* ids, half8 (&k)[D / 32]) const {
    const _Float16* at[2];
#pragma unroll
    for (int i = 0; i < (kLines ? 2 : 1); ++i) {
      const int t = kLines ? __shfl(tok, ((threadIdx.x & 63) >> 3) + 8 * i) : tok;
      at[i] = base + block(ids[t >> 4]) + (t & 15) * D;
    }
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
      k[i] = piece<true>(kLines ? at[i & 1] + (i >> 1) * 64 : at[0] + i * 32);
  }
  __device__ __forceinline__ void arrange(half8 (&k)[D / 32]) const {
    if constexpr (kLines) {
#pragma unroll
      for (int i = 0; i < D / 32; i += 2) {
        put[0] = k[i];
        put[64] = k[i + 1];
        wave_lds_barrier();
        k[i] = *got0;
        k[i + 1] = *got1;
        wave_lds_barrier();
      }
    }
  }
};

template <int WV>
struct ScoreShared {
  // partial (max, sum) pairs per wavefront and row: those of the four lane groups,
  // or (wide workgroups, whose LDS is short) already merged within the wavefront
  static constexpr int kParts = WV == kNarrow ? 4 : 1;
  struct Pairs {
    float m[WV][kParts][64];
    float z[WV][kParts][64];
  };
  float fin[64];
  // (one place: side by side they would exceed what the selection needs, which is what
  // says how many workgroups a CU takes: scores of 2048 heads of 4700-5600 tokens, 64
  // channels, window 32, 702 us with them apart, 640 so)
  union {
    Pairs rows;          // until fin is known
    KeyTiles<WV> tiles;  // from there on
  };
};

// Scores one (request, layer, head); store(j, a_j) receives the un-pooled
// column sum of every prefix token j.  All threads of the workgroup call.
// `old_ids` are the request's pre-compression block ids (global or LDS copy).
// The window queries of a (request, layer, head) in MFMA operand layout (rows
// past the window are zero), resident in registers for every pass over K.
template <int D, int NT>
__device__ __forceinline__ void load_window_queries(const BatchParams& p, const ReqDesc& rd, int lh,
                                                    half8 (&qreg)[NT][D / 32]) {
  constexpr int KS = D / 32;
  const int lane = threadIdx.x & 63;
  const int c16 = lane & 15;
  const int q4 = lane >> 4;
  const int W = rd.window;
  const _Float16* qbase = p.q_window + rd.q_off + (size_t)lh * W * D;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int row = nt * 16 + c16;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      half8 z = {0, 0, 0, 0, 0, 0, 0, 0};
      qreg[nt][ks] = (row < W) ? load_half8(qbase + (size_t)row * D + ks * 32 + q4 * 8) : z;
    }
  }
}

// Pass 1 over blocks [b0, b1): every lane's online (max, sum) of its query rows'
// logits -> sh.m, sh.z.  ids: the block ids, indexed from block 0.
template <int D, int NT, int WV, bool kLaneAnew>
__device__ __forceinline__ void snapkv_rows(const BatchParams& p, const ReqDesc& rd, int lh,
                                            const int32_t* ids, int b0, int b1, ScoreShared<WV>& sh,
                                            const half8 (&qreg)[NT][D / 32]) {
  constexpr int KS = D / 32;
  const int L = rd.seq_len;
  const int W = rd.window;  // <= 16 NT; the rows past it are padding
  const int lane = lane_number<kLaneAnew>();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15;
  const int q4 = lane >> 4;
  const KeyBlocks<D, WV, false> keys(p, lh, nullptr);
  const float c = p.scale_log2e;
  const int n_unmasked = (L - W) >> 4;  // blocks that lie wholly before the window
  float m[NT], z[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m[nt] = -3.0e38f;
    z[nt] = 0.f;
  }
  stream_tiles<half8[KS]>(
      own_tiles(b1 - b0, wave, WV),
      [&](int i, half8(&k)[KS]) { keys.template load<false>(ids[b0 + wave + WV * i], k); },
      [&](int i, const half8(&kc)[KS]) {
        const int b = b0 + wave + WV * i;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(kc[ks], qreg[nt][ks], acc, 0, 0, 0);
          float t[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) t[r] = acc[r] * c;
          if (b >= n_unmasked) {
            // query i at position L-W+i sees tokens <= its own position
            const int limit = L - W + nt * 16 + c16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int tok = b * 16 + q4 * 4 + r;
              if (tok > limit) t[r] = -INFINITY;
            }
          }
          const float bm = fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]));
          const float mn = fmaxf(m[nt], bm);
          float zz = z[nt] * __builtin_amdgcn_exp2f(m[nt] - mn);
#pragma unroll
          for (int r = 0; r < 4; ++r) zz += __builtin_amdgcn_exp2f(t[r] - mn);
          z[nt] = zz;
          m[nt] = mn;
        }
      });
  constexpr int kParts = ScoreShared<WV>::kParts;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if constexpr (kParts == 1) {
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float mo = __shfl_xor(m[nt], o), zo = __shfl_xor(z[nt], o);
        const float mm = fmaxf(m[nt], mo);
        z[nt] = z[nt] * __builtin_amdgcn_exp2f(m[nt] - mm) + zo * __builtin_amdgcn_exp2f(mo - mm);
        m[nt] = mm;
      }
    }
    if (q4 < kParts) {
      sh.rows.m[wave][q4 % kParts][nt * 16 + c16] = m[nt];
      sh.rows.z[wave][q4 % kParts][nt * 16 + c16] = z[nt];
    }
  }
}

// The workgroup's (max, sum) of a row from the partial pairs of snapkv_rows.
template <int WV>
__device__ __forceinline__ void merged_row(const ScoreShared<WV>& sh, int row, float& mm, float& zz) {
  constexpr int kParts = ScoreShared<WV>::kParts;
  mm = -3.0e38f;
  for (int w = 0; w < WV; ++w)
    for (int q = 0; q < kParts; ++q) mm = fmaxf(mm, sh.rows.m[w][q][row]);
  zz = 0.f;
  for (int w = 0; w < WV; ++w)
    for (int q = 0; q < kParts; ++q)
      zz += sh.rows.z[w][q][row] * __builtin_amdgcn_exp2f(sh.rows.m[w][q][row] - mm);
}

// Pass 2 over blocks [b0, b1) of the prefix: column sums of the soft-maxed rows;
// fin: log2 of every row's denominator.
template <int D, int NT, int WV, bool kLaneAnew, typename Store>
__device__ __forceinline__ void snapkv_columns(const BatchParams& p, const ReqDesc& rd, int lh,
                                               const int32_t* ids, int b0, int b1, const float* fin, KeyTiles<WV>& tiles,
                                               const half8 (&qreg)[NT][D / 32], Store store) {
  constexpr int KS = D / 32;
  const int lane = lane_number<kLaneAnew>();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15;
  const int q4 = lane >> 4;
  const KeyBlocks<D, WV, true> keys(p, lh, tiles.piece);
  const float c = p.scale_log2e;
  const int n_prefix = rd.seq_len - rd.window;
  float mrow[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) mrow[nt][r] = fin[nt * 16 + q4 * 4 + r];
  // from the end of the prefix backwards: the blocks that the first pass read
  // last are the ones most likely to be still in a cache
  stream_tiles<half8[KS]>(
      own_tiles(b1 - b0, wave, WV),
      [&](int i, half8(&k)[KS]) { keys.template load<true>(ids[b1 - 1 - wave - WV * i], k); },
      [&](int i, half8(&kc)[KS]) {
        keys.arrange(kc);
        float colsum = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(qreg[nt][ks], kc[ks], acc, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            colsum += __builtin_amdgcn_exp2f(acc[r] * c - mrow[nt][r]);
        }
        colsum = quarter_sum(colsum);
        const int tok = (b1 - 1 - wave - WV * i) * 16 + c16;
        if (q4 == 0 && tok < n_prefix) store(tok, colsum);
      });
}

// where a unit's window rows begin in the packed log-sum-exps
template <int D>
__device__ __forceinline__ size_t lse_offset(const ReqDesc& rd, int lh) {
  return (size_t)(rd.q_off / D) + (size_t)lh * rd.window;
}

template <int D, int NT, int WV, bool kLaneAnew, typename Store>
__device__ __forceinline__ void snapkv_unit_q(const BatchParams& p, const ReqDesc& rd, int lh,
                                              const int32_t* old_ids, ScoreShared<WV>& sh,
                                              half8 (&qreg)[NT][D / 32], Store store) {
  const int L = rd.seq_len;
  const int W = rd.window;
  // log2 of every row's soft-max denominator goes to sh.fin: handed in by the
  // caller (natural log, from its attention kernel), or pass 1
  if (p.lse_window != nullptr) {  // uniform
    if (threadIdx.x < 64)
      sh.fin[threadIdx.x] = (int)threadIdx.x < W
                                ? p.lse_window[lse_offset<D>(rd, lh) + threadIdx.x] * 1.44269504088896340736f
                                : INFINITY;  // padded rows contribute exp2(-inf) = 0
    __syncthreads();
  } else {
    snapkv_rows<D, NT, WV, kLaneAnew>(p, rd, lh, old_ids, 0, (L + 15) >> 4, sh, qreg);
    __syncthreads();
    if (threadIdx.x < 64) {
      float mm, zz;
      merged_row<WV>(sh, threadIdx.x, mm, zz);
      sh.fin[threadIdx.x] = (int)threadIdx.x < W ? mm + log2f(zz)
                                                 : INFINITY;  // padded rows contribute exp2(-inf) = 0
    }
    __syncthreads();
  }
  if (p.lse_out != nullptr) {  // uniform: the caller asked for the denominators only
    if ((int)threadIdx.x < W)
      p.lse_out[lse_offset<D>(rd, lh) + threadIdx.x] = sh.fin[threadIdx.x] * 0.69314718055994530942f;
    return;
  }
  snapkv_columns<D, NT, WV, kLaneAnew>(p, rd, lh, old_ids, 0, (L - W + 15) >> 4, sh.fin, sh.tiles, qreg, store);
}

template <int D, int NT, int WV, bool kLaneAnew, typename Store>
__device__ __forceinline__ void snapkv_unit(const BatchParams& p, const ReqDesc& rd, int lh,
                                            const int32_t* old_ids, ScoreShared<WV>& sh, Store store) {
  half8 qreg[NT][D / 32];
  load_window_queries<D, NT>(p, rd, lh, qreg);
  snapkv_unit_q<D, NT, WV, kLaneAnew>(p, rd, lh, old_ids, sh, qreg, store);
}

// ---------------------------------------------------------------------------
// key-norm score: raw[j] = -||k_j||_2
// ---------------------------------------------------------------------------
//
// One workgroup per (request, layer, head); a wavefront reads one 16-token
// chunk with fully coalesced 128-bit loads (64 lanes x 16 B = 1 KiB per
// instruction) and reduces the squares over the lanes that share a row.

template <int D, int WV, typename Store>
__device__ __forceinline__ void knorm_unit(const BatchParams& p, const ReqDesc& rd, int lh,
                                           const int32_t* old_ids, int b0, int b1, Store store) {
  constexpr int LPR = D / 8;     // lanes per token row
  constexpr int RPI = 64 / LPR;  // rows per load instruction
  constexpr int NI = 16 / RPI;   // load instructions per block
  const int layer = lh / p.n_heads;
  const int head = lh - layer * p.n_heads;
  const int L = rd.seq_len;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t blk_stride = (size_t)2 * p.n_heads * 16 * D;
  const _Float16* kbase = p.kv + (size_t)layer * p.n_blocks * blk_stride +
                          (size_t)head * 16 * D + lane * 8;
  stream_tiles<half8[NI]>(
      own_tiles(b1 - b0, wave, WV),
      [&](int i, half8(&v)[NI]) {
        const int blk = clamp_block(__builtin_amdgcn_readfirstlane(old_ids[b0 + wave + WV * i]), p.n_blocks);
        const _Float16* kp = kbase + (size_t)blk * blk_stride;
#pragma unroll
        for (int k = 0; k < NI; ++k) v[k] = load_half8(kp + k * 512);
      },
      [&](int i, const half8(&v)[NI]) {
        const int b = b0 + wave + WV * i;
#pragma unroll
        for (int k = 0; k < NI; ++k) {
          float s = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = (float)v[k][e];
            s += x * x;
          }
#pragma unroll
          for (int o = 1; o < LPR; o <<= 1)  // (sums so far are equal in the lanes that a mirror exchanges)
            s += o == 1 ? from_lane<0xB1>(s) : o == 2 ? from_lane<0x4E>(s) : o == 4 ? from_lane<0x141>(s) : from_lane<0x140>(s);
          const int tok = b * 16 + k * RPI + lane / LPR;
          if ((lane % LPR) == 0 && tok < L) store(tok, -sqrtf(s));
        }
      });
}

// ---------------------------------------------------------------------------
// per-head top-budget selection
// ---------------------------------------------------------------------------
//
// One workgroup per (request, layer, head).  Only the tokens before the
// observation window compete (window tokens are always kept), so the kernel
// selects the budget-minus-window best of the prefix and appends the window.
//
//   1. the un-pooled scores lie in LDS; they are max-pooled and turned into
//      order-preserving 32-bit keys, in the same words;
//   2. the threshold (the k-th largest key) is found by a bucket select: 2048
//      linear buckets over a range that holds it (so the histogram is spread
//      even when every score shares its exponent), then the keys of the one
//      bucket that holds the threshold are compacted to a candidate list; up to
//      256 candidates are ranked against each other at once, a longer list is
//      refined with 2048 buckets per pass until a bucket is a single key;
//   3. the kept indices are emitted in ascending token order by a ballot /
//      popcount compaction in which keys equal to the threshold are admitted
//      in index order until the budget is met (ties go to the lower index).
//
// Ownership of tokens: a wavefront owns a contiguous segment (a multiple of 256
// tokens) and a lane four consecutive tokens of each 256.  What bounds this
// phase is LDS latency (one workgroup has four wavefronts and every step waits
// for its reads) and, for short heads, instruction fetch: the pooling window of a
// lane's four tokens comes from three 16-byte reads instead of seven dependent
// 4-byte reads per token, and every sweep is a loop over chunks whose per-token
// words stay in LDS (with the chunks unrolled and the words in registers the
// kernels were 200 KB of code against 64 KB of instruction cache, and a head of
// 640 tokens spent as long in the selection as one of 4000 should).

__device__ __forceinline__ uint32_t score_key(float s) {
  s += 0.0f;  // -0 and +0 compare equal, give them one key
  const uint32_t u = __float_as_uint(s);
  // (0 is the key of no token; what is not a number may have any bits, all of them too)
  return (u & 0x80000000u) ? max(~u, 1u) : (u | 0x80000000u);
}

static constexpr int kBuckets = 2048;
static constexpr int kBucketBits = 11;
static constexpr int kMaxCand = 2048;

typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32x4 lds_words4(const uint32_t* p) {
  return *reinterpret_cast<const uint32x4*>(p);
}
__device__ __forceinline__ void set_lds_words4(uint32_t* p, uint32x4 v) {
  *reinterpret_cast<uint32x4*>(p) = v;
}

// first token of a wavefront's segment
template <int WV>
__device__ __forceinline__ int segment_tokens(int n) {
  return (((n + WV - 1) / WV) + kChunk - 1) & ~(kChunk - 1);
}

// Replaces the words of a wavefront's segment [j0, j1) by f(c), which may read any
// word in reach of a pooling window (at most 31 tokens): a chunk is written only
// after the next one has been read, and the first and the last, which other
// wavefronts' windows reach, by finish(), after a barrier.
struct SegmentRewrite {
  uint32x4 first, pending;
  int n = 0;
  template <typename F>
  __device__ __forceinline__ void run(uint32_t* stage, int j0, int j1, F f) {
    const int lane4 = 4 * (threadIdx.x & 63);
    for (int base = j0; base < j1; base += kChunk, ++n) {  // uniform over the wavefront
      const int c = base + lane4;
      uint32x4 v = {0u, 0u, 0u, 0u};
      if (c < j1) v = f(c);
      wave_lds_barrier();  // (per lane the words read and written here never meet: nothing else keeps them in order)
      if (n == 0) {
        first = v;
      } else {
        if (n > 1) set_lds_words4(stage + c - kChunk, pending);  // (a chunk before the last is whole)
        pending = v;
      }
    }
  }
  __device__ __forceinline__ void finish(uint32_t* stage, int j0, int j1) const {
    const int c0 = j0 + 4 * (threadIdx.x & 63), c1 = c0 + (n - 1) * kChunk;
    if (n > 0 && c0 < j1) set_lds_words4(stage + c0, first);
    if (n > 1 && c1 < j1) set_lds_words4(stage + c1, pending);
  }
};

// four bits per lane -> one bit per token of the chunk at `base`
__device__ __forceinline__ void set_token_bits(uint32_t* map, int base, uint32_t nibble) {
  const int lane = threadIdx.x & 63;
  uint32_t bits = nibble << (4 * (lane & 7));
  bits |= from_lane_u32<0xB1>(bits);   // the other lane of the pair,
  bits |= from_lane_u32<0x4E>(bits);   // the other pair of the quad,
  bits |= from_lane_u32<0x141>(bits);  // the other quad of the eight
  if ((lane & 7) == 0) map[base / 32 + (lane >> 3)] = bits;
}
__device__ __forceinline__ uint32_t token_bits(const uint32_t* map, int base) {
  const int lane = threadIdx.x & 63;
  return (map[base / 32 + (lane >> 3)] >> (4 * (lane & 7))) & 0xFu;
}

// Writes `front` and `back` to the words around stage[0 .. n) that pooling reads.
__device__ __forceinline__ void fill_stage_margins(uint32_t* stage, int n, uint32_t front, uint32_t back) {
  if (threadIdx.x < kStageFront) stage[(int)threadIdx.x - kStageFront] = front;
  if (threadIdx.x < 8) stage[n + threadIdx.x] = back;  // n + 7 < the padded length + 8
}

// (begin(w): what a maximum or minimum that holds w may begin with.  A constant for
// the packed bounds: with w the 64-channel pruned kernels were 2 % slower.)
struct PoolMaxScore {  // largest score; what is not a number is left out where there are numbers
  static __device__ __forceinline__ uint32_t begin(uint32_t w) { return w; }
  static __device__ __forceinline__ uint32_t get(uint32_t w) { return w; }
  static __device__ __forceinline__ uint32_t join(uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }
};
struct PoolMaxWord {  // largest whole word (non-negative floats compare like their bits)
  static __device__ __forceinline__ uint32_t begin(uint32_t) { return 0u; }
  static __device__ __forceinline__ uint32_t get(uint32_t w) { return w; }
  static __device__ __forceinline__ uint32_t join(uint32_t a, uint32_t b) { return max(a, b); }
};
struct PoolMaxLow {  // largest low half
  static __device__ __forceinline__ uint32_t begin(uint32_t) { return 0u; }
  static __device__ __forceinline__ uint32_t get(uint32_t w) { return w & 0xFFFFu; }
  static __device__ __forceinline__ uint32_t join(uint32_t a, uint32_t b) { return max(a, b); }
};

// The pooling windows [c + e - h, c + e + h] of the four tokens c + e (c a
// multiple of 4) over stage[0 .. n) and its margins: three 16-byte reads up to
// h = 4, more groups beyond.  h = 3 (a pooling width of 7, the usual one) has code
// of its own, in which the part of the windows that all four share is taken once.
template <bool kThree>
struct PoolWindow {
  uint32x4 left, mid, right;
  const uint32_t* stage;
  int c, h, n;
  __device__ __forceinline__ PoolWindow(const uint32_t* stage_, int c_, int h_, int n_)
      : stage(stage_), c(c_), h(h_), n(n_) {
    mid = lds_words4(stage + c);
    if constexpr (kThree) {
      left = lds_words4(stage + c - 4);
      right = lds_words4(stage + c + 4);
    }
  }
  template <typename Op>
  __device__ __forceinline__ void reduce(uint32_t (&out)[4]) const {
    if constexpr (kThree) {
      const uint32_t core = Op::join(Op::join(Op::get(mid[0]), Op::get(mid[1])),
                                     Op::join(Op::get(mid[2]), Op::get(mid[3])));
      const uint32_t l2 = Op::get(left[3]), l1 = Op::join(Op::get(left[2]), l2),
                     l0 = Op::join(Op::get(left[1]), l1);
      const uint32_t r1 = Op::get(right[0]), r2 = Op::join(r1, Op::get(right[1])),
                     r3 = Op::join(r2, Op::get(right[2]));
      out[0] = Op::join(core, l0);
      out[1] = Op::join(core, Op::join(l1, r1));
      out[2] = Op::join(core, Op::join(l2, r2));
      out[3] = Op::join(core, r3);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = Op::get(mid[e]);
      if (h == 0) return;  // uniform, as all that follows
      if (h <= 4) {
        const uint32x4 w0 = lds_words4(stage + c - 4), w1 = lds_words4(stage + c + 4);
        uint32_t v[12];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = Op::get(w0[e]);
          v[4 + e] = out[e];
          v[8 + e] = Op::get(w1[e]);
        }
#pragma unroll
        for (int d = 1; d <= 4; ++d) {
          if (d > h) break;
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = Op::join(out[e], Op::join(v[4 + e - d], v[4 + e + d]));
        }
        return;
      }
      uint32_t shared = Op::begin(out[0]);  // (in all four windows: h > 4)
      const int reach = (h + 3) >> 2;  // groups to either side
      for (int g = -reach; g <= reach; ++g) {
        const int at = c + 4 * g;
        if (at < -kStageFront || at >= n) continue;  // (the margins cover one group to either side)
        const uint32x4 w = lds_words4(stage + at);
        if (4 * abs(g) + 3 <= h) {  // uniform: in all four windows
          shared = Op::join(shared, Op::join(Op::join(Op::get(w[0]), Op::get(w[1])),
                                             Op::join(Op::get(w[2]), Op::get(w[3]))));
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (abs(4 * g + k - e) <= h) out[e] = Op::join(out[e], Op::get(w[k]));
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = Op::join(out[e], shared);
    }
  }
};

// hist[b[e]] += 1 for four buckets (kNoBucket: none); neighbouring tokens share
// their pooled maximum more often than not, so equal neighbours go in one add
static constexpr uint32_t kNoBucket = 0xFFFFFFFFu;
__device__ __forceinline__ void hist_add4(int* hist, const uint32_t (&b)[4]) {
  int run = 1;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (e < 3 && b[e] == b[(e + 1) & 3]) {
      ++run;
    } else {
      if (b[e] != kNoBucket) atomicAdd(&hist[b[e]], run);
      run = 1;
    }
  }
}

// The bucket that holds the `rank`-th largest entry of a histogram -> sel[0],
// the rank inside it -> sel[1].  All threads call; ends with a barrier.
template <int WV>
__device__ __forceinline__ void bucket_of_rank(const int* hist, int rank, int* wsum, int* sel) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kScan = WV == 12 ? 512 : 64 * WV;  // threads that share the buckets
  constexpr int kOwn = kBuckets / kScan;           // thread t owns buckets [kOwn t, kOwn t + kOwn)
  static_assert(kScan <= 64 * WV && kOwn * kScan == kBuckets, "buckets per thread");
  int own[kOwn];
  int s = 0;
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    own[i] = tid < kScan ? hist[tid * kOwn + i] : 0;
    s += own[i];
  }
  const int v = wave_scan_add(s);
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < WV; ++w) {
    if (w < wave) base += wsum[w];
    total += wsum[w];
  }
  int above = total - (v + base);  // keys in buckets above this thread's
#pragma unroll
  for (int i = kOwn - 1; i >= 0; --i) {
    if (above < rank && above + own[i] >= rank) {
      sel[0] = tid * kOwn + i;
      sel[1] = rank - above;
    }
    above += own[i];
  }
  __syncthreads();
}

template <int WV>
struct alignas(16) SelectShared {
  int hist[kBuckets];
  uint32_t cand[kMaxCand];
  int wsum[WV];
  uint32_t wmin[WV], wmax[WV];
  int sel[2];
  int n_cand;
  int cnt[WV][2];  // keys above and keys not below the hinted range
};

// Selects the kept tokens of one (request, layer, head) and writes them, in
// ascending order, to `kept` (nullable, global memory) and, over the words of
// stage[] (which hold the keys until a barrier before that), as 16-bit indices for
// the copy that follows in the same workgroup.  stage[0 .. n_sel): the un-pooled
// scores as floats, written by this workgroup and made visible by a barrier;
// map: room for one bit per token.  hint_lo, hint_hi: keys that are known to
// enclose the threshold (0, ~0: nothing is known).  All threads of the workgroup
// call.
template <bool kThree, int WV>
__device__ __forceinline__ void select_unit_h(const BatchParams& p, const ReqDesc& rd, int lh,
                                              uint32_t* stage, uint32_t* map, int32_t* kept,
                                              SelectShared<WV>& sh, uint32_t hint_lo, uint32_t hint_hi) {
  int* hist = sh.hist;
  uint32_t* cand = sh.cand;
  int* sel = sh.sel;
  const int L = rd.seq_len;
  const int B = rd.budget;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool snap = rd.method == 1 /* FC_METHOD_SNAPKV */;
  const int n_sel = snap ? L - rd.window : L;  // tokens that compete
  const int k_sel = snap ? B - rd.window : B;  // how many of them are kept
  float* out = p.scores_out ? p.scores_out + rd.score_off + (size_t)lh * L : nullptr;
  uint16_t* kept16 = reinterpret_cast<uint16_t*>(stage);  // (budget <= length: half of the words)
  auto keep_token = [&](int t, int j) {
    kept16[t] = (uint16_t)j;
    if (kept) kept[t] = j;
  };
  const int seg = segment_tokens<WV>(n_sel);
  const int j0 = wave * seg;
  const int j1 = min(n_sel, j0 + seg);

  // ---- 1. final scores -> keys, min / max -------------------------------------
  // (a window that reaches over an end holds the token there: its value again changes no maximum)
  if (n_sel > 0) fill_stage_margins(stage, n_sel, stage[0], stage[n_sel - 1]);
  if (tid == 0) sh.n_cand = 0;
  for (int i = tid; i < kBuckets; i += 64 * WV) hist[i] = 0;
  __syncthreads();
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  int n_above = 0, n_reach = 0;  // keys above the hinted range, keys not below it
  SegmentRewrite keys;
  keys.run(stage, j0, j1, [&](int c) {
    const PoolWindow<kThree> pw(stage, c, rd.pool_kernel >> 1, n_sel);
    uint32_t v[4];
    if (snap) {
      pw.template reduce<PoolMaxScore>(v);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = pw.mid[e];
    }
    uint32x4 k4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t k = 0u;  // no token: below every key
      if (c + e < j1) {
        k = score_key(__uint_as_float(v[e]));
        kmin = min(kmin, k);
        kmax = max(kmax, k);
        n_above += k > hint_hi ? 1 : 0;
        n_reach += k >= hint_lo ? 1 : 0;
      }
      k4[e] = k;
    }
    return k4;
  });
  kmin = wave_min(kmin);
  kmax = wave_max(kmax);
  n_above = wave_sum(n_above);
  n_reach = wave_sum(n_reach);
  if (lane == 0) {
    sh.wmin[wave] = kmin;
    sh.wmax[wave] = kmax;
    sh.cnt[wave][0] = n_above;
    sh.cnt[wave][1] = n_reach;
  }
  __syncthreads();
  keys.finish(stage, j0, j1);
  if (out) {
    __syncthreads();
    for (int j = tid; j < n_sel; j += 64 * WV) {
      const uint32_t k = stage[j];
      out[j] = __uint_as_float((k & 0x80000000u) ? k & 0x7FFFFFFFu : ~k);
    }
    for (int j = n_sel + tid; j < L; j += 64 * WV) out[j] = INFINITY;
  }
  n_above = n_reach = 0;
#pragma unroll
  for (int w = 0; w < WV; ++w) {
    kmin = min(kmin, sh.wmin[w]);
    kmax = max(kmax, sh.wmax[w]);
    n_above += sh.cnt[w][0];
    n_reach += sh.cnt[w][1];
  }
  // the k_sel-th largest key lies in the hinted range: search only there
  const bool narrowed = n_above < k_sel && n_reach >= k_sel;  // uniform
  if (narrowed) {
    kmin = max(kmin, hint_lo);
    kmax = min(kmax, hint_hi);
  }

  int t0 = 0;  // where this wavefront's kept tokens begin in the list
  if (k_sel > 0) {  // uniform
    // ---- 2. threshold = k_sel-th largest key -------------------------------------
    // each sweep: this wavefront's keys, four per lane, 0 where there is no token
    auto sweep = [&](auto f) {
      for (int base = j0; base < j1; base += kChunk) {  // uniform over the wavefront
        const int c = base + 4 * lane;
        uint32x4 k4 = {0u, 0u, 0u, 0u};
        if (c < j1) k4 = lds_words4(stage + c);
        f(base, k4);
      }
    };
    // the keys in [lo, lo + width) into 2048 buckets (width 0: up to kmax)
    auto count_keys = [&](uint32_t lo, int shift, uint32_t width) {
      sweep([&](int, uint32x4 k4) {
        uint32_t b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t k = k4[e], d = k - lo;
          b[e] = k >= lo && k != 0u && (width == 0u ? k <= kmax : d < width) ? d >> shift : kNoBucket;
        }
        hist_add4(hist, b);
      });
    };
    // the keys of [lo, hi], in no particular order, to the candidate list
    auto list_candidates = [&](uint32_t lo, uint32_t hi) {
      sweep([&](int, uint32x4 k4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t k = k4[e];
          if (k >= lo && k <= hi && k != 0u) {
            const int pos = atomicAdd(&sh.n_cand, 1);
            if (pos < kMaxCand) cand[pos] = k;
          }
        }
      });
    };
    // A short list is ranked by comparing every candidate with every other one: one
    // barrier instead of the six of two more histograms.  Up to one candidate per
    // thread, at most kDirect (the reads are 16 bytes, the same for all lanes).  A
    // range of at most kDirectRange keys is listed without a histogram before: that one
    // costs less than ranking more (heads of 256 tokens, 64 of them, the whole call:
    // 41.8 us with 256, 36.5 with 128, 33.4 with 64).
    constexpr int kDirect = 256, kDirectRange = 64;
    int remaining = narrowed ? k_sel - n_above : k_sel;  // rank among the keys up to kmax
    uint32_t lo = kmin, hi = kmax;
    if (!(narrowed && n_reach - n_above <= kDirectRange)) {
      const uint32_t range = kmax - kmin;
      const int shift = range ? max(0, 32 - __clz(range) - kBucketBits) : 0;
      count_keys(lo, shift, 0u);
      __syncthreads();
      bucket_of_rank<WV>(hist, remaining, sh.wsum, sel);
      remaining = sel[1];
      lo = kmin + ((uint32_t)sel[0] << shift);
      hi = min(kmax, lo + ((1u << shift) - 1u));
    }
    if (lo != hi) {
      list_candidates(lo, hi);
      __syncthreads();
      const int nc = sh.n_cand;
      if (nc <= kDirect) {
        const uint32_t mine = tid < nc ? cand[tid] : 0u;
        int gt = 0, eq = 0;
        for (int j = 0; j < nc && 64 * wave < nc; j += 4) {  // (a wavefront without a candidate has nothing to rank)
          const uint32x4 c4 = lds_words4(cand + j);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            gt += j + e < nc && c4[e] > mine ? 1 : 0;
            eq += j + e < nc && c4[e] == mine ? 1 : 0;
          }
        }
        if (tid < nc && gt < remaining && gt + eq >= remaining) {  // (equal candidates write the same)
          sel[0] = (int)mine;
          sel[1] = remaining - gt;
        }
        __syncthreads();
        lo = hi = (uint32_t)sel[0];
        remaining = sel[1];
      } else {
        const bool listed = nc <= kMaxCand;  // else refine over all keys with a range check
        while (lo != hi) {
          const uint32_t width = hi - lo + 1u;  // (0 only if the range is all keys, which pass 1 rules out)
          const int shift = max(0, 32 - __clz(hi - lo) - kBucketBits);
          for (int i = tid; i < kBuckets; i += 64 * WV) hist[i] = 0;
          __syncthreads();
          if (listed) {
            for (int j = tid; j < nc; j += 64 * WV) {
              const uint32_t d = cand[j] - lo;
              if (cand[j] >= lo && d < width) atomicAdd(&hist[d >> shift], 1);
            }
          } else {
            count_keys(lo, shift, width);
          }
          __syncthreads();
          bucket_of_rank<WV>(hist, remaining, sh.wsum, sel);
          remaining = sel[1];
          lo += (uint32_t)sel[0] << shift;
          hi = min(hi, lo + ((1u << shift) - 1u));
        }
      }
    }
    const uint32_t thr = lo;
    const int need_eq = remaining;

    // ---- 3. which tokens are kept, one bit each -----------------------------------
    int n_gt = 0, n_eq = 0;
    sweep([&](int, uint32x4 k4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        n_gt += __popcll(__ballot(k4[e] > thr));
        n_eq += __popcll(__ballot(k4[e] == thr));
      }
    });
    // (not in sh.cnt: a narrowed range that is a single key comes here without a
    // barrier, and slower wavefronts may still be reading the counts of step 1.  The
    // histogram is read before a barrier, or was only cleared, before one as well)
    int* const counts = hist;
    if (lane == 0) {
      counts[2 * wave] = n_gt;
      counts[2 * wave + 1] = n_eq;
    }
    __syncthreads();
    int gt_before = 0, eq_before = 0;
    for (int w = 0; w < wave; ++w) {
      gt_before += counts[2 * w];
      eq_before += counts[2 * w + 1];
    }
    t0 = gt_before + min(eq_before, need_eq);
    int eq_run = eq_before;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    sweep([&](int base, uint32x4 k4) {
      // (lanes are in token order, each with its four tokens in order)
      uint64_t eq[4];
      int eq_rank = eq_run;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        eq[e] = __ballot(k4[e] == thr);
        eq_rank += __popcll(eq[e] & lt_mask);
        eq_run += __popcll(eq[e]);
      }
      uint32_t nibble = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool is_eq = k4[e] == thr;
        if (k4[e] > thr || (is_eq && eq_rank < need_eq)) nibble |= 1u << e;
        eq_rank += is_eq ? 1 : 0;
      }
      set_token_bits(map, base, nibble);
    });
  }
  __syncthreads();  // nobody reads a key any more: the kept list takes over the words

  // ---- 4. the list ------------------------------------------------------------------
  if (k_sel > 0) {
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    for (int base = j0; base < j1; base += kChunk) {
      const uint32_t nibble = token_bits(map, base);
      int at = t0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t kp = __ballot((nibble >> e) & 1u);
        at += __popcll(kp & lt_mask);
        t0 += __popcll(kp);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((nibble >> e) & 1u) keep_token(at++, base + 4 * lane + e);
    }
  }
  if (snap)
    for (int j = tid; j < rd.window; j += 64 * WV) keep_token(k_sel + j, n_sel + j);  // forced window
}

template <int WV>
__device__ __forceinline__ void select_unit(const BatchParams& p, const ReqDesc& rd, int lh,
                                            uint32_t* stage, uint32_t* map, int32_t* kept,
                                            SelectShared<WV>& sh, uint32_t hint_lo = 0u,
                                            uint32_t hint_hi = 0xFFFFFFFFu) {
  if (rd.pool_kernel == 7)  // uniform
    select_unit_h<true, WV>(p, rd, lh, stage, map, kept, sh, hint_lo, hint_hi);
  else
    select_unit_h<false, WV>(p, rd, lh, stage, map, kept, sh, hint_lo, hint_hi);
}

// ---------------------------------------------------------------------------
// SnapKV-style score with a pruned second pass
// ---------------------------------------------------------------------------
//
// The second pass over K only serves the selection, and the selection only
// needs exact column sums near its threshold.  The first pass can bound every
// column sum: it accumulates the soft-max numerators 2^(logit - ref_i) against a
// per-row reference ref_i that is known when the token is read (log2 of the
// row's sum over what the workgroup has read so far, renewed at fixed steps by
// all wavefronts together), so the exact weight of logit (i, j) is that
// numerator times rho_i = 2^(ref_i - lse_i) <= 1, a factor that is only known at
// the end but is the same for every token of an epoch.  With c_j the sum of a
// token's numerators e_ij over the window rows and s_j the root of the sum of
// their squares, for any number m
//     a_j = sum_i e_ij rho_i = m c_j + sum_i e_ij (rho_i - m),
// and because no e_ij is negative, with (x)+ = max(x, 0) and Cauchy-Schwarz,
//     a_j <= m c_j + s_j sqrt(sum_i ((rho_i - m)+)^2),
//     a_j >= m c_j - s_j sqrt(sum_i ((m - rho_i)+)^2).
// A few values of m around the mean of the rho_i are tried for
// each side (the least upper bound over all m is the exact maximum of a_j over
// all non-negative e_ij with these two sums), next to
// c_j min_i rho_i <= a_j <= c_j max_i rho_i.  Both numbers of a token
// share its word of the LDS score array until the pass ends (c_j in the leading
// 20 bits, s_j / c_j <= 1 in the other 12), so the bounds cost no memory traffic.
// After the pass two histograms of the pooled bounds give T_lo <= T <= T_hi for the
// selection's threshold T.  Only a token whose own interval reaches into
// [T_lo, T_hi] is re-scored exactly, row by row (256 bytes each); every other one
// keeps its upper bound.  The plain selection that follows then returns exactly the
// set it would return from exact scores: a window that holds an unread token with a
// lower bound above T_hi is above T either way, and in every other window the unread
// tokens are below T_lo, so its maximum is exact or, like the exact one, below T_lo.
//
// The scores themselves are not produced (callers that ask for them take the
// two-pass path).  A reference can be overtaken by more than the fp32 exponent
// range only by inputs far outside any attention layer; the numerators then
// overflow, the row's log-sum-exp is not finite, and the head falls back to
// the two-pass code.

static constexpr int kBoundCentres = 3;  // values of m tried per side

struct BoundEpoch {  // the factors rho_i of one epoch over the window rows
  float rmax, rmin;               // largest (widened), smallest (narrowed)
  float m_up[kBoundCentres];      // centres for the upper bound ...
  float p_up[kBoundCentres];      // ... and sqrt(sum ((rho_i - m)+)^2) for each (widened)
  float m_dn[kBoundCentres];      // the same for the lower bound, with (m - rho_i)+
  float p_dn[kBoundCentres];
};

// rows that hold anything, rounded up to what one lane each at a renewal covers
template <int NT>
static constexpr int kBoundRows = NT == 1 ? 16 : NT == 2 ? 32 : 64;
// The selection needs most LDS of what a workgroup does, and how many of them a CU takes
// hangs on it; so what comes before it stays below that: no tiles where the pass loads
// straight, and those of the rescoring lie over all this, which is done with by then.
// (With tiles for both in here, and three or four query tiles, 3 KB above it: 64 channels,
// 2048 heads of 5000-5500 tokens, window 64, 745 us with three workgroups per CU, 626 with
// four.)
template <int WV, int ROWS, bool kHalf>
struct BoundShared {
  float fin[64];                            // log2 of every row's soft-max denominator
  float pub[2][WV][ROWS];                   // the wavefronts' row sums at a renewal, absolute log2
  float ref[bound_max_epochs<WV>()][ROWS];  // the reference of every epoch
  union {
    KeyTiles<WV, kHalf> tiles;                // during the pass
    BoundEpoch stat[bound_max_epochs<WV>()];  // after it
  };
};

struct BoundKeep {  // what survives into the selection's LDS
  int bad;          // a row's log-sum-exp is not finite: fall back
};

// A token's two sums during the pass, in one word: the leading 20 bits of the
// sum c of its numerators (truncated: at most 2^-11 below c) and, in 12 bits, a
// number k with sqrt(s2) <= k / 4095 * c, s2 the sum of their squares (the ratio
// is at most 1; where the squares left the fp32 range, or c is too small for
// them to be trusted, k = 4095 says just that).
__device__ __forceinline__ uint32_t pack_sums(float c, float s2) {
  // (hardware square root and reciprocal, 1 ulp each: the two steps added to k are 5e-4 of c)
  const float r = __builtin_amdgcn_sqrtf(s2) * __builtin_amdgcn_rcpf(c);  // not a number <= 1 when c is 0 or either sum overflowed
  const uint32_t k = (c >= 1.0e-12f && r <= 1.f) ? min(4095u, (uint32_t)(r * 4095.f) + 2u) : 4095u;
  return (__float_as_uint(c) & 0xFFFFF000u) | k;
}

// A token's bounds share one 32-bit word of LDS: the upper bound rounded up to
// its leading 16 bits, the lower bound rounded down to its leading 16 bits
// (both are non-negative floats).  0.8 % of slack against bounds that are tens
// of per cent apart.
__device__ __forceinline__ uint32_t pack_bounds(float lo, float hi) {
  const uint32_t h = (__float_as_uint(hi) + 0xFFFFu) >> 16;
  const uint32_t l = __float_as_uint(lo) >> 16;
  return (h << 16) | l;
}
__device__ __forceinline__ float upper_of(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ float lower_of(uint32_t w) { return __uint_as_float(w << 16); }


// kHalf (128 channels, narrow workgroups): every other block of a wavefront is read in
// whole lines with the hint that it is not wanted again.  Of long heads in a full chip
// little of what this pass reads is still in the memory-side cache when rows are read
// again; that half leaves the cache to the other one, and streams faster.  Where heads
// are short enough to be found there whole it costs (plan_fused_launches has the line).
// (A wavefront's branch on the block's number instead, to keep the end of a head, gains
// no more and costs 2 % where nothing is gained.)
template <int D, int WV>
static constexpr bool kHasHalfReuse = D == 128 && WV == kNarrow;
// With three and more query tiles its LDS is 3 KB above what the selection needs (the tiles
// lie next to the rows' references): it pays up to the length where a CU still takes as
// many workgroups of it (kPlanHalfReuseWords).
template <int NT, bool kHalf>
static constexpr bool kTilesCost = kHalf && NT > 2;

// First pass with bounds.  On return stage[j] holds the packed bounds of the
// column sum of every prefix token j and bs.fin the rows' log-sum-exps.  All
// threads of the workgroup call; ends with a barrier.
template <int D, int NT, int WV, bool kHalf, int ROWS>
__device__ __forceinline__ void snapkv_bounds(const BatchParams& p, const ReqDesc& rd, int lh,
                                              const int32_t* old_ids, BoundShared<WV, ROWS, kHalf>& bs,
                                              BoundKeep& keep, float* stage,
                                              half8 (&qreg)[NT][D / 32]) {
  constexpr int KS = D / 32;
  const int L = rd.seq_len;
  const int W = rd.window;
  const int lane = lane_number<true>();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15;
  const int q4 = lane >> 4;
  const KeyBlocks<D, WV, kHalf> keys(p, lh, bs.tiles.piece);
  const float c = p.scale_log2e;
  const int nb = (L + 15) >> 4;
  const int n_prefix = L - W;
  const int n_unmasked = n_prefix >> 4;
  // (past the end the last block again, so that no step branches around its request: stream_tiles)
  auto load_even = [&](int b, half8 (&k)[KS]) { keys.template load<false>(old_ids[min(b, nb - 1)], k); };
  auto load_odd = [&](int b, half8 (&k)[KS]) { keys.template load<kHalf>(old_ids[min(b, nb - 1)], k); };

  // Lane (q4, c16) holds the logits of token c16 of a block for the rows
  // 16 nt + 4 q4 + r: sums over the rows are in-lane adds, and row sums stay in
  // registers until a renewal.
  const int seg = bound_seg<WV>(L);
  float z[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) z[nt][r] = 0.f;
  // One row (my_row) per lane at renewals: the row 16 nt + 4 q4 + r belongs to the lanes
  // with c16 = 4 nt + r (modulo kRows), which is where the reduction below leaves
  // its sum.
  constexpr int kRows = NT == 1 ? 4 : NT == 2 ? 8 : 16;
  // (made anew at each renewal: kept through the loop, addresses of it were spilled, and a
  // reload waits for all keys on their way)
  auto row_of_lane = [&] {
    const int l = made_here(lane), slot = l & (kRows - 1);
    return (slot >> 2) * 16 + (l >> 4) * 4 + (slot & 3);
  };
  float my_ref = 0.f, my_share = -INFINITY;  // its reference; log2 of this wavefront's sum so far
  // sums of z[][] over the 16 lanes of a DPP row: plain additions while there are
  // fewer values than lanes, then halving exchanges
  auto row_sums = [&]() -> float {
    float v[kRows];
#pragma unroll
    for (int i = 0; i < kRows; ++i) v[i] = i < 4 * NT ? z[(i / 4) % NT][i % 4] : 0.f;
    const bool b3 = c16 & 8, b2 = c16 & 4, b1 = c16 & 2, b0 = c16 & 1;
    if constexpr (kRows == 16) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[i] = (b3 ? v[i + 8] : v[i]) + from_lane<0x140>(b3 ? v[i] : v[i + 8]);  // row_mirror: bit 3 flips
    } else {
#pragma unroll
      for (int i = 0; i < kRows; ++i) v[i] += from_lane<0x140>(v[i]);
    }
    if constexpr (kRows >= 8) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[i] = (b2 ? v[i + 4] : v[i]) + from_lane<0x141>(b2 ? v[i] : v[i + 4]);  // row_half_mirror: bit 2
    } else {
#pragma unroll
      for (int i = 0; i < kRows; ++i) v[i] += from_lane<0x141>(v[i]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      v[i] = (b1 ? v[i + 2] : v[i]) + from_lane<0x4E>(b1 ? v[i] : v[i + 2]);  // quad_perm [2,3,0,1]
    return (b0 ? v[1] : v[0]) + from_lane<0xB1>(b0 ? v[0] : v[1]);           // quad_perm [1,0,3,2]
  };
  // this wavefront's row sums so far, absolute log2 -> pub[buf]; starts new ones
  auto publish = [&](int buf, int my_row) {
    const float zs = row_sums();
    // (a sum that is not a number stays one: see merged)
    const float l = zs == 0.f ? -INFINITY : my_ref + log2f(zs);
    const float mx = fmaxf(my_share, l);
    const float both = (my_share == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(my_share - mx)) +
                       (l == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(l - mx));
    my_share = both == 0.f ? -INFINITY : mx + log2f(both);
    bs.pub[buf][wave][my_row] = my_share;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) z[nt][r] = 0.f;
  };
  // log2 of the workgroup's row sum from the published shares
  auto merged = [&](int buf, int row) {
    float l[WV];
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < WV; ++w) {
      l[w] = bs.pub[buf][w][row];
      mx = fmaxf(mx, l[w]);
    }
    // Numerators that overflowed make a share infinite and the sum below not a
    // number; from there on that row's references, sums and log-sum-exp are none
    // either, which is how the head is found to need the two-pass code.
    float zz = 0.f;
#pragma unroll
    for (int w = 0; w < WV; ++w) zz += l[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(l[w] - mx);
    return zz == 0.f ? 0.f : mx + log2f(zz);  // 0: nothing visible yet, any finite reference will do
  };

  const int T = (nb + WV - 1) / WV;  // steps; every wavefront walks all of them
  int epoch = 0, buf = 0;
  // one block's numerators.  kMode 0: the first block, no reference yet; 1: a
  // block before the window; 2: one that reaches into it
  auto numerators = [&](auto mode, int b, const half8 (&kc)[KS]) {
    constexpr int kMode = decltype(mode)::value;
    const int tok = b * 16 + c16;
    float cs = 0.f, ss = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(qreg[nt][ks], kc[ks], acc, 0, 0, 0);
      floatx4* const at = reinterpret_cast<floatx4*>(&bs.pub[buf][wave][nt * 16 + q4 * 4]);
      floatx4 ref;
      if constexpr (kMode == 0) {
        // the logits of the block's first token (none of the block's is masked; they
        // all get the trivial bounds, whatever they accumulate here)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          ref[r] = nt * 16 + q4 * 4 + r < W ? from_lane<0x150>(acc[r] * c)  // row_newbcast:0
                                            : INFINITY;                    // (padded rows: every numerator 0)
        if (c16 == 0) *at = ref;
      } else {
        ref = *at;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float x = fmaf(acc[r], c, -ref[r]);
        if constexpr (kMode == 2)  // query i at position L - W + i
          if (tok > L - W + nt * 16 + q4 * 4 + r) x = -INFINITY;
        const float e = __builtin_amdgcn_exp2f(x);
        z[nt][r] += e;
        cs += e;
        ss = fmaf(e, e, ss);
      }
    }
    cs = quarter_sum(cs);
    ss = quarter_sum(ss);
    if (q4 == 0 && tok < n_prefix) reinterpret_cast<uint32_t*>(stage)[tok] = pack_sums(cs, ss);
  };
  // one step: kc holds this wavefront's block b, kn takes the next one
  auto step = [&](int t, half8 (&kc)[KS], auto load_next) {
    const int b = wave + WV * t;
    load_next(b + WV);
    requests_first();
    keys.arrange(kc);
    if (bound_renews_before(t, seg)) {  // uniform over the workgroup
      const int my_row = row_of_lane();
      if (t == 1) my_ref = bs.pub[buf][wave][my_row];
      publish(buf, my_row);
      __syncthreads();
      ++epoch;
      const float nr = merged(buf, my_row);
      if (wave == 0) bs.ref[epoch][my_row] = nr;
      my_ref = my_row < W ? nr : INFINITY;
      // to the lanes that use it, through the wavefront's own words of the other
      // buffer (its readers of the last renewal have passed a barrier since)
      buf ^= 1;
      bs.pub[buf][wave][my_row] = my_ref;
    }
    if (b < n_unmasked)  // uniform per wavefront
      numerators(std::integral_constant<int, 1>{}, b, kc);
    else  // (a block past the end is masked whole)
      numerators(std::integral_constant<int, 2>{}, b, kc);
  };
  half8 ka[KS], kb[KS];
  load_even(wave, ka);
  load_odd(wave + WV, kb);
  keys.arrange(ka);
  numerators(std::integral_constant<int, 0>{}, wave, ka);
  int t = 1;
  for (; t + 1 < T; t += 2) {
    step(t, kb, [&](int b) { load_even(b, ka); });
    step(t + 1, ka, [&](int b) { load_odd(b, kb); });
  }
  if (t < T) step(t, kb, [](int) {});
  publish(buf, row_of_lane());
  __syncthreads();
  if (threadIdx.x < 64) {
    const int row = threadIdx.x;
    float lse = INFINITY;  // padded rows contribute exp2(-inf) = 0
    if (row < W) {
      lse = merged(buf, row);
      if (!(fabsf(lse) < 3.0e38f)) keep.bad = 1;
    }
    bs.fin[row] = lse;
  }
  __syncthreads();
  // the factors of every epoch, rho_i = 2^(ref_i - lse_i) over the window rows
  // (one per lane): range, and for centres at the mean and half a standard
  // deviation to either side of it the one-sided deviations
  for (int e = 1 + wave; e <= epoch; e += WV) {
    const bool ok = lane < W;
    const float rho = ok ? __builtin_amdgcn_exp2f(bs.ref[e][lane % ROWS] - bs.fin[lane]) : 0.f;
    // (non-negative: their bits compare like the values; what is not a number makes
    // the head fall back, whatever comes out here)
    const float lo = __uint_as_float(wave_min(ok ? __float_as_uint(rho) : 0x7F800000u));
    const float hi = __uint_as_float(wave_max(__float_as_uint(rho)));
    const float mean = wave_sum(rho) / (float)W;
    const float var = wave_sum(ok ? (rho - mean) * (rho - mean) : 0.f);
    const float half_sd = 0.5f * sqrtf(var / (float)W);
    float m_up[kBoundCentres], m_dn[kBoundCentres], p_up[kBoundCentres], p_dn[kBoundCentres];
#pragma unroll
    for (int k = 0; k < kBoundCentres; ++k) {
      // (any centre gives a valid bound; none below zero, so that widening the sum widens the bound)
      m_up[k] = fmaxf(mean + (float)(k - 1) * half_sd, 0.f);
      m_dn[k] = fmaxf(mean - (float)(k - 1) * half_sd, 0.f);
      const float du = ok ? fmaxf(rho - m_up[k], 0.f) : 0.f;
      const float dd = ok ? fmaxf(m_dn[k] - rho, 0.f) : 0.f;
      p_up[k] = wave_sum(du * du);
      p_dn[k] = wave_sum(dd * dd);
    }
    if (lane == 0) {
      // (margins far above the rounding of the numerators, the sums and the factors)
      BoundEpoch& st = bs.stat[e];
      st.rmax = hi * 1.0002f;
      st.rmin = lo * 0.9998f;
#pragma unroll
      for (int k = 0; k < kBoundCentres; ++k) {
        st.m_up[k] = m_up[k];
        st.m_dn[k] = m_dn[k];
        st.p_up[k] = sqrtf(p_up[k]) * 1.001f + 1.0e-6f * hi;
        st.p_dn[k] = sqrtf(p_dn[k]) * 1.001f + 1.0e-6f * hi;
      }
    }
  }
  __syncthreads();
  // per token: the two sums -> bounds, packed in place
  {
    const float trivial = (float)W;  // every row contributes at most 1
    for (int j = threadIdx.x; j < n_prefix; j += 64 * WV) {
      const int e = bound_epoch_of_step((j >> 4) / WV, seg);
      const uint32_t w = reinterpret_cast<const uint32_t*>(stage)[j];
      const float c_lo = __uint_as_float(w & 0xFFFFF000u);
      float lo = 0.f, hi = trivial;
      if (e > 0 && c_lo < 3.0e38f) {  // (a sum that left the fp32 range says nothing)
        const BoundEpoch& st = bs.stat[e];
        const float c_hi = c_lo * 1.00049f + 1.0e-30f;  // what the truncation to 20 bits took, at most
        const float s_hi = (float)(w & 0xFFFu) * (1.f / 4095.f) * c_hi;
        float h = c_hi * st.rmax, l = c_lo * st.rmin;
#pragma unroll
        for (int k = 0; k < kBoundCentres; ++k) {
          h = fminf(h, (st.m_up[k] * c_hi + s_hi * st.p_up[k]) * 1.0002f);
          l = fmaxf(l, (st.m_dn[k] * c_lo - s_hi * st.p_dn[k]) * 0.9998f);
        }
        lo = fmaxf(l, 0.f);
        hi = fminf(h, trivial);
      }
      reinterpret_cast<uint32_t*>(stage)[j] = pack_bounds(lo, hi);
    }
  }
  __syncthreads();
}

// Exact column sums of the tokens named by need[] (one bit per prefix token),
// row by row -> stage[].  mrow: the rows' log-sum-exps as the second product
// leaves the rows in registers.  Rows of 256 bytes are fetched in whole lines (8192 heads of
// 700 tokens: 606 -> 593 us with two query tiles, 697 -> 681 with four, 563 -> 560 with one);
// rows of 128 bytes, one line anyhow, are not (2048 heads of 6500 tokens, four tiles: 969
// straight, 995 us).
template <int D>
static constexpr bool kRescoreLines = D == 128;
// The tokens that a wavefront re-scores, taken from kWords words of the map at a time.
template <int WV>
struct RescoreLists {
  static constexpr int kWords = WV == kNarrow ? 32 : 16;
  uint16_t token[WV][kWords * 32];
};
template <int D, int WV>
struct RescoreShared {
  KeyTiles<WV, kRescoreLines<D>> tiles;
  RescoreLists<WV> lists;
};
template <int D, int NT, int WV>
__device__ __forceinline__ void snapkv_rescore(const BatchParams& p, const ReqDesc& rd, int lh,
                                               const int32_t* old_ids, const uint32_t* need, float* stage,
                                               half8* tiles, RescoreLists<WV>& lists, half8 (&qreg)[NT][D / 32],
                                               const float (&mrow)[NT][4]) {
  constexpr int KS = D / 32;
  constexpr int kWords = RescoreLists<WV>::kWords;
  const int lane = lane_number<true>();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15;
  const int q4 = lane >> 4;
  const KeyBlocks<D, WV, kRescoreLines<D>> keys(p, lh, tiles);
  const float c = p.scale_log2e;
  const int n_words = (rd.seq_len - rd.window + 31) >> 5;
  uint16_t* const list = lists.token[wave];
  // A wavefront walks its words of the bit map, a lane each, lists the tokens they name in
  // LDS and takes those sixteen at a time (found one after the other by scalar code, with
  // their rows waited for as stream_tiles says, they took twice as long: 10.6 us of the 79
  // that a head of 640 tokens spent, four heads on each CU, now 5.4).
  for (int w0 = wave; w0 < n_words; w0 += WV * kWords) {  // uniform over the wavefront
    const int w = w0 + WV * lane;
    uint32_t bits = lane < kWords && w < n_words ? need[w] : 0u;
    const int own = __popc(bits), upto = wave_scan_add(own);
    const int n = __builtin_amdgcn_readlane(upto, 63);
    for (int at = upto - own; bits; bits &= bits - 1, ++at) list[at] = (uint16_t)(w * 32 + __ffs(bits) - 1);
    wave_lds_barrier();
    // (the last tile's lanes without a token read the last row again and drop the result)
    auto token = [&](int i) { return (int)list[min(16 * i + c16, n - 1)]; };
    stream_tiles<half8[KS]>(
        (n + 15) >> 4, [&](int i, half8(&k)[KS]) { keys.load_rows(token(i), old_ids, k); },
        [&](int i, half8(&kc)[KS]) {
          keys.arrange(kc);
          float colsum = 0.f;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
              acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(qreg[nt][ks], kc[ks], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) colsum += __builtin_amdgcn_exp2f(acc[r] * c - mrow[nt][r]);
          }
          colsum = quarter_sum(colsum);
          if (q4 == 0 && 16 * i + c16 < n) stage[token(i)] = colsum;
        });
    wave_lds_barrier();
  }
}

// Between the two: which prefix tokens need their exact column sum.  stage[]
// holds the packed bounds; need[] is set (one bit per token), stage[j] of every
// token becomes its upper bound.  Tokens are owned and pooled as in select_unit_h;
// the histograms' sweep reads three 16-byte words per four tokens.
//
// What is named is read again, so the rule decides how much of K that is.  A token is
// named if its own interval meets [T_lo, T_hi]: 9 % of the prefix rows of heads of 4096
// tokens, window 64, a fifth kept, and 30 % at 900 tokens, half kept (fp64 model on
// N(0,1) keys with four channels scaled by 8).  Naming whatever can carry the maximum of
// an undecided window, also where that maximum lies below T_lo, named 16 and 44 %, and
// took two sweeps over the windows more: 64 prompts of 1280-7040 tokens, 4 layers of 32
// heads, 3154 -> 3066 us; one of 640 tokens, 32 layers, 83.3 -> 79.3.  A second histogram
// after half of them are re-scored, and then the few that are still open, would name 5
// and 19 %, but the further sweep, its barriers and the second wait for rows cost more
// (3103 and 88 us).
//
// The selection's threshold is returned between two keys.
template <bool kThree, int WV>
__device__ __forceinline__ void bound_classify_h(const ReqDesc& rd, uint32_t* stage, uint32_t* need,
                                                 SelectShared<WV>& sh, uint32_t& key_lo, uint32_t& key_hi) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_sel = rd.seq_len - rd.window;
  const int k_sel = rd.budget - rd.window;
  const int h = rd.pool_kernel >> 1;
  const int seg = segment_tokens<WV>(n_sel);
  const int j0 = wave * seg;
  const int j1 = min(n_sel, j0 + seg);
  int* hist_lo = sh.hist;
  int* hist_hi = reinterpret_cast<int*>(sh.cand);
  static_assert(kMaxCand >= kBuckets, "the candidate list doubles as the second histogram");
  fill_stage_margins(stage, n_sel, 0u, 0u);
  uint32_t vmax = 0u;
  for (int c = j0 + 4 * lane; c < j1; c += kChunk) {
    const uint32x4 w = lds_words4(stage + c);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < j1) vmax = max(vmax, w[e] & 0xFFFF0000u);
  }
  vmax = wave_max(vmax);
  if (lane == 0) sh.wmax[wave] = vmax;
  auto zero_histograms = [&] {
    for (int i = tid; i < kBuckets; i += 64 * WV) hist_lo[i] = hist_hi[i] = 0;
  };
  zero_histograms();
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WV; ++w) vmax = max(vmax, sh.wmax[w]);
  const bool trivial = k_sel <= 0 || k_sel >= n_sel;  // uniform: window only, or everything is kept
  if (!trivial) {
    // thresholds: the buckets that hold the k_sel-th largest lower and the k_sel-th
    // largest upper bound (two histograms from one evaluation of the pooled bounds);
    // buckets of 2^shift bit patterns from kmin upwards, what lies below kmin counts in bucket 0
    auto find_buckets = [&](uint32_t kmin, int shift) {
      for (int c = j0 + 4 * lane; c < j1; c += kChunk) {
        const PoolWindow<kThree> pw(stage, c, h, n_sel);
        uint32_t hi[4], lo[4];
        pw.template reduce<PoolMaxWord>(hi);
        pw.template reduce<PoolMaxLow>(lo);
        // (no bound exceeds the largest upper bound; the clamp keeps the index in range whatever the bounds hold)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t kh = hi[e] & 0xFFFF0000u, kl = lo[e] << 16;
          hi[e] = kh > kmin ? min((kh - kmin) >> shift, (uint32_t)kBuckets - 1u) : 0u;
          lo[e] = kl > kmin ? min((kl - kmin) >> shift, (uint32_t)kBuckets - 1u) : 0u;
          if (c + e >= j1) hi[e] = lo[e] = kNoBucket;
        }
        hist_add4(hist_hi, hi);
        hist_add4(hist_lo, lo);
      }
      __syncthreads();
      bucket_of_rank<WV>(hist_lo, k_sel, sh.wsum, sh.sel);
      const int blo = sh.sel[0];
      __syncthreads();
      bucket_of_rank<WV>(hist_hi, k_sel, sh.wsum, sh.sel);
      const int bhi = sh.sel[0];
      return make_int2(blo, bhi);
    };
    // The bounds carry 16 significant bits, the whole range from 0 to the largest
    // upper bound only fits 2048 buckets that are up to 12 % of a value wide.  So
    // first with buckets of 1.6 % (2^17 bit patterns) over the 32 octaves below
    // the largest upper bound; should the k_sel-th largest lower bound lie below
    // all of that, once more over the whole range.
    const int coarse = vmax ? max(0, 32 - __clz(vmax) - kBucketBits) : 0;
    constexpr int kFine = 17;
    uint32_t kmin = 0u;
    int shift = coarse;
    if (coarse > kFine) {
      kmin = vmax - ((uint32_t)kBuckets << kFine) + 1u;
      shift = kFine;
    }
    int2 bkt = find_buckets(kmin, shift);
    if (kmin != 0u && bkt.x == 0) {  // uniform
      __syncthreads();               // (everyone has read the histograms before they are cleared)
      zero_histograms();
      __syncthreads();
      kmin = 0u;
      shift = coarse;
      bkt = find_buckets(kmin, shift);
    }
    // (bucket 0 also holds what lies below kmin)
    const uint32_t t_lo = bkt.x == 0 ? 0u : kmin + ((uint32_t)bkt.x << shift);  // <= the threshold
    const uint32_t t_hi = kmin + (((uint32_t)bkt.y + 1u) << shift) - 1u;         // >= the threshold
    key_lo = t_lo | 0x80000000u;  // (score_key of a non-negative value)
    key_hi = t_hi | 0x80000000u;
    // (own words only; the histograms' readers of a neighbour's have passed a barrier since)
    for (int base = j0; base < j1; base += kChunk) {  // uniform over the wavefront
      const int c = base + 4 * lane;
      uint32_t named = 0u;
      if (c < j1) {
        uint32x4 w = lds_words4(stage + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t hi = w[e] & 0xFFFF0000u, lo = w[e] << 16;
          if (c + e < j1 && hi >= t_lo && lo <= t_hi) named |= 1u << e;
          w[e] = hi;
        }
        set_lds_words4(stage + c, w);
      }
      set_token_bits(need, base, named);
    }
  } else {
    for (int base = j0; base < j1; base += kChunk) {
      const int c = base + 4 * lane;
      if (c < j1) {
        uint32x4 w = lds_words4(stage + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] &= 0xFFFF0000u;
        set_lds_words4(stage + c, w);
      }
      set_token_bits(need, base, 0u);
    }
  }
  __syncthreads();
}

template <int WV>
__device__ __forceinline__ void bound_classify(const ReqDesc& rd, uint32_t* stage, uint32_t* need,
                                               SelectShared<WV>& sh, uint32_t& key_lo, uint32_t& key_hi) {
  key_lo = 0u;
  key_hi = 0xFFFFFFFFu;
  if (rd.pool_kernel == 7)  // uniform
    bound_classify_h<true, WV>(rd, stage, need, sh, key_lo, key_hi);
  else
    bound_classify_h<false, WV>(rd, stage, need, sh, key_lo, key_hi);
}

// Streaming requests need no score: the first min(n_sink, budget) tokens and
// the most recent budget - sinks tokens are kept.
__device__ __forceinline__ int streaming_token(const ReqDesc& rd, int n_sink, int t) {
  return t < min(n_sink, rd.budget) ? t : rd.seq_len - rd.budget + t;
}

template <int WV>
__device__ __forceinline__ void streaming_unit(const BatchParams& p, const ReqDesc& rd, int lh,
                                               int32_t* kept) {
  const int L = rd.seq_len;
  const int B = rd.budget;
  if (kept)
    for (int t = threadIdx.x; t < B; t += 64 * WV) kept[t] = streaming_token(rd, p.n_sink, t);
  if (p.scores_out) {
    const int sinks = min(p.n_sink, B);
    float* out = p.scores_out + rd.score_off + (size_t)lh * L;
    for (int j = threadIdx.x; j < L; j += 64 * WV)
      out[j] = (j < sinks || j >= L - (B - sinks)) ? INFINITY : 0.f;
  }
}

// ---------------------------------------------------------------------------
// gather / compact
// ---------------------------------------------------------------------------
//
// One workgroup per (request, layer, head); a wavefront fills one new block
// (16 output slots) at a time for K and V.  D/8 lanes move one row with
// 128-bit accesses, so a wavefront instruction moves 64/(D/8) rows; the
// destination chunk is contiguous.
//
// Bound by HBM when the chip is full and by the latency of one block's chain
// (kept index, block id, row) when it is not; the rows of a wavefront's next
// block are therefore requested before those of this one are stored.  (Where the
// ids of the new blocks are vector loads, as in the fused kernels of several requests,
// the wait for such an id is one for the rows just asked for as well; kept in registers
// instead, they took the copy to fewer wavefronts a SIMD, and 24 requests of 1000-3000
// tokens 726-821 -> 735-822 us at 128 channels, 344-411 -> 349-413 at 64.)

template <int D, int WV>
struct RowCopy {
  static constexpr int LPR = D / 8;
  static constexpr int RPI = 64 / LPR;
  static constexpr int NI = 16 / RPI;
  typedef half8 Rows[2 * NI];  // of one block: keys, then values
  const BatchParams& p;
  const int nb0, n_kept, wave, row_in_instr;
  size_t v_off, blk_stride;  // K chunk -> V chunk of a block; block -> block
  _Float16* base;

  // of the new blocks from nb0 on
  __device__ __forceinline__ RowCopy(const BatchParams& p_, const ReqDesc& rd, int lh, int nb0_)
      : p(p_), nb0(nb0_), n_kept(rd.budget), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        row_in_instr((threadIdx.x & 63) / LPR) {
    const int layer = lh / p.n_heads, head = lh - layer * p.n_heads;
    const size_t chunk = (size_t)16 * D;  // one (block, kv, head)
    v_off = (size_t)p.n_heads * chunk;
    blk_stride = 2 * v_off;
    base = p.kv + (size_t)layer * p.n_blocks * blk_stride + (size_t)head * chunk + (threadIdx.x % LPR) * 8;
  }
  __device__ __forceinline__ int block(int i) const { return nb0 + wave + WV * i; }  // the wavefront's i-th
  // source(row of the block, 0..15) -> {block id, slot}.  kInOrder: where the second row lies is
  // looked up when the first is asked for, and so on, which takes fewer registers (all at once,
  // kernels of 128 channels and one query tile lost a wavefront a SIMD, or spilled).
  template <bool kInOrder, typename Source>
  __device__ __forceinline__ void load(Rows& kv, Source source) const {
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int2 from = source(k * RPI + row_in_instr);
      const _Float16* src = base + (size_t)clamp_block(from.x, p.n_blocks) * blk_stride + (size_t)from.y * D;
      kv[k] = load_half8_nt(src);
      kv[NI + k] = load_half8_nt(src + v_off);
      if constexpr (kInOrder) requests_first();
    }
  }
  // (slots past the budget are not written)
  __device__ __forceinline__ void store(int nbk, int id, const Rows& kv) const {
    _Float16* dst = base + (size_t)clamp_block(id, p.n_blocks) * blk_stride;
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int row = k * RPI + row_in_instr;
      if (nbk * 16 + row < n_kept) {
        store_half8_nt(dst + (size_t)row * D, kv[k]);
        store_half8_nt(dst + (size_t)row * D + v_off, kv[NI + k]);
      }
    }
  }
};

// block_at(i) and new_at(i): the request's i-th old and new block; kept_at(t): the token that
// goes to slot t.  kStreaming: nothing was scored, all workgroups do nothing but copy, and more
// requests in flight only make the chip change between reading and writing more often.  Wide
// workgroups ask for their rows in order, and as their ids may be in either of two places
// (gather_fused), each row waits for the one before; all at once / in order, half of the tokens
// kept, 128 channels: 256 heads of 900-1000 tokens 29.0 / 26.9 us, 512 of 3000-6000 252 / 248,
// of 9000-16000, a third kept, 533 / 520; 64 channels: 256 of 2000-4000 35.4 / 33.8, 512 of
// 9000-16000 254 / 251.  In place, and narrow ones (see launch_fused), all at once (so is what was
// scored at 64 channels, in place: key norms, 2048 heads of 900-3000 194 / 197): 256 heads of
// 2000-4000 in place 63.5 / 66.5, 3840 of 1400-4300, 64 channels, 328 / 354.
template <int D, int WV, bool kStreaming, typename BlockAt, typename NewAt, typename KeptAt>
__device__ __forceinline__ void gather_unit(const BatchParams& p, const ReqDesc& rd, int lh, BlockAt block_at,
                                            NewAt new_at, KeptAt kept_at) {
  const int nb = rd.n_new;
  const RowCopy<D, WV> c(p, rd, lh, 0);
  typedef typename RowCopy<D, WV>::Rows Rows;
  auto source = [&](int nbk, int row) {
    // (slots past the budget load the last kept row again and drop it)
    const int idx = min(max(kept_at(min(nbk * 16 + row, rd.budget - 1)), 0), rd.seq_len - 1);
    return int2{block_at(idx >> 4), idx & 15};
  };
  if (p.in_place) {
    Rows kv;
    // Output t overwrites slot t while kept[t] >= t: a chunk of WV*16
    // outputs only reads slots at or after its own start, so reading the whole
    // chunk, a barrier, then writing it never destroys a row that is still
    // needed (later chunks read strictly later slots).
    for (int c0 = 0; c0 < nb; c0 += WV) {
      const int nbk = c0 + c.wave;
      if (nbk < nb) c.template load<!kStreaming && D == 128>(kv, [&](int row) { return source(nbk, row); });
      __syncthreads();  // uniform: c0 and in_place are the same for all threads
      if (nbk < nb) c.store(nbk, block_at(nbk), kv);  // (the request's own first blocks)
    }
    return;
  }
  if constexpr (kStreaming && WV != kNarrow) {
    Rows kc, kn;
    int nbk = c.wave;
    if (nbk < nb) c.template load<true>(kc, [&](int row) { return source(nbk, row); });
    for (; nbk < nb; nbk += WV) {
      if (nbk + WV < nb) c.template load<true>(kn, [&](int row) { return source(nbk + WV, row); });
      c.store(nbk, new_at(nbk), kc);
#pragma unroll
      for (int k = 0; k < 2 * c.NI; ++k) kc[k] = kn[k];
    }
  } else {
    stream_tiles<Rows>(
        own_tiles(nb, c.wave, WV),
        [&](int i, Rows& kv) { c.template load<!kStreaming>(kv, [&](int row) { return source(c.block(i), row); }); },
        [&](int i, const Rows& kv) { c.store(c.block(i), new_at(c.block(i)), kv); });
  }
}

// (of requests without plan_alloc none is)
template <bool kOnly>
__device__ __forceinline__ bool is_streaming(const ReqDesc& rd) {
  return !kOnly && rd.method == 3 /* FC_METHOD_STREAMING */;
}

// The copy at the end of a fused kernel: the kept list is where the selection
// left it in LDS, streaming units compute theirs; ids_in_lds: sm_ids holds the
// block ids (streaming units may have more blocks than fit).
template <int D, int WV, bool kOnly>
__device__ __forceinline__ void gather_fused(const BatchParams& p, const ReqDesc& rd, int lh,
                                             const uint32_t* words, const int32_t* sm_ids, bool ids_in_lds,
                                             const int32_t* sm_new) {
  const uint16_t* kept16 = reinterpret_cast<const uint16_t*>(words);
  auto new_at = [&](int i) {
    if constexpr (kOnly) return sm_new[i];
    else return p.new_ids[rd.new_off + i];
  };
  if (is_streaming<kOnly>(rd))  // uniform
    gather_unit<D, WV, true>(
        p, rd, lh, [&](int i) { return ids_in_lds ? sm_ids[i] : p.old_ids[rd.old_off + i]; }, new_at,
        [&](int t) { return streaming_token(rd, p.n_sink, t); });
  else  // (what is scored has its ids in LDS: one from either place comes by a load that waits for all others)
    gather_unit<D, WV, false>(
        p, rd, lh, [&](int i) { return sm_ids[i]; }, new_at, [&](int t) { return (int)kept16[t]; });
}

// ---------------------------------------------------------------------------
// fused per-unit kernel: score -> select -> gather in one workgroup
// ---------------------------------------------------------------------------
//
// For heads whose scores fit the workgroup's LDS share the three steps run
// back to back in the workgroup that owns the (request, layer, head): the
// column sums (or key norms) go straight into LDS, the selection works on
// them in place and the copy follows.  The scores never travel through HBM,
// the stage is one launch per workgroup shape, and the LDS/ALU-bound selection of
// one workgroup overlaps the HBM-bound streaming of the others on the same CU.
// One launch serves all methods (the unit's descriptor says which); NT =
// ceil(window / 16), 0 when the launch holds no SnapKV unit, kMixedTiles when its
// units differ.

// f(the number of query tiles): NT itself, or (kMixedTiles: a launch whose SnapKV
// units have windows of different classes) what the unit's window needs.
static constexpr int kMixedTiles = 5;
template <int NT, typename F>
__device__ __forceinline__ void for_query_tiles(int window, F f) {
  if constexpr (NT == kMixedTiles) {
    switch ((window + 15) >> 4) {  // uniform
      case 1: f(std::integral_constant<int, 1>{}); break;
      case 2: f(std::integral_constant<int, 2>{}); break;
      case 3: f(std::integral_constant<int, 3>{}); break;
      default: f(std::integral_constant<int, 4>{}); break;
    }
  } else if constexpr (NT > 0) {
    f(std::integral_constant<int, NT>{});
  }
}

// kOnly: a call of one request whose only launch this is, without plan_alloc and without a
// reclaim launch.  Its workgroups read the table and the stack themselves, and the last one
// that says so (behind a barrier after which nothing of either is left to read; the count
// only orders those reads before the writes, no data passes through it) writes them anew
// when its own copy is under way.  A launch is 2.5 to 3 us of the host's time, and
// plan_alloc, which the main kernel waited for, about 2 of the GPU's (plan_one_launch has
// what that gives and where it stops).  Counted when the ids have been read instead, so
// that not the last one writes, the counts of all workgroups come at once and stand before
// their keys: one prompt of 640 tokens, 1024 heads, 66.4 -> 73.7 us.  Kernels of their own:
// as a branch in those of all calls it cost these up to 3 % (registers).
template <bool kOnly>
__device__ __forceinline__ ReqDesc fused_request(const BatchParams& p, int slot) {
  if constexpr (kOnly) {
    ReqDesc rd = {};
    rd.seq_len = p.only.seq_len;
    rd.budget = p.only.budget;
    rd.method = p.only.method;
    rd.table_row = p.only.table_row;
    rd.n_old = p.only.n_old;
    rd.n_new = p.only.n_new;
    rd.q_off = p.only.q_off;
    rd.window = p.only.window;
    rd.pool_kernel = p.only.pool_kernel;
    return rd;
  } else {
    return p.descs[p.order_fused[slot]];
  }
}
// The request's block ids to LDS; false: they stay where plan_alloc left them.
template <int WV, bool kOnly>
__device__ __forceinline__ bool stage_block_ids(const BatchParams& p, const ReqDesc& rd, int lh, int32_t* sm_ids,
                                                int32_t* sm_new) {
  if constexpr (kOnly) {
    const int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
    if (!p.in_place)
      for (int i = threadIdx.x; i < rd.n_new; i += 64 * WV) sm_new[i] = p.stack[p.top_before - 1 - i];
    for (int i = threadIdx.x; i < rd.n_old; i += 64 * WV) sm_ids[i] = clamp_block(row[i], p.n_blocks);
    return true;  // (kOnlyMaxIds: there is room)
  } else {
    if (p.main_reclaims && lh == 0) reclaim_request(p, rd);
    const bool ids_in_lds = rd.n_old <= p.ids_room;  // streaming units may be longer
    if (ids_in_lds)
      for (int i = threadIdx.x; i < rd.n_old; i += 64 * WV)
        sm_ids[i] = clamp_block(p.old_ids[rd.old_off + i], p.n_blocks);
    return ids_in_lds;
  }
}
// How many workgroups came here before (the first wavefront's).
__device__ __forceinline__ int arrive(const BatchParams& p) {
  int before = -1;
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(p.arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = __builtin_amdgcn_readfirstlane(before);
  }
  return before;
}
// (one wavefront; ids: room for all of them, nobody else's any more)
__device__ __forceinline__ void reclaim_only(const BatchParams& p, const ReqDesc& rd, int32_t* ids) {
  const int lane = threadIdx.x;
  const int32_t* row = p.block_tables + (size_t)rd.table_row * p.max_blocks;
  for (int i = lane; i < rd.n_old; i += 64) ids[i] = row[i];
  if (!p.in_place)
    for (int i = lane; i < rd.n_new; i += 64) ids[rd.n_old + i] = p.stack[p.top_before - 1 - i];
  wave_lds_barrier();
  reclaim_request(p, rd, ids, ids + rd.n_old, lane, 64);
  if (lane == 0) __hip_atomic_store(p.arrivals, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wavefronts per SIMD that the registers must allow (1: as many as they come to), where that
// takes no vector spills and pays.  16 prompts of 200-480 tokens, 4 layers of 32 heads, with
// scores, free / bounded: 128 channels, window 48 (3 and 4 wavefronts) 80.8 / 75.7 us; 64
// channels, window 16 (7, by the scalar registers, and 8) 50.4 / 43.1; wide ones at 64 channels,
// of which a CU takes two only if all eight fit, 512 heads of 900-1000 tokens 47.0 / 39.2.
// Two and four tiles would spill: 73.8 / 94.3 at 128 channels, window 32, and 52.7 / 68.7 at 64,
// window 64.  Without SnapKV units key norms gain (39.0 / 33.6), but streaming, which HBM bounds,
// loses (755 / 769).
__host__ __device__ constexpr int scored_occupancy(int d, int nt, int wv) {
  return d == 64 && (nt == 1 || (nt == 0 && wv != kNarrow)) ? 8
         : wv != kNarrow                                    ? wv / 4
         : nt == 3                                          ? (d == 64 ? 5 : 4)
         : nt == 1                                          ? 5
                                                            : 1;
}
template <int D, int NT, int WV, bool kOnly>
__device__ __forceinline__ void fused_unit(const BatchParams& p) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ union {
    ScoreShared<WV> score;
    SelectShared<WV> select;
    int32_t ids[kOnlyMaxIds];
  } sh;
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = fused_request<kOnly>(p, slot);
  uint32_t* words = lds + kStageFront;
  float* stage = reinterpret_cast<float*>(words);
  uint32_t* map = lds + stage_words(rd.seq_len);  // one bit per token
  // the request's block ids, read once per workgroup (every later use is an LDS read)
  int32_t* sm_ids = reinterpret_cast<int32_t*>(lds + p.ids_at);
  int32_t* kept = p.kept_out ? p.kept_out + rd.kept_off + (size_t)lh * rd.budget : nullptr;
  int32_t* sm_new = reinterpret_cast<int32_t*>(lds + p.new_ids_at);
  const bool ids_in_lds = stage_block_ids<WV, kOnly>(p, rd, lh, sm_ids, sm_new);
  __syncthreads();
  if (is_streaming<kOnly>(rd)) {  // uniform per workgroup
    streaming_unit<WV>(p, rd, lh, kept);
  } else {
    bool snap = false;
    if constexpr (NT > 0) snap = rd.method == 1 /* FC_METHOD_SNAPKV */;
    if (snap) {
      for_query_tiles<NT>(rd.window, [&](auto nt) {
        snapkv_unit<D, decltype(nt)::value, WV, true>(p, rd, lh, sm_ids, sh.score,
                                                      [&](int j, float v) { stage[j] = v; });
      });
    } else {
      knorm_unit<D, WV>(p, rd, lh, sm_ids, 0, rd.n_old, [&](int j, float v) { stage[j] = v; });
    }
    __syncthreads();
    select_unit<WV>(p, rd, lh, words, map, kept, sh.select);
  }
  __syncthreads();  // the kept list is complete
  if constexpr (kOnly) {
    const int arrived = arrive(p);
    gather_fused<D, WV, true>(p, rd, lh, words, sm_ids, true, sm_new);
    if (arrived == (int)gridDim.x - 1) reclaim_only(p, rd, sh.ids);
  } else {
    gather_fused<D, WV, false>(p, rd, lh, words, sm_ids, ids_in_lds, sm_new);
  }
}
template <int D, int NT, int WV>
__global__ __launch_bounds__(64 * WV, scored_occupancy(D, NT, WV)) void fused_unit_kernel(BatchParams p) {
  fused_unit<D, NT, WV, false>(p);
}
template <int D, int WV>  // (of a scored request, key norms: the others are pruned)
__global__ __launch_bounds__(64 * WV, scored_occupancy(D, 0, WV)) void fused_unit_only_kernel(BatchParams p) {
  fused_unit<D, 0, WV, true>(p);
}

// Wavefronts per SIMD that the registers must allow: what the kernel needs without
// spilling in its loops.  (At 128 channels the forms with four and mixed query tiles spill
// 3 to 9 vector registers, at 64 the narrow one of mixed tiles 2, outside of the streaming loops.)  The wide one of one
// tile at 64 channels must leave room for a second workgroup: 512 heads of 900-1000 tokens
// 46.0 -> 39.8 us, of 4900-5100 141.9 -> 129.8.
__host__ __device__ constexpr int bounded_occupancy(int d, int nt, int wv) {
  return wv != kNarrow ? (d == 64 && nt == 1 ? 8 : wv / 4) : d == 64 ? (nt <= 2 ? 5 : 4) : nt == 1 ? 5 : nt == 2 ? 4 : 3;
}

// The fused kernel with the pruned second pass for its SnapKV units (see
// snapkv_bounds); key-norm and streaming units that ride in the launch run as in
// fused_unit_kernel.  Dynamic LDS: the scores, then one bit per token, then the
// block ids.
template <int D, int NT, int WV, bool kHalf, bool kOnly>
__device__ __forceinline__ void fused_bounded(const BatchParams& p) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ union {
    ScoreShared<WV> score;
    SelectShared<WV> select;
    BoundShared<WV, kBoundRows<NT>, kHalf> bound;
    RescoreShared<D, WV> rescore;  // (the bounds and the classification are done with theirs)
    int32_t ids[kOnlyMaxIds];
  } sh;
  static_assert(WV != kNarrow || kTilesCost<NT, kHalf> || sizeof(sh) <= sizeof(SelectShared<WV>),
                "the selection sets how many workgroups a CU takes");
  __shared__ BoundKeep keep;
  const int n_lh = p.n_layers * p.n_heads;
  const int slot = blockIdx.x / n_lh;
  const int lh = blockIdx.x - slot * n_lh;
  const ReqDesc rd = fused_request<kOnly>(p, slot);
  uint32_t* words = lds + kStageFront;  // per token: its bounds, then its score
  float* stage = reinterpret_cast<float*>(words);
  uint32_t* map = lds + stage_words(rd.seq_len);  // one bit per token
  int32_t* sm_ids = reinterpret_cast<int32_t*>(lds + p.ids_at);
  int32_t* kept = p.kept_out ? p.kept_out + rd.kept_off + (size_t)lh * rd.budget : nullptr;
  int32_t* sm_new = reinterpret_cast<int32_t*>(lds + p.new_ids_at);
  const bool ids_in_lds = stage_block_ids<WV, kOnly>(p, rd, lh, sm_ids, sm_new);
  if (threadIdx.x == 0) keep.bad = 0;
  __syncthreads();
  if (is_streaming<kOnly>(rd)) {  // uniform per workgroup
    streaming_unit<WV>(p, rd, lh, kept);
  } else {
    uint32_t key_lo = 0u, key_hi = 0xFFFFFFFFu;  // what is known of the selection's threshold
    if (rd.method == 1 /* FC_METHOD_SNAPKV */) {
      for_query_tiles<NT>(rd.window, [&](auto nt) {
        constexpr int N = decltype(nt)::value;
        constexpr int KS = D / 32;
        const int q4 = (threadIdx.x & 63) >> 4;
        half8 qreg[N][KS];
        load_window_queries<D, N>(p, rd, lh, qreg);
        const bool prune = rd.seq_len >= max(p.prune_from.tiles[N - 1], kBoundMinLen<WV>);  // uniform
        if (prune) snapkv_bounds<D, N, WV, kHalf>(p, rd, lh, sm_ids, sh.bound, keep, stage, qreg);
        if (!prune || keep.bad) {  // bad: not representable against a running reference
          snapkv_unit_q<D, N, WV, true>(p, rd, lh, sm_ids, sh.score, qreg, [&](int j, float v) { stage[j] = v; });
        } else {
          float mrow[N][4];
#pragma unroll
          for (int t = 0; t < N; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) mrow[t][r] = sh.bound.fin[t * 16 + q4 * 4 + r];
          __syncthreads();  // the log-sum-exps are in registers: the selection's LDS may take over
          bound_classify<WV>(rd, words, map, sh.select, key_lo, key_hi);
          snapkv_rescore<D, N, WV>(p, rd, lh, sm_ids, map, stage, sh.rescore.tiles.piece, sh.rescore.lists, qreg, mrow);
        }
      });
    } else {
      knorm_unit<D, WV>(p, rd, lh, sm_ids, 0, rd.n_old, [&](int j, float v) { stage[j] = v; });
    }
    __syncthreads();
    select_unit<WV>(p, rd, lh, words, map, kept, sh.select, key_lo, key_hi);
  }
  __syncthreads();  // the kept list is complete
  if constexpr (kOnly) {
    const int arrived = arrive(p);
    gather_fused<D, WV, true>(p, rd, lh, words, sm_ids, true, sm_new);
    if (arrived == (int)gridDim.x - 1) reclaim_only(p, rd, sh.ids);
  } else {
    gather_fused<D, WV, false>(p, rd, lh, words, sm_ids, ids_in_lds, sm_new);
  }
}
template <int D, int NT, int WV, bool kHalf>
__global__ __launch_bounds__(64 * WV, bounded_occupancy(D, NT, WV)) void fused_bounded_kernel(BatchParams p) {
  fused_bounded<D, NT, WV, kHalf, false>(p);
}
template <int D, int NT, int WV>
__global__ __launch_bounds__(64 * WV, bounded_occupancy(D, NT, WV)) void fused_bounded_only_kernel(BatchParams p) {
  fused_bounded<D, NT, WV, false, true>(p);
}

// what a wide workgroup may ask for next to its static LDS
static constexpr int kLdsPerCu = 160 * 1024;

// Narrow workgroups of the pruned kernel that fit the LDS of a CU (which is given out in
// pieces of 1280 bytes) next to `words` each.
template <int NT, bool kHalf>
static constexpr int narrow_per_cu(int words) {
  constexpr int bound = (int)sizeof(BoundShared<kNarrow, kBoundRows<NT>, kHalf>), rest = (int)sizeof(SelectShared<kNarrow>);
  return kLdsPerCu / (((bound > rest ? bound : rest) + 16 + 4 * words + 1279) / 1280 * 1280);
}
static constexpr int kMostNarrowWords = fused_lds(kFusedMaxLen, kFusedMaxLen / 16, false).words;
static_assert(narrow_per_cu<2, true>(kMostNarrowWords) == narrow_per_cu<2, false>(kMostNarrowWords) &&
                  narrow_per_cu<4, true>(kPlanHalfReuseWords) == narrow_per_cu<4, false>(kMostNarrowWords) &&
                  narrow_per_cu<4, true>(kPlanHalfReuseWords + 4) < narrow_per_cu<4, false>(kMostNarrowWords),
              "plan_fused_launches");

// One fused launch of workgroups of narrow or wide shape.
template <int D, int NT, bool kWideShape>
static void launch_fused_one(const BatchParams& p, size_t lds, hipStream_t s) {
  constexpr int WV = kWideShape ? kWide<D, NT> : kNarrow;
  const unsigned grid = (unsigned)p.n_fused * p.n_layers * p.n_heads;
  if (p.arrivals) {
    if constexpr (NT == 0)
      fused_unit_only_kernel<D, WV><<<grid, 64 * WV, lds, s>>>(p);
    else if constexpr (NT < kMixedTiles)
      fused_bounded_only_kernel<D, NT, WV><<<grid, 64 * WV, lds, s>>>(p);
    return;
  }
  if constexpr (NT > 0) {
    if (p.bounded) {
      if constexpr (kHasHalfReuse<D, WV>) {
        if (p.half_reuse) {
          fused_bounded_kernel<D, NT, WV, true><<<grid, 64 * WV, lds, s>>>(p);
          return;
        }
      }
      fused_bounded_kernel<D, NT, WV, false><<<grid, 64 * WV, lds, s>>>(p);
      return;
    }
  }
  fused_unit_kernel<D, NT, WV><<<grid, 64 * WV, lds, s>>>(p);
}

template <int D, bool kWideShape>
static hipError_t launch_fused_d(const BatchParams& p, int query_tiles, size_t lds, hipStream_t s) {
  switch (query_tiles) {
    case 0: launch_fused_one<D, 0, kWideShape>(p, lds, s); break;
    case 1: launch_fused_one<D, 1, kWideShape>(p, lds, s); break;
    case 2: launch_fused_one<D, 2, kWideShape>(p, lds, s); break;
    case 3: launch_fused_one<D, 3, kWideShape>(p, lds, s); break;
    case 4: launch_fused_one<D, 4, kWideShape>(p, lds, s); break;
    case kMixedTiles: launch_fused_one<D, kMixedTiles, kWideShape>(p, lds, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int D, int NT>
static hipError_t wide_setup_one() {
  constexpr int WV = kWide<D, NT>;
  constexpr int most = fused_lds(kFusedWideMaxLen, kFusedWideMaxLen / 16, true).words * 4;
  static_assert(most + (int)sizeof(BoundShared<WV, kBoundRows<NT>, false>) + 64 <= kLdsPerCu, "LDS of the longest head");
  static_assert(most + (int)sizeof(SelectShared<WV>) + 64 <= kLdsPerCu, "LDS of the longest head");
  static_assert(most + (int)sizeof(ScoreShared<WV>) + 64 <= kLdsPerCu, "LDS of the longest head");
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_unit_kernel<D, NT, WV>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, most);
  if constexpr (NT > 0)
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_bounded_kernel<D, NT, WV, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, most);
  // (the kernels without plan_alloc stay below the 64 KB that need no setting: kOnlyMaxIds)
  static_assert(4 * (fused_lds(kOnlyMaxIds * kPlanBlockSize, kOnlyMaxIds, true).words + kOnlyMaxIds) +
                        (int)sizeof(BoundShared<WV, kBoundRows<NT>, false>) + 64 <= 64 * 1024 &&
                    4 * (fused_lds(kOnlyMaxIds * kPlanBlockSize, kOnlyMaxIds, true).words + kOnlyMaxIds) +
                        (int)sizeof(SelectShared<WV>) + 64 <= 64 * 1024, "LDS of a request without plan_alloc");
  return e;
}

template <int D>
static hipError_t wide_setup_d() {
  hipError_t e = wide_setup_one<D, 0>();
  if (e == hipSuccess) e = wide_setup_one<D, 1>();
  if (e == hipSuccess) e = wide_setup_one<D, 2>();
  if (e == hipSuccess) e = wide_setup_one<D, 3>();
  if (e == hipSuccess) e = wide_setup_one<D, 4>();
  if (e == hipSuccess) e = wide_setup_one<D, kMixedTiles>();
  return e;
}

}  // namespace fc
