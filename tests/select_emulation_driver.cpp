// The selection and the classification of csrc/fc_unit.h on the CPU (see
// wave_emulator.h).  Built, fed and checked by test_select_emulation.py.
// Input, one case after the other, words in hexadecimal:
//   waves snap n_sel window k_sel pool_kernel hint_lo hint_hi classify order, then n_sel words
//   (floats), and with classify = 1 another n_sel words: the packed bounds, classified before
//   the words (exact scores) of the tokens that are named take their place.
// order: bit 0 lanes, bit 1 wavefronts from the highest down.
// Output per case: key_lo key_hi, the kept tokens, the final scores, one name per token.
#include "wave_emulator.h"

#include "../paper_2503_08461_amd/csrc/fc_unit.h"

#include <algorithm>
#include <memory>

using namespace fc;

template <int WV>
static void run_case(const ReqDesc& rd, int n_sel, const std::vector<uint32_t>& words,
                     const std::vector<uint32_t>& bounds, uint32_t key_lo, uint32_t key_hi, int order) {
  const int L = rd.seq_len;
  // LDS: the per-token words, then the map (filled with what must not matter)
  std::vector<uint32_t> lds(stage_words(L) + need_words(L), 0xDEADBEEFu);
  uint32_t* stage = lds.data() + kStageFront;
  uint32_t* map = lds.data() + stage_words(L);
  auto sh = std::make_unique<SelectShared<WV>>();
  std::fill_n(reinterpret_cast<char*>(sh.get()), sizeof(*sh), (char)0x5A);
  std::vector<int32_t> kept(rd.budget, -7);
  std::vector<float> scores(L, -7.f);
  std::vector<int> named(n_sel, 0);
  BatchParams p = {};
  p.scores_out = scores.data();
  if (!bounds.empty()) {
    std::copy(bounds.begin(), bounds.end(), stage);
    emu::run_block(WV, order & 2, order & 1, [&] {
      uint32_t lo = 0, hi = 0;
      bound_classify<WV>(rd, stage, map, *sh, lo, hi);
      key_lo = lo;
      key_hi = hi;
    });
    for (int j = 0; j < n_sel; ++j) {
      named[j] = (map[j >> 5] >> (j & 31)) & 1u;
      if (named[j]) stage[j] = words[j];
    }
  } else {
    std::copy(words.begin(), words.end(), stage);
  }
  emu::run_block(WV, order & 2, order & 1, [&] {
    select_unit<WV>(p, rd, 0, stage, map, kept.data(), *sh, key_lo, key_hi);
  });
  printf("%x %x\n", key_lo, key_hi);
  for (int32_t k : kept) printf("%d ", k);
  printf("\n");
  for (float s : scores) printf("%x ", __builtin_bit_cast(uint32_t, s));
  printf("\n");
  for (int b : named) printf("%d ", b);
  printf("\n");
}

int main() {
  int waves, snap, n_sel, window, k_sel, width, classify, order;
  uint32_t lo, hi;
  while (scanf("%d %d %d %d %d %d %x %x %d %d", &waves, &snap, &n_sel, &window, &k_sel, &width, &lo, &hi,
               &classify, &order) == 10) {
    auto read = [&](int n) {
      std::vector<uint32_t> v(n);
      for (uint32_t& x : v)
        if (scanf("%x", &x) != 1) exit(2);
      return v;
    };
    const std::vector<uint32_t> words = read(n_sel), bounds = read(classify ? n_sel : 0);
    ReqDesc rd = {};
    rd.method = snap ? 1 : 2;
    rd.window = snap ? window : 0;
    rd.seq_len = n_sel + rd.window;
    rd.budget = k_sel + rd.window;
    rd.pool_kernel = width;
    if (waves == 4)
      run_case<4>(rd, n_sel, words, bounds, lo, hi, order);
    else if (waves == 12)
      run_case<12>(rd, n_sel, words, bounds, lo, hi, order);
    else
      run_case<16>(rd, n_sel, words, bounds, lo, hi, order);
    fflush(stdout);
  }
  return 0;
}
