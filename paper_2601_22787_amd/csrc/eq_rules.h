// Host rules that choose how a call is launched.  No device code, so that
// they can be checked without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace eq_detail {

// Version 1, rows that are not whole steps: whether the GEMV decodes and
// multiplies in one kernel, or decodes to codes first and multiplies those, a
// block per row.  In the fused kernel every row that ends inside a chunk costs
// its wavefront some 0.1 to 0.5 us of its chain (more with more batch rows).
// That is hidden where compute units have several chunks each (fewer are
// enough for long rows, whose separate product has more to read) and small
// where a chunk holds few rows.  Both ways timed at 5340 points (65 to 11000
// columns, chunks of 1024 to 65536, 64 to 256 lanes, 4 to 16384 chunks, batch 1
// to 8): the rule's choice takes 1.01 times the faster one's time on average,
// 1.43 at worst (always the fused kernel: 1.17 at batch 1 to 1.60 at batch 8,
// 16 at worst; never: 1.61 to 1.29, 13 at worst).
inline bool ragged_fused(uint32_t n_chunks, uint32_t cols, uint32_t chunk_syms, uint32_t B,
                         uint32_t cus) {
  const double t = B == 1 ? 1.0 : B == 2 ? 1.25 : B <= 4 ? 2.0 : 3.0;
  return n_chunks * (1.0 + double(B) * cols / 8192.0) >= t * cus ||
         cols >= (B == 1 ? 0.25 : 0.4) * chunk_syms;
}

// Version 2: wavefronts per block for layers of n[0..k-1] tiles (each layer's
// tiles in blocks of their own, a wavefront per tile), blocks of tb + waves x
// wl bytes of LDS; 0 if not even one wavefront fits.  Start from one block
// per compute unit (total tiles / CUs wavefronts) and add wavefronts until
// the blocks fit one round (the blocks that LDS lets each compute unit hold
// at once); when no count up to the limit does, take the count in [limit / 2,
// limit] of the smallest estimate (the larger on ties): each round costs
// kChain, a tile's chain of steps, plus the wavefronts that share a compute
// unit, so fewer rounds come first and even ones second.
// Against all counts timed (1482 to 10952 tiles of 64 to 256 rows and 64 to
// 256 columns; codes, BF16 and the GEMV at batch 1, 2, 4 and 8): the choice
// takes 1.00 to 1.01 times the fastest count's time on average per operation,
// 1.11 at worst, with any kChain from 4 to 30.  The rounds alone of one
// resident block per unit: 1.21 at worst (batch 4); rounds x wavefronts
// without the chain: 1.01 to 1.12, 1.56 at worst.
struct WaveChoice {
  uint32_t waves;
  uint64_t cost;  // the estimate
};
inline WaveChoice choose_waves(const uint32_t *n, uint32_t k, uint32_t wmax, size_t tb, size_t wl,
                               uint32_t lds, uint32_t cus) {
  constexpr uint64_t kChain = 16;
  while (wmax > 0 && tb + size_t(wmax) * wl > size_t(lds)) --wmax;
  if (wmax == 0) return {0, 0};
  uint64_t total = 0;
  for (uint32_t i = 0; i < k; ++i) total += n[i];
  auto blocks = [&](uint32_t w) {
    uint64_t b = 0;
    for (uint32_t i = 0; i < k; ++i) b += (n[i] + w - 1) / w;
    return b;
  };
  auto resident = [&](uint32_t w) { return uint64_t(size_t(lds) / (tb + size_t(w) * wl)); };
  auto cost = [&](uint32_t w) {
    const uint64_t r = resident(w), b = blocks(w), last = b % (cus * r);
    return b / (cus * r) * (kChain + r * w) + (last ? kChain + (last + cus - 1) / cus * w : 0);
  };
  uint32_t w = uint32_t(std::min<uint64_t>(std::max<uint64_t>((total + cus - 1) / cus, 1), wmax));
  while (w < wmax && blocks(w) > cus * resident(w)) ++w;
  if (blocks(w) > cus * resident(w)) {
    uint64_t best = ~uint64_t(0);
    for (uint32_t v = wmax; v >= 1 && v >= (wmax + 1) / 2; --v) {
      if (cost(v) < best) {
        best = cost(v);
        w = v;
      }
    }
  }
  return {w, cost(w)};
}

// Version 2, codes and BF16: 64-code output segments instead of 32-code ones,
// from both ways' estimates.  tile_rows: the tallest tiles'; out: output
// bytes; words, codes: stream words and codes of all layers.  At the same
// rounds and wavefronts 64-code segments take 0.90 to 0.97 of the time.
// Their rings leave room for fewer wavefronts, and more rounds cost more than
// that (4096 tiles of 128 x 128 to codes: 43 us in one round of 16, 62 in two
// of 8; 4096 of 256 x 256 to BF16: 304 against 347; 12544 of 64 x 256 to codes:
// 112 against 125), except at 64- and 128-row tiles where the output outgrows
// the memory-side cache and the stores, not the decode, bound the launch: a
// seventh more of the estimate (14336 of 64 x 256 to BF16, 470 MB: 213 -> 182 us
// at 2 bits a code, 266 -> 247 at 4), or three tenths at few bits (7168 of 128 x
// 256 to BF16: 229 -> 191 us at 2 bits, but 269 against 290 at 3.5; 8192 to
// codes, 268 MB: 194 -> 171 at 2, but 235 against 256 at 3.5; to codes, 235 MB:
// 140 against 165 at 2).
inline bool long_segments(uint64_t cost32, uint64_t cost64, uint32_t tile_rows, uint64_t out,
                          uint64_t words, uint64_t codes) {
  if (cost64 <= cost32) return true;
  const bool few_bits = 64 * words <= 11 * codes;  // at most 2.75 bits a code
  return tile_rows <= 128 && out > (uint64_t(240) << 20) &&
         100 * cost64 <= (few_bits ? 130 : 115) * cost32;
}

}  // namespace eq_detail
