// The order of the scores and the bins of the selection by blocks: the arithmetic alone, without a GPU type, so that a CPU build
// can be tested over all score values.
#pragma once
#include <stdint.h>
#ifdef __HIP__
#define DMA_SELECT_FN __device__ __forceinline__
#else
#define DMA_SELECT_FN inline
#endif

namespace dma {

// Bins of a block, and of a checkpoint, which has far more keys before it (65536 tokens x 32 heads, window 16384, checkpoints alone,
// 1024 / 2048 / 4096 bins: 75 / 52 / 48 us).
constexpr int BIN_BITS = 10, CK_BIN_BITS = 12;
// Keys that the two bins may hold beside those of the ranks between: runs of ties are narrowed down, not compared key by key (2 x
// 4096 tokens x 16 heads, window 1024, a third of the scores the same: 512 / 256 of them 97 / 54 us).
constexpr int NEAR = 256;
constexpr int CAP = 256 + NEAR;  // keys that the ranking takes

DMA_SELECT_FN uint32_t float_bits(float x) { return __builtin_bit_cast(uint32_t, x); }
DMA_SELECT_FN float bits_float(uint32_t x) { return __builtin_bit_cast(float, x); }
// Ascending unsigned order of the result == descending float order of z (-0 and +0 compare equal).
DMA_SELECT_FN uint32_t desc_key(float z) {
  z = z + 0.0f;
  uint32_t u = float_bits(z);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ~u;
}
// A score with this key.
DMA_SELECT_FN float key_value(uint32_t key) {
  const uint32_t u = ~key;
  return bits_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// Bins between the best and the worst score: equal steps of the bits of z + add, so of about the logarithm.  Scores are
// exponentials of a gate of either sign, and equal steps of the score leave nearly all of them in one bin once they spread
// over a few powers of two.  Whole dma_mask_gen, 16384 x 32, window 2048, us, a sort / steps of the score / these: gates of -0.5 to
// -2 110 / 60 / 63, of 4 108 / 307 / 60, of 1 with three times the spread 109 / 303 / 74.  add: none for scores within 24 powers
// of two of the best; a 2^24th of the best where some are lower (one zero would else take most of the bins: 109 / 60 / 96 with
// zeros; scores over 80 powers of two 108 / 310 / 132, a few outliers of 1e30 110 / 312 / 152); with negative scores so much that
// the worst is an eighth of the spread (nearly equal steps of the score: normal scores 110 / 60 / 61).
template <int BITS> struct Bins {
  float add, top, low;
  uint32_t first;  // bits of top + add
  int shift;
  bool ok;  // the scores are finite and not all the same
  // kmin: the best key.  kmax: the worst that matters
  DMA_SELECT_FN void init(uint32_t kmin, uint32_t kmax) {
    top = key_value(kmin);
    low = key_value(kmax);
    const float range = top - low, least = top * 0x1p-24f;
    add = low < 0.f ? range * 0.125f - low : low < least ? least : 0.f;
    first = float_bits(top + add);
    const uint32_t last = float_bits(low + add);
    ok = range > 0.f && add < __builtin_inff() && first < 0x7f800000u && last < first;  // (false for NaN)
    const int bits = 32 - __builtin_clz(first - last | 1u);
    shift = bits > BITS ? bits - BITS : 0;
  }
  // never falls along descending scores from top to low
  DMA_SELECT_FN uint32_t of(float z) const { return (first - float_bits(z + add)) >> shift; }
  // ... and on for what is behind that: the last bin or beyond the bins
  DMA_SELECT_FN uint32_t of_behind(float z) const {
    const int32_t bits = (int32_t)float_bits(z + add);
    return (first - (uint32_t)(bits > 0 ? bits : 0)) >> shift;
  }
  DMA_SELECT_FN uint32_t of_any(float z) const { return of(__builtin_fminf(__builtin_fmaxf(z, low), top)); }
  // the first key that is not before a bin (one behind that of low, if there is none)
  DMA_SELECT_FN uint32_t bound(uint32_t bin) const {
    uint32_t lo = desc_key(top), hi = desc_key(low) + 1;
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (of(key_value(mid)) < bin) lo = mid + 1; else hi = mid;
    }
    return lo;
  }
};

}  // namespace dma
