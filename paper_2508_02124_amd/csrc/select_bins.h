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

// Bins of a block, and of a checkpoint, which has far more keys before it (65536 tokens x 32 heads, window 16384, checkpoints
// alone, 1024 / 2048 / 4096 bins: 75 / 52 / 48 us).
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

// Bins between two of the scores, the best and the worst of a sample; what lies beyond takes the first or the last bin.  Equal
// steps of the bits of z + add, so of about the logarithm: scores are exponentials of a gate of either sign, and equal steps
// of the score leave nearly all of them in one bin once they spread over a few powers of two.  A sample, because a few outliers
// or zeros must not decide how long a step is.  add: none, or with negative scores so much that the worst is an eighth of the
// spread (nearly equal steps of the score).
// Whole dma_mask_gen, 16384 x 32, window 2048, us, a sort / equal steps of the score / equal steps of the bits, both between the best
// and the worst of all / these: gates of -0.5 to -2 110 / 60 / 63 / 61, of 4 109 / 307 / 60 / 59, of 1 with three times the spread
// 109 / 303 / 74 / 64, of 6 with it 108 / 310 / 133 / 68, a few outliers of 1e30 110 / 312 / 152 / 107, a tenth of them -inf
// 110 / 235 / 138 / 81, normal scores 108 / 59 / 62 / 61.
template <int BITS> struct Bins {
  float add;
  uint32_t first, last;  // bits of top + add and of low + add
  int shift;
  bool ok;  // top and low are finite and not the same
  DMA_SELECT_FN void init(uint32_t kmin, uint32_t kmax) {  // (kmin > kmax: nothing was sampled)
    const float top = key_value(kmin), low = key_value(kmax), range = top - low;
    add = low < 0.f ? range * 0.125f - low : 0.f;
    first = float_bits(top + add);
    last = float_bits(low + add);
    ok = kmin < kmax && range < __builtin_inff() && add < __builtin_inff() && first < 0x7f800000u && last < first;  // (false for NaN)
    const int bits = 32 - __builtin_clz(first - last | 1u);
    shift = bits > BITS ? bits - BITS : 0;
  }
  // never falls along descending scores; the last bin for what is not a number (the sum has made it quiet)
  DMA_SELECT_FN uint32_t of(float z) const {
    const float y = z + add, y0 = bits_float(last), y1 = bits_float(first);
#ifdef __HIP__
    return (first - float_bits(__builtin_amdgcn_fmed3f(y, y0, y1))) >> shift;
#else
    return (first - float_bits(__builtin_fminf(__builtin_fmaxf(y, y0), y1))) >> shift;
#endif
  }
  DMA_SELECT_FN bool behind(float z) const { return z + add < bits_float(last); }
  // z + add of the scores in bins b0 to b1: from least to most
  DMA_SELECT_FN float most(uint32_t b0) const { return b0 == 0 ? __builtin_inff() : bits_float(first - (b0 << shift)); }
  DMA_SELECT_FN float least(uint32_t b1) const {
    return b1 >= (first - last) >> shift ? -__builtin_inff() : bits_float(first - ((b1 + 1) << shift) + 1);
  }
  // the first key that is not before a bin, or, if `cut`, is behind; one behind that of -inf, if there is none
  DMA_SELECT_FN uint32_t bound(uint32_t bin, bool cut) const {
    uint32_t lo = desc_key(__builtin_inff()), hi = desc_key(-__builtin_inff()) + 1;
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (of(key_value(mid)) < bin && !(cut && behind(key_value(mid)))) lo = mid + 1; else hi = mid;
    }
    return lo;
  }
};

}  // namespace dma
