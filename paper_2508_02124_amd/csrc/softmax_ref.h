// The reference maximum of the online softmax, in the exp2 domain: the arithmetic alone, without a GPU type, so that a
// CPU build can be tested over all score values.
#pragma once
#include <float.h>
#include <stdint.h>
#ifdef __HIP__
#define DMA_FN __device__ __forceinline__
#else
#define DMA_FN static inline
#endif

namespace dma {

// The reference of a row that has kept nothing yet: a masked score (-inf) then gets the weight exp2(-inf) = 0, as with
// any other reference, and every other score an infinite weight, so that its sum asks for the maximum.  (With -inf
// here a masked score would give -inf + inf: the forward is compiled for arithmetic without NaNs.)
constexpr float REF_NONE = -FLT_MAX;
// Largest sum of a lane's sixteen weights of one unit that is taken without a look at the maximum (2^8), as the bits of
// a float: sums are not negative.  (A float limit needs a register more: the kernel of 64 channels 254 -> 271 us at
// 65536 packed tokens x 16 heads.)
constexpr uint32_t SUM_LIMIT = 0x43800000u;

// Argument of exp2 of a score's weight.
DMA_FN float weight_exponent(float score, float c2, float ref) { return __builtin_fmaf(score, c2, -ref); }

// Largest exponent of a row's greatest weight: sums of 2^16 such weights times values up to 2^10 are finite.
constexpr float MAX_EXPONENT = 100.f;

// The reference for weights whose largest score is top.  The product is rounded and weight_exponent's is not, so the
// largest weight is 2^e with e up to half of the product's last place.  That cancels in the softmax (rows that keep
// nothing but keys masked by a bias of -1e9: all weights 2^e) until 2^e overflows, as it can from a bias of -1.5e9 on: then
// the next float above is taken, the weights are 0, and what the row keeps later counts alone.
DMA_FN float reference_of(float top, float c2) {
  float ref = __builtin_fmaxf(top * c2, REF_NONE);  // (top = -inf: nothing kept)
  if (weight_exponent(top, c2, ref) > MAX_EXPONENT) {
    const int32_t b = __builtin_bit_cast(int32_t, ref);
    ref = __builtin_bit_cast(float, b + (b < 0 ? -1 : 1));
  }
  return ref;
}

}  // namespace dma
