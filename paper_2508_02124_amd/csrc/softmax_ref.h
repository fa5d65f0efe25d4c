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

// Argument of exp2 of a score's weight.
DMA_FN float weight_exponent(float score, float c2, float ref) { return __builtin_fmaf(score, c2, -ref); }

// The reference for weights whose largest score is top.  The product is rounded and weight_exponent's is not: where
// its last place is worth more than a few powers of two (keys masked by a bias of -1e10 or below, and nothing else kept
// so far), exp2 of the difference alone could be infinite.  Then the next float above is taken, and no weight exceeds 1.
DMA_FN float reference_of(float top, float c2) {
  float ref = __builtin_fmaxf(top * c2, -FLT_MAX);  // (top = -inf: nothing kept; -inf - -inf is not formed)
  if (weight_exponent(top, c2, ref) > 1.f) {
    const int32_t b = __builtin_bit_cast(int32_t, ref);
    ref = __builtin_bit_cast(float, b + (b < 0 ? -1 : 1));
  }
  return ref;
}

}  // namespace dma
