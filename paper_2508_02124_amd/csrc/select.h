// The selection of the causal plan, by blocks (select.hip).
#pragma once
#include "common.h"

namespace dma {

constexpr int CK_SEG = 4096;   // keys between two checkpoints of a long document
constexpr int CK_DOC = 16384;  // documents longer than this have them (below, their launch costs more than shorter reads save)
// Documents longer than this are sorted instead: the checkpoints' cost grows with the square of the length.  us of
// dma_mask_gen, sorted / by blocks, random scores: 65536 tokens x 8 heads 276 / 124, 131072 x 8 470 / 302, 262144 x 8
// 825 / 590 (32 heads fill the chip, and then the square counts: about equal).
constexpr int SELECT_MAX = 131072;

struct SelectArgs {
  const float* z;
  const int32_t* cu;
  const int4* blk;
  int32_t* parent;     // [H_q][T]: key evicted by each row; -1: none; -2: the row's own key never enters
  float* ck_z;         // [H_q][T]: checkpoints' scores
  int32_t* ck_idx;     // [H_q][T]: and indices in their document
  int T, n_docs, nblk_cap, k;
  int ck_min;          // documents longer than this have checkpoints
};

#ifdef __HIPCC__
// Ascending unsigned order of the result == descending float order of z (-0 and +0 compare equal).
__device__ __forceinline__ uint32_t desc_key(float z) {
  z = z + 0.0f;
  uint32_t u = __float_as_uint(z);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ~u;
}
#endif

// longest: upper bound on the documents' length (a wrong one changes no result)
int launch_evictions(const SelectArgs& a, int longest, int H_q, hipStream_t st);

}  // namespace dma
