// The selection of the causal plan, by blocks (select.hip), and what the decode selection shares with it.
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
// Wave-wide inclusive sum, minimum and maximum in registers (data-parallel moves: a lane shuffle through LDS takes ten times as
// long).
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp(uint32_t identity, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)x, CTRL, ROWS, 0xf, false);
}
template <typename F> __device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, F&& op) {
  x = op(x, dpp<0x111, 0xf>(identity, x));  // row_shr:1, 2, 4, 8
  x = op(x, dpp<0x112, 0xf>(identity, x));
  x = op(x, dpp<0x114, 0xf>(identity, x));
  x = op(x, dpp<0x118, 0xf>(identity, x));
  x = op(x, dpp<0x142, 0xa>(identity, x));  // row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
  return op(x, dpp<0x143, 0xc>(identity, x));
}
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
#endif

// longest: upper bound on the documents' length (a wrong one changes no result)
int launch_evictions(const SelectArgs& a, int longest, int H_q, hipStream_t st);

}  // namespace dma
