// The selection of the causal plan, by blocks (select.hip), and what the decode selection shares with it.
#pragma once
#include "common.h"
#include "select_bins.h"

namespace dma {

constexpr int CK_SEG = 4096;   // keys between two checkpoints of a long document
constexpr int CK_DOC = 16384;  // documents longer than this have them (below, their launch costs more than shorter reads save)
// Documents longer than this are sorted instead: the checkpoints' cost grows with the square of the length, and scores of few values
// take more passes.  us of dma_mask_gen, window 2048, sorted / by blocks, random scores and scores of sixteen values: 131072 tokens x
// 8 heads 482 / 149 and 424 / 234, x 32 810 / 342 and 693 / 498, 262144 x 32 1771 / 770 and 1245 / 1282, 524288 x 32
// 5107 / 1995 and 2454 / 3787: up to this length neither loses.
constexpr int SELECT_MAX = 131072;

struct SelectArgs {
  const float* z;
  const int32_t* cu;
  const int4* blk;
  int32_t* parent;     // [H_q][T]: key evicted by each row; -1: none; -2: the row's own key never enters
  int32_t* expiry;     // [H_q][T]: the document's end, or the row itself if its key never enters (the slot kernels set those of evicted keys)
  float* ck_z;         // [H_q][T]: checkpoints' scores
  int32_t* ck_idx;     // [H_q][T]: and indices in their document
  int T, n_docs, nblk_cap, k;
  int ck_min;          // documents longer than this have checkpoints
};

#ifdef __HIPCC__
// Checkpoints of a document that starts at a: number p stands before its key c = CK_SEG (p + 1) and is stored at the place of
// the CK_SEG keys before c.  It holds the weakest ck_keys(k) of the keys kept by row c - 1 (k <= CK_SEG: all of them, and up
// to three more), in any order, but the last of them first if there are others.
__device__ __forceinline__ int ck_keys(int k) { return k < CK_SEG ? (k + 3) & ~3 : CK_SEG; }
// Place of piece p of document d among the pieces of SEG keys of all documents.
template <int SEG> __device__ __forceinline__ int piece_slot(int a, int d, int p) { return a / SEG + d + p; }
// The document of a place: the largest d with piece_slot(cu[d], d, 0) <= slot.
template <int SEG> __device__ __forceinline__ int piece_doc(const int32_t* __restrict__ cu, int n_docs, int slot) {
  int lo = 0, hi = n_docs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (piece_slot<SEG>(cu[mid], mid, 0) <= slot) lo = mid; else hi = mid;
  }
  return lo;
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

// longest: upper bound on the documents' length (a wrong one changes no result).  The caller asks for launch errors.
void launch_evictions(const SelectArgs& a, int longest, int H_q, hipStream_t st);

}  // namespace dma
