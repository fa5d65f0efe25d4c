// Forward pass (Eq. 5-6; online softmax of Alg. 1, query-stationary so O, l, m stay in registers).
//
// One workgroup = one block of BQ = 256 query rows of one head (8 waves) or half of one (4 waves); wave w owns 32 of
// its rows.  The keys a block needs are gathered a tile at a time (64 keys, or 32) into rings of four LDS stages by
// asynchronous global->LDS copies issued two to three tiles ahead (no staging registers): first the slot table row of
// the block (residents active for every row of the block: no mask needed, empty slots carry
// z = -inf), then the block's partial list (keys entering or expiring inside the block: pairs
// outside j <= i < e_j get a score of -inf).  The key ids of a tile are themselves copied
// into an LDS ring two tiles before the tile's K copies are issued, so no register ever waits on a load.
//
// Work is done in units of 32 keys.  The wave computes S^T = K Q^T (keys x queries) so that each lane holds one query
// column: the softmax statistics are per lane, and the exponentiated block is already laid out
// as the B operand of O^T += V^T P^T.  The bias z is not added after the product: the accumulator
// starts at z / scale, so scale * acc is the biased score and one FMA gives the exp2 argument.  The step of a unit also
// holds the next unit's S product and the previous unit's PV product, interleaved with its exponentials instruction by
// instruction.
//
// What bounds it: at 64K tokens, 32 heads, d = 128, window 16384 a tile of 64 keys takes 3100 cycles against 2048 of the
// matrix pipe, at a clock that the power limit holds at 1.8 to 1.9 GHz: fewer instructions and fewer bytes moved give
// more than a tighter schedule (leaving out the copies alone raises the clock by 15 %).  Each wave doing the whole
// chain of a tile at a time took 15.1 ms there, this form 13.9; 16384 tokens, window 2048: 592 -> 548 us; 16 heads of
// 256 channels, where no second wave of a SIMD fills the gaps: 882 -> 628 us.
#include "common.h"
#include "softmax_ref.h"
#include <cmath>

namespace dma {

struct FwdArgs {
  const uint16_t *Q, *K, *V;
  uint16_t* O;
  const float* zq;      // z / softmax_scale
  float* LSE;
  const int32_t* expiry;
  const int4* blk;
  const int32_t* slot_tab;
  const int32_t* pcnt;
  const int32_t* plist;
  const char* consts;   // [0,256) zeros; +256: float -inf; +260: int 0; +264: int -1; +272: softmax scale, scale * log2(e)
  int T, H_q, H_kv, k, nblk_cap, kpad;
};

// (second launch bound = waves per SIMD: at D = 64 the kernel is held to 128 registers so that two
// workgroups share a compute unit -- four waves per SIMD hide the element-wise work, which weighs
// twice as much per MFMA there; at D = 128 the accumulators alone need more than that)
// NW waves per workgroup: 8 (one 256-row block per workgroup) or 4 (half a block); UT 32-key units per tile.  Four waves
// with tiles of 32 keys leave room for a second workgroup on the compute unit: the two waves of a SIMD then belong to
// different workgroups and do not meet at the same barriers.
// PARTS: waves that share the same 32 rows.  Each takes its own units of every tile, with statistics of its own; at the
// end the first one takes in the others' (all are the same softmax).  For calls of so few blocks that a wave would else
// walk its keys alone on its SIMD, with nothing to fill the gaps between the products' results and their uses.
template <int D, int NW, int UT, int PARTS = 1>
__global__ __launch_bounds__(NW * 64, D == 64 && PARTS == 1 ? 4 : ((NW == 8 || D == 256) ? 1 : 2)) void fwd_kernel(FwdArgs p) {
  using TL = TileLayout<D>;
  constexpr int KS = D / 16;          // contraction steps of K Q^T
  constexpr int CB = D / 32;          // 32-channel blocks of O^T
  constexpr int CPR = D / 8;          // 16-byte chunks per row
  constexpr int RPL = 64 / CPR;       // rows covered by one wave-wide 16-byte copy
  constexpr int KT = 32 * UT * PARTS; // keys per tile
  constexpr int WL = KT / RPL / NW;   // such copies per wave per K (or V) tile
  constexpr int NS = 4;               // ring stages
  constexpr int NT = NW * 64;         // threads
  constexpr int RW = NW / PARTS;      // 32-row groups
  constexpr int HALVES = 8 / RW;      // workgroups per 256-row block
  constexpr int TILE = KT * D;        // elements of one K or V tile
  __shared__ __align__(16) uint16_t ringK[NS * TILE];
  __shared__ __align__(16) uint16_t ringV[NS * TILE];
  __shared__ __align__(16) int ids_ring[2 * NS][64];  // (rows of 64: what one wave-wide copy writes)
  __shared__ __align__(16) float z_ring[NS][64];
  __shared__ __align__(16) int e_ring[NS][64];

  int h, item;
  if (!xcd_map(wg_id(), p.H_q, p.nblk_cap * HALVES, h, item)) return;
  const int bi = p.nblk_cap - 1 - item / HALVES;  // long blocks first
  const int tid = thread_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, n = l & 31, hh = l >> 5;
  const int wr = w % RW, part = w / RW;
  const int32_t* slot_row = p.slot_tab + ((size_t)h * p.nblk_cap + bi) * p.kpad;
  const int32_t* c_m1 = reinterpret_cast<const int32_t*>(p.consts + 264);
  // The key ids of the first tiles are requested with the block's table entry, as if all of these were slot columns: one
  // memory latency less before the first rows (where there are fewer, the others are requested again below).  65536
  // tokens, window 1024: 1320 -> 1275 us.  (64 channels: two workgroups per compute unit hide that latency, and the
  // registers do not: 253 -> 275.)
  constexpr int FIRST = 5;
  constexpr bool EARLY = D != 64 || PARTS > 1;
  if (EARLY && w == 0) {
#pragma unroll
    for (int tt = 0; tt < FIRST; tt++) {
      const int c = tt * KT + (l & (KT - 1));
      dma4(c < p.kpad ? slot_row + c : c_m1, &ids_ring[tt % (2 * NS)][0]);
    }
  }
  const int4 info = p.blk[bi];
  const int np_keys = p.pcnt[(size_t)h * p.nblk_cap + bi];
  const float c2 = *reinterpret_cast<const float*>(p.consts + PLAN_C2_OFF);  // softmax scale * log2(e)
  if (info.x < 0) {
    wait_vmcnt<0>();  // (no copy may outlive the workgroup)
    return;
  }
  const int blk_row0 = info.y, row1 = info.z, doc0 = info.w;
  const int row0 = blk_row0 + (item % HALVES) * (RW * 32);  // first row of this workgroup's part of the block
  if (row0 >= row1) {
    wait_vmcnt<0>();
    return;
  }
  const int g = h / (p.H_q / p.H_kv);
  const int ncol = min(p.k, blk_row0 - doc0);
  const int nc = (ncol + KT - 1) / KT;
  const int shift = (NS - nc % NS) % NS;  // ring stage of tile 0: tile t takes stage (t + shift) % NS
  const int nt = nc + (np_keys + KT - 1) / KT;
  const int32_t* plist_row = p.plist + ((size_t)h * p.nblk_cap + bi) * MAXPART;
  const float* zqh = p.zq + (size_t)h * p.T;
  const int32_t* eh = p.expiry + (size_t)h * p.T;
  const float* c_ninf = reinterpret_cast<const float*>(p.consts + 256);
  const int32_t* c_zero = reinterpret_cast<const int32_t*>(p.consts + 260);

  // ---- asynchronous producers (every wave issues the same number of copies for every tile index,
  // real or past the end, so the outstanding-copy counts below are constants).  A gathered row is
  // addressed as a wave-uniform base (the kv-head's first row) plus a 32-bit byte offset
  // id * row pitch + the lane's chunk; an empty slot (id < 0) copies row 0 instead, which its score
  // of -inf keeps out of every sum.
  const void* Kg = uniform_ptr(p.K + (size_t)g * D);
  const void* Vg = uniform_ptr(p.V + (size_t)g * D);
  const uint32_t row_pitch = (uint32_t)p.H_kv * D * 2;
  uint32_t lane_chunk[WL];  // byte offset of the lane's 16-byte chunk within its row, per copy
  int lane_row[WL];         // tile row the lane copies
#pragma unroll
  for (int j = 0; j < WL; j++) {
    lane_row[j] = (w * WL + j) * RPL + l / CPR;
    lane_chunk[j] = (uint32_t)(((l % CPR) ^ TL::swz(lane_row[j])) * 16);
  }
  const uint32_t ldsK = lds_addr(ringK) + (uint32_t)(w * WL * RPL * D * 2);
  const uint32_t ldsV = lds_addr(ringV) + (uint32_t)(w * WL * RPL * D * 2);
  auto issue_ids = [&](int tt) {
    if (w == 0) {
      const int32_t* src = c_m1;
      const int ll = l & (KT - 1);
      if (tt < nc) {
        src = slot_row + tt * KT + ll;
      } else if (tt < nt) {
        const int q = (tt - nc) * KT + ll;
        if (q < np_keys) src = plist_row + q;
      }
      dma4(src, &ids_ring[tt % (2 * NS)][0]);
    }
  };
  // rows of tile tt: the key ids first (an LDS read), the copies once they are there
  auto row_ids = [&](int tt, int (&idv)[WL]) __attribute__((always_inline)) {
    const int* idr = ids_ring[tt % (2 * NS)];
#pragma unroll
    for (int j = 0; j < WL; j++) idv[j] = idr[lane_row[j]];
  };
  auto copy_rows = [&](const void* base, uint32_t lds, int stage, const int (&idv)[WL]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WL; j++)
      dma16u(base, mul24((uint32_t)max(idv[j], 0), row_pitch) + lane_chunk[j],
             lds + (uint32_t)((stage * TILE + j * RPL * D) * 2));
  };
  auto issue_rows = [&](const void* base, uint32_t lds, int tt) __attribute__((always_inline)) {
    int idv[WL];
    row_ids(tt, idv);
    copy_rows(base, lds, (tt + shift) % NS, idv);
  };
  auto issue_scalars = [&](int tt) {
    if (w == 1) {
      const int idl = ids_ring[tt % (2 * NS)][l];
      dma4(idl >= 0 ? zqh + idl : c_ninf, &z_ring[(tt + shift) % NS][0]);
      dma4(idl >= 0 ? (const void*)(eh + idl) : (const void*)c_zero, &e_ring[(tt + shift) % NS][0]);
    }
  };
  // Iteration t of the tile loops requests the ids of tile t + 5, K rows and scalars of tile t + 3 and V rows of tile
  // t + 2, and starts when everything requested before iteration t - 1 has landed: K up to tile t + 1, V up to tile t.
  auto issue_small = [&](int t) __attribute__((always_inline)) {
    issue_ids(t + 5);
    issue_scalars(t + 3);
  };
  auto wait_tile = [&]() {
    if (w == 0) wait_vmcnt<2 * WL + 1>();
    else if (w == 1) wait_vmcnt<2 * WL + 2>();
    else wait_vmcnt<2 * WL>();
  };

  if (EARLY) {
    if (w == 0 && nc < FIRST) {
      wait_vmcnt<0>();
      for (int tt = nc; tt < FIRST; tt++) issue_ids(tt);
    }
  } else {
    for (int tt = 0; tt < FIRST; tt++) issue_ids(tt);
  }
  // query fragments (B operand of K Q^T): lane holds row qi, channels 16*ks + 8*hh .. +8
  const int qi = row0 + 32 * wr + n;
  bf16x8 qreg[KS];
  {
    // (EARLY: rows past the end repeat the last one: the same number of loads for every wave, and results that nothing stores)
    const uint16_t* qrow = p.Q + ((size_t)(EARLY ? min(qi, row1 - 1) : qi) * p.H_q + h) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      uint4 raw = make_uint4(0, 0, 0, 0);
      if (EARLY || qi < row1) raw = *reinterpret_cast<const uint4*>(qrow + 16 * ks);
      qreg[ks] = __builtin_bit_cast(bf16x8, raw);
    }
  }
  // The pipelined loop's first step multiplies the (zero) weights before the first unit with the last unit of the ring
  // stage before it (of their part): those rows have to hold numbers.
  for (int c = tid; c < PARTS * 32 * CPR; c += NT)
    reinterpret_cast<uint4*>(ringV + (shift + NS - 1) % NS * TILE + (c / (32 * CPR) * UT + UT - 1) * 32 * D)[c % (32 * CPR)] =
        make_uint4(0, 0, 0, 0);
  if (EARLY) {
    wait_vmcnt<KS>();  // the ids; the loads of Q may still be on their way
  } else {
    wait_vmcnt<0>();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) settle(qreg[ks]);
  }
  lds_barrier();
  for (int i = 0; i < 3; i++) {
    issue_rows(Kg, ldsK, i);
    issue_scalars(i);
    if (i < 2) issue_rows(Vg, ldsV, i);
  }
  if (EARLY) {
#pragma unroll
    for (int ks = 0; ks < KS; ks++) settle(qreg[ks]);
  }

  // The lane's fragment addresses with the ring bases folded in: inside the (stage-unrolled) main
  // loop every LDS read is one of these registers plus an immediate.  The part's first unit is folded in too.
  const int unit0 = 32 * UT * part;
  FragOffsets<D> fo;
  fo.init(l);
  uint32_t kfrag[KS], vfrag[CB][2];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    kfrag[ks] = lds_addr(ringK) + 2 * (fo.row(ks) + unit0 * D);
    settle(kfrag[ks]);
  }
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int q = 0; q < 2; q++) {
      vfrag[cb][q] = lds_addr(ringV) + 2 * (fo.tr(cb, q) + unit0 * D);
      settle(vfrag[cb][q]);
    }
  uint32_t zlane = lds_addr(&z_ring[0][unit0 + 4 * hh]);
  const uint32_t jlane = lds_addr(&ids_ring[0][unit0 + 4 * hh]), elane = lds_addr(&e_ring[0][unit0 + 4 * hh]);
  settle(zlane);
  f32x16 oacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int v = 0; v < 16; v++) oacc[cb][v] = 0.f;
  float m_run = REF_NONE, lsum = 0.f;
  uint32_t limit = 0;  // largest sum without a look at the maximum: nothing in the first 64 keys, then SUM_LIMIT

  // S^T of one unit; its accumulator starts at z / scale, so that scale * acc is the biased score.  so, zo: byte offsets
  // of the unit in the K ring and in the ring of the scalars.
  auto start_scores = [&](uint32_t zo) __attribute__((always_inline)) {
    f32x16 s;
#pragma unroll
    for (int gq = 0; gq < 4; gq++) {
      const f32x4 zz = lds_load<f32x4>(zlane + zo + 32 * gq);
#pragma unroll
      for (int u = 0; u < 4; u++) s[4 * gq + u] = zz[u];
    }
    return s;
  };
  auto scores = [&](f32x16& s, uint32_t so) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ks++) s = mfma32(lds_load<bf16x8>(kfrag[ks] + so), qreg[ks], s);
  };
  // Weights of one unit from its scores, and the statistics.  The reference maximum m_run of a row moves only when a
  // weight would get large: the exponentials are formed with the old one and summed, and only if a lane's sum shows a
  // weight that could exceed 2^8 is the unit's maximum looked for, O and l rescaled and the unit's weights formed
  // again.  Same softmax; no maximum in the common case.  The first 64 keys always go that way: the largest weight of a
  // row is then mostly 1, which bf16 holds exactly (rows of a few hundred keys: error of O 2.01e-3 -> 1.97e-3).
  auto exponentials = [&](const f32x16& s, bf16x8 (&pb)[2]) __attribute__((always_inline)) {
    float l0 = 0.f, l1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const float pv = fast_exp2(weight_exponent(s[v], c2, m_run));
      if (v & 1) l1 += pv; else l0 += pv;
      pb[v >> 3][v & 7] = (__bf16)pv;
    }
    return l0 + l1;
  };
  auto take_sum = [&](const f32x16& s, bf16x8 (&pb)[2], float sum) __attribute__((always_inline)) {
    if (__builtin_expect(__any(__builtin_bit_cast(uint32_t, sum) > limit), 0)) {
      float mx = fmaxf(s[0], s[1]);
#pragma unroll
      for (int v = 2; v < 16; v++) mx = fmaxf(mx, s[v]);
      mx = reference_of(half_swap_max(mx), c2);
      const bool grow = mx > m_run;
      const float alpha = grow ? fast_exp2(m_run - mx) : 1.f;  // (nothing kept so far: O and l are 0)
      m_run = grow ? mx : m_run;
      lsum *= alpha;
#pragma unroll
      for (int cb = 0; cb < CB; cb++)
#pragma unroll
        for (int v = 0; v < 16; v++) oacc[cb][v] *= alpha;
      sum = exponentials(s, pb);
    }
    lsum += sum;
  };
  auto value_frag = [&](int i, uint32_t so) __attribute__((always_inline)) {  // A operand of the i-th product of O^T += V^T P^T
    const int c = i / CB, cb = i % CB;
    const s16x4 lo = lds_read_tr_at(vfrag[cb][0] + so + 2 * 16 * c * D);
    const s16x4 hi = lds_read_tr_at(vfrag[cb][1] + so + 2 * 16 * c * D);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // O^T += V^T P^T of one unit
  auto accumulate = [&](const bf16x8 (&pb)[2], uint32_t so) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * CB; i++) oacc[i % CB] = mfma32(value_frag(i, so), pb[i / CB], oacc[i % CB]);
  };
  constexpr uint32_t UB = 2 * 32 * D;  // bytes of one unit in a ring

  int t = 0;
  wait_vmcnt<0>();
  lds_barrier();
  // ---- tiles, software-pipelined: the step of unit i holds the products S(i + 1) and O += V P(i - 1) and the
  // exponentials of unit i, which depend on none of them, so that the matrix pipe has work while the wave issues the
  // element-wise instructions.  The order is fixed where one or two waves share a SIMD: a product, the LDS read of the
  // fragment LEAD products ahead, and a share of the element-wise work.
  bf16x8 pn0[2];  // weights of the unit before
  pn0[0] = pn0[1] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  f32x16 sc = start_scores(4 * 64 * shift);
  scores(sc, shift * (2 * TILE));
  // Partial tiles: a unit is active if some key of it is, on any of this wave's 32 rows.
  const int rfirst = row0 + 32 * wr;
  // full: every key is on all of them, and there is nothing to mask (in a document's first block, and the entering keys seen
  // from later rows).  Asked for at 64 channels, where a mask is a third of a unit's instructions: packed 65536 tokens x 16
  // heads 279 -> 275 us, with scores that rise along the keys 345 -> 333.  (At 128 the pipelined step is longer by more than
  // that with few rows: 7 documents in 10007 x 8 heads 45.3 -> 45.9, 20 in 30000 x 16 217 -> 214.)
  auto active = [&](int tt, int st, int u, bool* full = nullptr) __attribute__((always_inline)) {  // unit u of tile tt, in ring stage st
    const int jl = ids_ring[tt % (2 * NS)][unit0 + 32 * u + n], el = e_ring[st][unit0 + 32 * u + n];
    if (full) *full = __all((jl <= rfirst) & (el > rfirst + 31));
    return (bool)__any((jl <= rfirst + 31) & (el > rfirst));  // (an empty entry has el = 0)
  };
  bool act0 = true, act1 = true;  // the unit before, this unit is active
  constexpr int NM = KS + 2 * CB;  // products of a step: KS of the next unit's scores, then 2 CB of the previous unit's output
  // (64 channels: four waves share a SIMD and overlap by themselves; their 128 registers do not hold fragments read
  // ahead, nor the masks of a pipelined partial step: there the order is the compiler's and partial units run one by one)
  constexpr bool FIXED = D != 64 || PARTS > 1;
  constexpr int LEAD = D == 256 ? 6 : D == 128 ? 4 : FIXED ? 2 : 0;
  auto tile = [&](auto stc, auto maskedc) __attribute__((always_inline)) {
    constexpr int ST = decltype(stc)::value;  // (t + shift) % NS
    constexpr bool MASKED = decltype(maskedc)::value;
    if (t > 0) {
      wait_tile();
      lds_barrier();
    }
    issue_small(t);
    static_for<UT>([&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      constexpr int ss = u + 1 < UT ? ST : (ST + 1) % NS, su = u + 1 < UT ? u + 1 : 0;
      constexpr int vs = u > 0 ? ST : (ST + NS - 1) % NS, vu = u > 0 ? u - 1 : UT - 1;
      constexpr uint32_t ko = ss * (2 * TILE) + su * UB, vo = vs * (2 * TILE) + vu * UB;
      int idv[WL];
      bool prev = true, cur = true, next = true;
      if constexpr (MASKED) {
        // (A list is three runs: entering keys that stay, other entering keys, each by first active row, then expiring
        // ones by last.)  The step of three inactive units is skipped.  At the start of a run of active ones there is no output product: a weight of zero
        // must not meet the infinite value of a key that no row of the wave keeps.  (fwd, us, with those products ->
        // without: 16 documents of 4096 x 4 heads, window 256, scores that rise along the keys 138 -> 123; random
        // scores: unchanged.)
        prev = act0, cur = act1, next = active(u + 1 < UT ? t : t + 1, ss, su);
        act0 = cur;
        act1 = next;
        if (prev | cur) {  // pairs outside [j, e_j) get no weight
          const uint32_t js = jlane + 4 * ((t % (2 * NS)) * 64 + 32 * u);
#pragma unroll
          for (int gq = 0; gq < 4; gq++) {
            const i32x4 jj = lds_load<i32x4>(js + 32 * gq);
            const i32x4 ee = lds_load<i32x4>(elane + 4 * (ST * 64 + 32 * u) + 32 * gq);
#pragma unroll
            for (int v = 0; v < 4; v++) sc[4 * gq + v] = ((qi >= jj[v]) & (qi < ee[v])) ? sc[4 * gq + v] : -INFINITY;
          }
        }
      }
      f32x16 sn;
      bf16x8 pn[2];
      float sum = 0.f;
      auto step = [&]() __attribute__((always_inline)) {
        sn = start_scores(4 * (ss * 64 + 32 * su));
        bf16x8 fr[LEAD + 1];
        float pv[16], l0 = 0.f, l1 = 0.f;
        auto frag = [&](auto mc) __attribute__((always_inline)) {
          constexpr int m = decltype(mc)::value;
          if constexpr (m < KS) fr[m % (LEAD + 1)] = lds_load<bf16x8>(kfrag[m] + ko);
          else if constexpr (m < NM) fr[m % (LEAD + 1)] = value_frag(m - KS, vo);
        };
        static_for<LEAD>(frag);
        if constexpr (FIXED) __builtin_amdgcn_sched_barrier(0);
        static_for<NM>([&](auto mc) __attribute__((always_inline)) {
          constexpr int m = decltype(mc)::value;
          if constexpr (u == 0 && m == 0) row_ids(t + 3, idv);
          if constexpr (u == UT - 1 && m == NM / 2) row_ids(t + 2, idv);
          frag(std::integral_constant<int, m + LEAD>{});
          if constexpr (m < KS) sn = mfma32(fr[m % (LEAD + 1)], qreg[m], sn);
          else oacc[(m - KS) % CB] = mfma32(fr[m % (LEAD + 1)], pn0[(m - KS) / CB], oacc[(m - KS) % CB]);
          // element-wise work of unit i: the exponentials of some scores, sum and rounding of those before
          constexpr int e0 = m * 16 / (NM - 2) < 16 ? m * 16 / (NM - 2) : 16;
          constexpr int e1 = (m + 1) * 16 / (NM - 2) < 16 ? (m + 1) * 16 / (NM - 2) : 16;
          constexpr int f0 = m > 0 ? (m - 1) * 16 / (NM - 2) : 0;
#pragma unroll
          for (int v = e0; v < e1; v++) pv[v] = fast_exp2(weight_exponent(sc[v], c2, m_run));
#pragma unroll
          for (int v = f0; v < e0; v++) {
            if (v & 1) l1 += pv[v]; else l0 += pv[v];
            pn[v >> 3][v & 7] = (__bf16)pv[v];
          }
          if constexpr (u == 0 && m == NM / 2 - 2) copy_rows(Kg, ldsK, (ST + 3) % NS, idv);
          if constexpr (u == UT - 1 && m == NM - 2) copy_rows(Vg, ldsV, (ST + 2) % NS, idv);
          if constexpr (FIXED) __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (FIXED) {
          settle(pn[0]);
          settle(pn[1]);
        }
        sum = l0 + l1;
      };
      if (!MASKED || prev) {
        step();
      } else {
        if constexpr (u == 0) {
          row_ids(t + 3, idv);
          copy_rows(Kg, ldsK, (ST + 3) % NS, idv);
        }
        if constexpr (u == UT - 1) {
          row_ids(t + 2, idv);
          copy_rows(Vg, ldsV, (ST + 2) % NS, idv);
        }
        sn = sc;  // (what no active unit needs keeps its value)
        pn[0] = pn0[0];
        pn[1] = pn0[1];
        if (next) {
          sn = start_scores(4 * (ss * 64 + 32 * su));
          scores(sn, ko);
        }
        if (cur) sum = exponentials(sc, pn);
      }
      take_sum(sc, pn, sum);
      sc = sn;
      pn0[0] = pn[0];
      pn0[1] = pn[1];
    });
    t++;
    limit = t * UT >= 2 ? SUM_LIMIT : 0u;
  };
  // (Ring stages are shifted so that the last clean tile takes the last stage and the first partial one stage 0: one
  // way in and one way out of each loop, and no register moves at their ends.)
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  constexpr std::integral_constant<int, 2> s2{};
  constexpr std::integral_constant<int, 3> s3{};
  for (int base = -shift; base < nc; base += NS) {
    if (base >= 0) tile(s0, std::false_type{});
    if (base + 1 >= 0) tile(s1, std::false_type{});
    if (base + 2 >= 0) tile(s2, std::false_type{});
    tile(s3, std::false_type{});
  }
  if constexpr (!FIXED) {
    if (nc > 0) accumulate(pn0, (NS - 1) * (2 * TILE) + (UT - 1) * UB);
    for (; t < nt; t++) {
      if (t > 0) {
        wait_tile();
        lds_barrier();
      }
      issue_small(t);
      issue_rows(Kg, ldsK, t + 3);
      issue_rows(Vg, ldsV, t + 2);
      const int st = (t + shift) % NS, ist = t % (2 * NS);
#pragma unroll 1
      for (int u = 0; u < UT; u++) {
        bool full;
        if (!active(t, st, u, &full)) continue;
        const uint32_t zo = 4 * (st * 64 + 32 * u), so = st * (2 * TILE) + u * UB;
        f32x16 s = start_scores(zo);
        const uint32_t js = jlane + 4 * (ist * 64 + 32 * u);
        if (!full) {
#pragma unroll
          for (int gq = 0; gq < 4; gq++) {
            const i32x4 jj = lds_load<i32x4>(js + 32 * gq);
            const i32x4 ee = lds_load<i32x4>(elane + zo + 32 * gq);
#pragma unroll
            for (int v = 0; v < 4; v++) s[4 * gq + v] = ((qi >= jj[v]) & (qi < ee[v])) ? s[4 * gq + v] : -INFINITY;
          }
        }
        scores(s, so);
        bf16x8 pb[2];
        const float sum = exponentials(s, pb);
        take_sum(s, pb, sum);
        accumulate(pb, so);
      }
      limit = (t + 1) * UT >= 2 ? SUM_LIMIT : 0u;
    }
  } else {
    act1 = active(nc, 0, 0);  // (its ids and scalars are there: tile nc - 1 waited for those of one tile more)
    for (int base = nc; base < nt; base += NS) {
      tile(s0, std::true_type{});
      if (base + 1 < nt) tile(s1, std::true_type{});
      if (base + 2 < nt) tile(s2, std::true_type{});
      if (base + 3 < nt) tile(s3, std::true_type{});
    }
    static_assert(NS == 4, "the loops are unrolled over the ring stages");
    if (act0) accumulate(pn0, ((nt + shift + NS - 1) % NS) * (2 * TILE) + (UT - 1) * UB);
  }

  // epilogue: drain the (dummy) copies still in flight, normalise, stage O through LDS for
  // coalesced rows, write LSE
  wait_vmcnt<0>();
  lds_barrier();
  if constexpr (PARTS > 1) {
    // (a part that kept nothing has l = 0, O = 0 and the lowest reference)
    static_assert(PARTS == 2 && NS * TILE * 2 >= RW * D * 128 && RW <= NS, "the second part's O takes the K ring");
    f32x4* o2 = reinterpret_cast<f32x4*>(ringK) + wr * (4 * CB * 64) + l;
    float *m2 = &z_ring[wr][l], *l2 = reinterpret_cast<float*>(&e_ring[wr][l]);
    if (part == 1) {
#pragma unroll
      for (int cb = 0; cb < CB; cb++)
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
          f32x4 x;
#pragma unroll
          for (int u = 0; u < 4; u++) x[u] = oacc[cb][4 * gq + u];
          o2[(4 * cb + gq) * 64] = x;
        }
      *m2 = m_run;
      *l2 = lsum;
    }
    lds_barrier();
    if (part == 0) {
      const float mo = *m2, m = fmaxf(m_run, mo), f0 = fast_exp2(m_run - m), f1 = fast_exp2(mo - m);
      m_run = m;
      lsum = lsum * f0 + *l2 * f1;
#pragma unroll
      for (int cb = 0; cb < CB; cb++)
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
          const f32x4 x = o2[(4 * cb + gq) * 64];
#pragma unroll
          for (int u = 0; u < 4; u++) oacc[cb][4 * gq + u] = oacc[cb][4 * gq + u] * f0 + x[u] * f1;
        }
    }
  }
  uint16_t* Os = PARTS > 1 ? ringV : ringK;  // [RW * 32][D] with the tile swizzle
  static_assert(NS * KT >= RW * 32, "O staging aliases a ring");
  if (part == 0) {
    const float ltot = half_swap_sum(lsum);
    const float inv = 1.f / ltot;
    if (hh == 0 && qi < row1) p.LSE[(size_t)h * p.T + qi] = (m_run + __builtin_amdgcn_logf(ltot)) * LN2;
#pragma unroll
    for (int cb = 0; cb < CB; cb++)
#pragma unroll
      for (int gq = 0; gq < 4; gq++) {
        bf16x4 o4;
#pragma unroll
        for (int u = 0; u < 4; u++) o4[u] = (__bf16)(oacc[cb][4 * gq + u] * inv);
        *reinterpret_cast<bf16x4*>(&Os[TL::off(32 * wr + n, 4 * cb + gq) + 4 * hh]) = o4;
      }
  }
  lds_barrier();
#pragma unroll
  for (int it = 0; it < RW * 32 * CPR / NT; it++) {
    const int c = tid + NT * it, r = c / CPR, col = c % CPR;
    if (row0 + r < row1)
      *reinterpret_cast<uint4*>(p.O + ((size_t)(row0 + r) * p.H_q + h) * D + 8 * col) =
          *reinterpret_cast<const uint4*>(&Os[TL::off(r, col)]);
  }
}

int launch_fwd(const Ptrs& p, const void* Q, const void* K, const void* V, const float* z, const int32_t* expiry,
               const int32_t* cu, void* O, float* LSE, hipStream_t st) {
  (void)cu;
  (void)z;
  const dma_shape& s = p.s;
  const PlanLayout& L = p.pl;
  FwdArgs a;
  a.Q = (const uint16_t*)Q; a.K = (const uint16_t*)K; a.V = (const uint16_t*)V; a.O = (uint16_t*)O;
  a.zq = (const float*)(p.plan + L.off_zq); a.LSE = LSE; a.expiry = expiry;
  a.blk = (const int4*)(p.plan + L.off_blk);
  a.slot_tab = (const int32_t*)(p.plan + L.off_slot);
  a.pcnt = (const int32_t*)(p.plan + L.off_pcnt);
  a.plist = (const int32_t*)(p.plan + L.off_plist);
  a.consts = p.plan + L.off_consts;
  a.T = s.T; a.H_q = s.H_q; a.H_kv = s.H_kv; a.k = s.k; a.nblk_cap = L.nblk_cap; a.kpad = L.kpad;
  prof_begin(DMA_STAGE_FWD, st);
  // 64 and 128 channels, all half blocks fit the chip at once: half blocks of eight waves, two of them for the same rows
  // (the call alone, us; whole blocks at 64 channels / this: 256 tokens x 2 heads 10.8 / 8.8, 1000 x 16 27.4 / 18.8,
  // 2048 x 16 27.9 / 20.3, 2 x 1500 x 16, too many, 29.0 / 31.0; half blocks of four waves at 128 channels / this: 512 x 32
  // 19.3 / 17.7, 1019 x 32 29.3 / 26.1, 2048 x 16 of window 1024 40.8 / 33.9, 16000 x 2 41.2 / 35.5; too many: 5 x 800 x 8
  // of window 256 28.3 / 31.7, 1300 x 32 37.3 / 35.6).
  // 128 channels otherwise: whole blocks of eight waves, unless they would leave the chip idle: half blocks with tiles of 32
  // keys, two per compute unit, where whole blocks would keep less than 4/5 of it busy: the last round of blocks is not
  // full, or, in a single round, documents are not much longer than the window, so that blocks differ in length
  // (2048 x 32 53.6 / 51.7, 7 documents in 10007 x 8 window 333 49.4 / 46.9; above the line 8192 x 8 53.2 / 57.7,
  // 2 x 4096 x 16 92 / 98).
  const double blocks = typical_blocks(s), rounds = std::ceil(blocks / CUS);
  const double len = (double)s.T / s.n_docs, window = s.k < len ? s.k : len;
  const double busy = blocks / (CUS * rounds) * (1. - window / (2. * len) / rounds);
  const bool few = 2 * most_blocks(s) <= CUS;
  // 256 channels: half blocks of four waves, one per SIMD with the whole register file (the output
  // accumulators alone are 128 registers per wave).
  if (s.d == 256) fwd_kernel<256, 4, 1><<<xcd_grid(s.H_q, 2l * L.nblk_cap), 256, 0, st>>>(a);
  else if (s.d == 64 && few) fwd_kernel<64, 8, 1, 2><<<xcd_grid(s.H_q, 2l * L.nblk_cap), 512, 0, st>>>(a);
  else if (s.d == 64) fwd_kernel<64, 8, 2><<<xcd_grid(s.H_q, L.nblk_cap), 512, 0, st>>>(a);
  else if (few) fwd_kernel<128, 8, 1, 2><<<xcd_grid(s.H_q, 2l * L.nblk_cap), 512, 0, st>>>(a);
  else if (busy < 0.8) fwd_kernel<128, 4, 1><<<xcd_grid(s.H_q, 2l * L.nblk_cap), 256, 0, st>>>(a);
  else fwd_kernel<128, 8, 2><<<xcd_grid(s.H_q, L.nblk_cap), 512, 0, st>>>(a);
  prof_end(DMA_STAGE_FWD, st);
  return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
}

}  // namespace dma
