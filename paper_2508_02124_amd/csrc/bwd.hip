// Backward pass (Eq. 7-10; the tile arithmetic of Alg. 2 with D_i = rowsum(dO o O)).
//
// Two kernels share the work so that no accumulator is spread over workgroups at tile granularity:
//
//  * dq_kernel, query-stationary (the forward's structure and copy ring): per block of BQ rows it
//    recomputes S^T and dP^T on the gathered key tiles, forms dS^T = P^T o (dP^T - D) and
//    accumulates dQ^T += K^T dS^T in registers.  It also produces D and LSE * log2(e) for the
//    other kernel.
//
//  * dkv_kernel, key-stationary: a workgroup owns SG slot columns of one head and sweeps query
//    blocks in steps of 32 rows, fed by a ring of asynchronous Q / dO copies.  A slot column always
//    holds one resident key, so its tiles are dense and need no mask; K and V fragments of the
//    resident stay in registers and LDS together with the dK^T, dV^T and dz accumulators.  When the
//    resident of a column changes, the finished key is flushed with a handful of fp32 atomics (dK
//    and dV are shared by the q-heads of a group) and the column is re-armed.  The same kernel, in
//    "partial" mode, handles the keys that expire inside a block or enter it without staying: columns
//    come from the blocks' partial lists, elements are masked with j <= i < e_j, and every column changes at
//    every block of the (short) sweep.
//
// The dS / P blocks are produced in the accumulator layout of S = Q K^T (dkv) or S^T = K Q^T (dq),
// which is exactly the B-operand layout of the products that consume them; the other operand of
// those products is read from row-major LDS tiles with transposing LDS reads.
#include "common.h"
#include <cmath>

namespace dma {

struct BwdArgs {
  const uint16_t *Q, *K, *V, *O, *dO;
  uint16_t* dQ;
  const float *zq, *LSE;  // zq = z / softmax_scale
  float *Dws, *L2ws, *dK32, *dV32, *dz;
  const int32_t* expiry;
  const int4* blk;
  const int32_t* slot_tab;
  const int32_t* pcnt;
  const int32_t* pent;
  const int32_t* plist;
  const char* consts;  // [0,256) zeros; +256: float -inf; +260: int 0; +264: int -1; +268: float +inf; +272: softmax scale, scale * log2(e)
  int T, H_q, H_kv, k, nblk_cap, kpad, causal;
  int seg;       // query blocks swept by one clean-mode work item of dkv_kernel
  int seg_part;  // ... by one partial-mode work item
  size_t zero_n4;  // float4 elements from dK32 to the end of dV32 (cleared by dq_kernel)
  size_t dz_n;     // elements of dz (cleared by dq_kernel)
  float *dW, *dA;  // gradients of the score parameters (cleared by dq_kernel), or no elements
  int dW_n, dA_n;
  unsigned grid_dq;  // workgroups of the dq_kernel launch
  unsigned grid_clean;  // workgroups of the slot sweeps in the dkv_kernel launch (a multiple of 8)
};

// ------------------------------------------------------------------ dQ (and D, LSE * log2 e)
// NW waves per workgroup: 8 (a whole 256-row block) or 4 (half a block); UT 32-key units per tile, as in the forward
// kernel.  Software-pipelined like it: the step of unit i holds the products dP(i), S(i + 1) and dQ += K dS(i), and its
// element-wise work runs under the products that do not need it: P(i) under dP(i), dS(i) under S(i + 1).  What bounds it
// is what bounds the forward: the power limit's clock, then the matrix pipe.  Against the whole chain of a tile at a time
// (us): 16384 tokens x 32 heads 872 -> 798; 16 heads of 256 channels, one wave per SIMD, 1172 -> 890; 2 x 4096 x 16
// heads 141 -> 126; packed 65536 x 16 heads of 64 channels, not pipelined (three waves per SIMD; pipelined 426 there),
// but with its rows addressed by immediates and dP started at -D: 425 -> 402.
// PARTS: waves that share the same 32 rows, each with its own units of every tile, as in the forward kernel; their dQ are
// added at the end.  Whole backward, one / two of them at 128 channels (us): 1019 tokens x 32 heads 95.3 / 92.4, 2048 x 16
// of window 1024 138 / 132, 300 x 32 47 / 47 (at 64 channels, three waves per SIMD without: 31.0 / 31.5, 69.3 / 70.3).
template <int D, int NW, int UT, int PARTS = 1>
__global__ __launch_bounds__(NW * 64, D == 64 ? 3 : 1) void dq_kernel(BwdArgs p) {
  using TL = TileLayout<D>;
  constexpr int KT = 32 * UT * PARTS;
  constexpr int KS = D / 16, CB = D / 32, CPR = D / 8, RPL = 64 / CPR, WL = KT / RPL / NW;
  constexpr bool PIPED = D != 64;
  constexpr int NS = PIPED ? 4 : 2, AHEAD = NS - 1;  // ring stages; tiles between a copy's request and its use
  constexpr int TILE = KT * D, NT = NW * 64, RW = NW / PARTS, HALVES = 8 / RW;
  __shared__ __align__(16) uint16_t ring[2 * NS * TILE];  // K stages, then V stages
  __shared__ __align__(16) int ids_ring[2 * NS][64];  // (rows of 64: what one wave-wide copy writes)
  __shared__ __align__(16) float z_ring[NS][64];
  __shared__ __align__(16) int e_ring[NS][64];

  // This launch also clears what the key-stationary launches behind it accumulate into with atomics
  // (the fp32 dK / dV buffers, dz, and dW and dA where they follow): every workgroup, also one without a block, takes its share of
  // the stores; this kernel is bound by the matrix cores, so they cost no time here.
  {
    const size_t nth = (size_t)p.grid_dq * NT, gid = (size_t)wg_id() * NT + thread_id();
    float4* acc4 = reinterpret_cast<float4*>(p.dK32);
    for (size_t i = gid; i < p.zero_n4; i += nth) acc4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (size_t i = gid; i < p.dz_n; i += nth) p.dz[i] = 0.f;
    for (size_t i = gid; i < (size_t)p.dW_n; i += nth) p.dW[i] = 0.f;
    for (size_t i = gid; i < (size_t)p.dA_n; i += nth) p.dA[i] = 0.f;
  }
  int h, item;
  if (!xcd_map(wg_id(), p.H_q, p.nblk_cap * HALVES, h, item)) return;
  const int bi = p.nblk_cap - 1 - item / HALVES;  // long blocks first
  const int4 info = p.blk[bi];
  const int np_keys = p.pcnt[(size_t)h * p.nblk_cap + bi];
  const float scale = *reinterpret_cast<const float*>(p.consts + PLAN_SCALE_OFF);
  const float c2 = *reinterpret_cast<const float*>(p.consts + PLAN_C2_OFF);
  if (info.x < 0) return;
  const int blk_row0 = info.y, row1 = info.z, doc0 = info.w;
  const int row0 = blk_row0 + (item % HALVES) * (RW * 32);  // first row of this workgroup's part of the block
  if (row0 >= row1) return;
  const int g = h / (p.H_q / p.H_kv);
  const int tid = thread_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, n = l & 31, hh = l >> 5;
  const int wr = w % RW, part = w / RW;
  const int ncol = min(p.k, blk_row0 - doc0);
  const int nc = (ncol + KT - 1) / KT;
  const int nt = nc + (np_keys + KT - 1) / KT;
  const int shift = (NS - nc % NS) % NS;  // ring stage of tile 0: tile t takes stage (t + shift) % NS
  const int32_t* slot_row = p.slot_tab + ((size_t)h * p.nblk_cap + bi) * p.kpad;
  const int32_t* plist_row = p.plist + ((size_t)h * p.nblk_cap + bi) * MAXPART;
  const float* zqh = p.zq + (size_t)h * p.T;
  const int32_t* eh = p.expiry + (size_t)h * p.T;
  const float* c_ninf = reinterpret_cast<const float*>(p.consts + 256);
  const int32_t* c_zero = reinterpret_cast<const int32_t*>(p.consts + 260);
  const int32_t* c_m1 = reinterpret_cast<const int32_t*>(p.consts + 264);

  // gathered rows: wave-uniform base of the kv-head plus a 32-bit byte offset (id * row pitch + the
  // lane's chunk); an empty slot (id < 0) copies row 0, which its score of -inf keeps out of every sum
  constexpr uint32_t VOFF = 2 * NS * TILE;  // bytes from a K row to the V row of the same key
  const void* Kg = uniform_ptr(p.K + (size_t)g * D);
  const void* Vg = uniform_ptr(p.V + (size_t)g * D);
  const uint32_t row_pitch = (uint32_t)p.H_kv * D * 2;
  uint32_t lane_chunk[WL];
  int lane_row[WL];
#pragma unroll
  for (int j = 0; j < WL; j++) {
    lane_row[j] = (w * WL + j) * RPL + l / CPR;
    lane_chunk[j] = (uint32_t)(((l % CPR) ^ TL::swz(lane_row[j])) * 16);
  }
  const uint32_t ldsK = lds_addr(ring) + (uint32_t)(w * WL * RPL * D * 2);
  const uint32_t ldsV = ldsK + VOFF;
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
  auto row_ids = [&](int tt, int (&idv)[WL]) __attribute__((always_inline)) {
    const int* idr = ids_ring[tt % (2 * NS)];
#pragma unroll
    for (int j = 0; j < WL; j++) idv[j] = idr[lane_row[j]];
  };
  auto copy_rows = [&](int stage, const int (&idv)[WL]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WL; j++) {
      const uint32_t off = mul24((uint32_t)max(idv[j], 0), row_pitch) + lane_chunk[j];
      const uint32_t dst = (uint32_t)((stage * TILE + j * RPL * D) * 2);
      dma16u(Kg, off, ldsK + dst);
      dma16u(Vg, off, ldsV + dst);
    }
  };
  auto issue_scalars = [&](int tt) {
    if (w == 1) {
      const int idl = ids_ring[tt % (2 * NS)][l];
      dma4(idl >= 0 ? zqh + idl : c_ninf, &z_ring[(tt + shift) % NS][0]);
      dma4(idl >= 0 ? (const void*)(eh + idl) : (const void*)c_zero, &e_ring[(tt + shift) % NS][0]);
    }
  };
  // Iteration t of the tile loops requests the ids of tile t + AHEAD + 2 and the rows and scalars of tile t + AHEAD.  It
  // starts when everything requested before iteration t - 1 has landed (tiles up to t + 1), or, without pipelining,
  // everything (tile t).
  auto wait_tile = [&]() {
    if (!PIPED) wait_vmcnt<0>();
    else if (w == 0) wait_vmcnt<2 * WL + 1>();
    else if (w == 1) wait_vmcnt<2 * WL + 2>();
    else wait_vmcnt<2 * WL>();
  };

  for (int tt = 0; tt < AHEAD + 2; tt++) issue_ids(tt);
  wait_vmcnt<0>();
  lds_barrier();
  for (int i = 0; i < AHEAD; i++) {
    int idv[WL];
    row_ids(i, idv);
    copy_rows((i + shift) % NS, idv);
    issue_scalars(i);
  }

  const int qi = row0 + 32 * wr + n;
  const bool qvalid = qi < row1;
  bf16x8 qreg[KS], doreg[KS];
  float Dsum = 0.f;
  {
    const size_t off = ((size_t)qi * p.H_q + h) * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      uint4 rq = make_uint4(0, 0, 0, 0), rd = rq, ro = rq;
      if (qvalid) {
        rq = *reinterpret_cast<const uint4*>(p.Q + off + 16 * ks);
        rd = *reinterpret_cast<const uint4*>(p.dO + off + 16 * ks);
        ro = *reinterpret_cast<const uint4*>(p.O + off + 16 * ks);
      }
      qreg[ks] = __builtin_bit_cast(bf16x8, rq);
      doreg[ks] = __builtin_bit_cast(bf16x8, rd);
      const bf16x8 ov = __builtin_bit_cast(bf16x8, ro);
#pragma unroll
      for (int e = 0; e < 8; e++) Dsum = fmaf((float)doreg[ks][e], (float)ov[e], Dsum);
    }
  }
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    settle(qreg[ks]);
    settle(doreg[ks]);
  }
  Dsum = half_swap_sum(Dsum);
  float lse2 = qvalid ? p.LSE[(size_t)h * p.T + qi] * LOG2E : INFINITY;
  // A row whose weights are all 0 (LSE = -inf: it keeps nothing but keys that are masked beyond the range of the
  // exponents) has P = 0 here too, not infinities that would reach the dV of its keys.
  if (lse2 == -INFINITY) lse2 = INFINITY;
  settle(lse2);
  if (qvalid && hh == 0 && part == 0) {
    p.Dws[(size_t)h * p.T + qi] = -Dsum;  // (negated: the key-stationary kernel starts its dP accumulators at -D_i)
    p.L2ws[(size_t)h * p.T + qi] = lse2;
  }
  // fragment addresses with the ring bases folded in: inside the stage-unrolled main loop every LDS
  // read is one of these registers plus an immediate; the part's first unit is folded in too
  const int unit0 = 32 * UT * part;
  FragOffsets<D> fo;
  fo.init(l);
  uint32_t kfrag[KS], ktr[CB][2];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    kfrag[ks] = lds_addr(ring) + 2 * (fo.row(ks) + unit0 * D);
    settle(kfrag[ks]);
  }
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int q = 0; q < 2; q++) {
      ktr[cb][q] = lds_addr(ring) + 2 * (fo.tr(cb, q) + unit0 * D);
      settle(ktr[cb][q]);
    }
  uint32_t zlane = lds_addr(&z_ring[0][unit0 + 4 * hh]);
  const uint32_t jlane = lds_addr(&ids_ring[0][unit0 + 4 * hh]), elane = lds_addr(&e_ring[0][unit0 + 4 * hh]);
  settle(zlane);
  f32x16 dqacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int v = 0; v < 16; v++) dqacc[cb][v] = 0.f;

  // S^T of a unit starts at z / scale, so that scale * acc is the biased score; its dP^T starts at -D_i
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
  f32x16 dpacc;
  auto start_dp = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; v++) dpacc[v] = -Dsum;
  };
  constexpr uint32_t UB = 2 * 32 * D;  // bytes of one unit in a ring
  constexpr int NM = 2 * KS + 2 * CB;  // products of a step: dP(i), S(i + 1), dQ(i)
  constexpr int LEAD = D == 256 ? 5 : D == 128 ? 3 : 1;  // fragments read ahead of their product
  static_assert(NM % (LEAD + 1) == 0, "the fragments read ahead for the next step keep their registers");
  bf16x8 fr[LEAD + 1];
  // A operand of product m of the step of unit (stage vs, u), whose next unit is (stage ss, su): byte offsets vo, ko
  auto frag = [&](auto mc, uint32_t vo, uint32_t ko) __attribute__((always_inline)) {
    constexpr int m = decltype(mc)::value;
    if constexpr (m < KS) {
      // (VOFF is beyond an instruction's offset at 128 channels and more: one addition, formed where it is used -- eight
      // more address registers would spill)
      uint32_t a = kfrag[m];
      asm volatile("v_add_u32 %0, %1, %2" : "=v"(a) : "n"(VOFF), "v"(kfrag[m]));
      fr[m % (LEAD + 1)] = lds_load<bf16x8>(a + vo);
    } else if constexpr (m < 2 * KS) {
      fr[m % (LEAD + 1)] = lds_load<bf16x8>(kfrag[m - KS] + ko);
    } else {
      constexpr int c = (m - 2 * KS) / CB, cb = (m - 2 * KS) % CB;
      const s16x4 lo = lds_read_tr_at(ktr[cb][0] + vo + 2 * 16 * c * D);
      const s16x4 hi = lds_read_tr_at(ktr[cb][1] + vo + 2 * 16 * c * D);
      fr[m % (LEAD + 1)] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  int t = 0;
  wait_vmcnt<0>();  // the copies of the first tiles, and the ordinary loads and stores above: from here on only copies are in flight
  lds_barrier();
  f32x16 sc;
  if constexpr (PIPED) {
    sc = start_scores(4 * 64 * shift);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sc = mfma32(lds_load<bf16x8>(kfrag[ks] + shift * (2 * TILE)), qreg[ks], sc);
    start_dp();
    static_for<LEAD>([&](auto mc) __attribute__((always_inline)) { frag(mc, shift * (2 * TILE), 0); });
  }
  // Partial tiles: a unit is active if some key of it is, on any of this wave's 32 rows, and full if every key is on all of
  // them (nothing to mask).  Backward, us, scores that rise along the keys: packed 65536 x 16 heads of 64 channels 1558 ->
  // 1545, 20 documents in 30000 x 16 of 128 1048 -> 1038; random scores 1026 -> 1024, 846 -> 843.
  const int rfirst = row0 + 32 * wr;
  auto active = [&](int tt, int st, int u, bool& full) __attribute__((always_inline)) {  // unit u of tile tt, in ring stage st
    const int jl = ids_ring[tt % (2 * NS)][unit0 + 32 * u + n], el = e_ring[st][unit0 + 32 * u + n];
    full = __all((jl <= rfirst) & (el > rfirst + 31));
    return (bool)__any((jl <= rfirst + 31) & (el > rfirst));  // (an empty entry has el = 0)
  };
  bool act0 = true, full0 = false;  // this unit is active, is full
  auto tile = [&](auto stc, auto maskedc) __attribute__((always_inline)) {
    constexpr int ST = decltype(stc)::value;  // (t + shift) % NS
    constexpr bool MASKED = decltype(maskedc)::value;
    if (t > 0) {
      wait_tile();
      lds_barrier();
    }
    issue_ids(t + AHEAD + 2);
    issue_scalars(t + AHEAD);
    static_for<UT>([&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      constexpr int ss = u + 1 < UT ? ST : (ST + 1) % NS, su = u + 1 < UT ? u + 1 : 0;
      constexpr uint32_t ko = ss * (2 * TILE) + su * UB, vo = ST * (2 * TILE) + u * UB;
      int idv[WL];
      bool masked = false;
      auto mask = [&]() __attribute__((always_inline)) {
        // pairs outside [j, e_j) get P = 0 and dS = 0 exactly
        const uint32_t js = jlane + 4 * ((t % (2 * NS)) * 64 + 32 * u);
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
          const i32x4 jj = lds_load<i32x4>(js + 32 * gq);
          const i32x4 ee = lds_load<i32x4>(elane + 4 * (ST * 64 + 32 * u) + 32 * gq);
#pragma unroll
          for (int v = 0; v < 4; v++) sc[4 * gq + v] = ((qi >= jj[v]) & (qi < ee[v])) ? sc[4 * gq + v] : -INFINITY;
        }
      };
      if constexpr (MASKED) {
        // Skip the step of an inactive unit; the scores of the next one, if that is active, are all there is to do (a P of
        // zero must not meet an infinite value or key)
        bool full = full0;
        const bool act1 = PIPED ? active(u + 1 < UT ? t : t + 1, ss, su, full0) : active(t, ST, u, full);
        const bool run = PIPED ? act0 : act1;
        act0 = act1;
        masked = !full;
        if (!run) {
          if constexpr (PIPED) {
            if (act1) {
              sc = start_scores(4 * (ss * 64 + 32 * su));
#pragma unroll
              for (int ks = 0; ks < KS; ks++) sc = mfma32(lds_load<bf16x8>(kfrag[ks] + ko), qreg[ks], sc);
            }
            static_for<LEAD>([&](auto mc) __attribute__((always_inline)) { frag(mc, ko, 0); });
          }
          if constexpr (u == 0) {
            row_ids(t + AHEAD, idv);
            copy_rows((ST + AHEAD) % NS, idv);
          }
          return;
        }
        if constexpr (PIPED)
          if (masked) mask();
      }
      bf16x8 dsb[2];
      if constexpr (!PIPED) {
        if constexpr (u == 0) row_ids(t + AHEAD, idv);
        sc = start_scores(4 * (ST * 64 + 32 * u));
        start_dp();
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
          sc = mfma32(lds_load<bf16x8>(kfrag[ks] + vo), qreg[ks], sc);
          dpacc = mfma32(lds_load<bf16x8>(kfrag[ks] + (VOFF + vo)), doreg[ks], dpacc);
        }
        if constexpr (u == 0) copy_rows((ST + AHEAD) % NS, idv);
        if constexpr (MASKED)
          if (masked) mask();
#pragma unroll
        for (int v = 0; v < 16; v++) dsb[v >> 3][v & 7] = (__bf16)(fast_exp2(fmaf(sc[v], c2, -lse2)) * dpacc[v]);
        static_for<2 * CB>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value;
          frag(std::integral_constant<int, 2 * KS + i>{}, vo, 0);
          dqacc[i % CB] = mfma32(fr[i % (LEAD + 1)], dsb[i / CB], dqacc[i % CB]);
        });
        return;
      }
      f32x16 sn;
      float pv[16];
      static_for<NM>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        if constexpr (u == 0 && m == 0) row_ids(t + AHEAD, idv);
        if constexpr (m == KS / 2) sn = start_scores(4 * (ss * 64 + 32 * su));
        if constexpr (m + LEAD < NM) frag(std::integral_constant<int, m + LEAD>{}, vo, ko);
        else frag(std::integral_constant<int, m + LEAD - NM>{}, ko, 0);
        if constexpr (m < KS) dpacc = mfma32(fr[m % (LEAD + 1)], doreg[m], dpacc);
        else if constexpr (m < 2 * KS) sn = mfma32(fr[m % (LEAD + 1)], qreg[m - KS], sn);
        else dqacc[(m - 2 * KS) % CB] = mfma32(fr[m % (LEAD + 1)], dsb[(m - 2 * KS) / CB], dqacc[(m - 2 * KS) % CB]);
        if constexpr (m < KS) {  // P(i)
#pragma unroll
          for (int v = m * 16 / KS; v < (m + 1) * 16 / KS; v++) pv[v] = fast_exp2(fmaf(sc[v], c2, -lse2));
        }
        // dS(i): its first half before the first products with it, the second under those
        constexpr int f0 = KS + KS / 4, fn = KS - KS / 4;
        if constexpr (m >= f0 && m < 2 * KS) {
#pragma unroll
          for (int v = (m - f0) * 8 / fn; v < (m + 1 - f0) * 8 / fn; v++) dsb[0][v] = (__bf16)(pv[v] * dpacc[v]);
        }
        if constexpr (m >= 2 * KS && m < 2 * KS + CB) {
#pragma unroll
          for (int v = (m - 2 * KS) * 8 / CB; v < (m + 1 - 2 * KS) * 8 / CB; v++) dsb[1][v] = (__bf16)(pv[8 + v] * dpacc[8 + v]);
        }
        if constexpr (m == NM - 2) start_dp();
        if constexpr (u == 0 && m == KS + 1) copy_rows((ST + AHEAD) % NS, idv);
        __builtin_amdgcn_sched_barrier(0);
      });
      sc = sn;
    });
    t++;
  };
  constexpr std::integral_constant<int, 0> s0{};
  constexpr std::integral_constant<int, 1> s1{};
  for (int base = -shift; base < nc; base += NS) {
    if (base >= 0) tile(s0, std::false_type{});
    if constexpr (NS == 4) {
      if (base + 1 >= 0) tile(s1, std::false_type{});
      if (base + 2 >= 0) tile(std::integral_constant<int, 2 % NS>{}, std::false_type{});
    }
    tile(std::integral_constant<int, NS - 1>{}, std::false_type{});
  }
  if constexpr (PIPED) act0 = active(nc, 0, 0, full0);  // (its ids and scalars are there: tile nc - 1 waited for those of one tile more)
  for (int base = nc; base < nt; base += NS) {
    tile(s0, std::true_type{});
    if (base + 1 < nt) tile(s1, std::true_type{});
    if constexpr (NS == 4) {
      if (base + 2 < nt) tile(std::integral_constant<int, 2 % NS>{}, std::true_type{});
      if (base + 3 < nt) tile(std::integral_constant<int, 3 % NS>{}, std::true_type{});
    }
  }
  static_assert(NS == 4 || NS == 2, "the loops are unrolled over the ring stages");

  wait_vmcnt<0>();
  lds_barrier();
  if constexpr (PARTS > 1) {
    static_assert(PARTS == 2 && NS * TILE * 2 >= RW * D * 128, "the second part's dQ takes the K ring");
    f32x4* dq2 = reinterpret_cast<f32x4*>(ring) + wr * (4 * CB * 64) + l;
    if (part == 1) {
#pragma unroll
      for (int cb = 0; cb < CB; cb++)
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
          f32x4 x;
#pragma unroll
          for (int u = 0; u < 4; u++) x[u] = dqacc[cb][4 * gq + u];
          dq2[(4 * cb + gq) * 64] = x;
        }
    }
    lds_barrier();
    if (part == 0) {
#pragma unroll
      for (int cb = 0; cb < CB; cb++)
#pragma unroll
        for (int gq = 0; gq < 4; gq++) {
          const f32x4 x = dq2[(4 * cb + gq) * 64];
#pragma unroll
          for (int u = 0; u < 4; u++) dqacc[cb][4 * gq + u] += x[u];
        }
    }
  }
  uint16_t* Os = PARTS > 1 ? ring + NS * TILE : ring;  // [RW * 32][D] staging with the tile swizzle
  static_assert(NS * KT >= RW * 32, "dQ staging aliases the K ring, or the V ring");
  if (part == 0)
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int gq = 0; gq < 4; gq++) {
      bf16x4 o4;
#pragma unroll
      for (int u = 0; u < 4; u++) o4[u] = (__bf16)(dqacc[cb][4 * gq + u] * scale);
      *reinterpret_cast<bf16x4*>(&Os[TL::off(32 * wr + n, 4 * cb + gq) + 4 * hh]) = o4;
    }
  lds_barrier();
#pragma unroll
  for (int it = 0; it < RW * 32 * CPR / NT; it++) {
    const int c = tid + NT * it, r = c / CPR, col = c % CPR;
    if (row0 + r < row1)
      *reinterpret_cast<uint4*>(p.dQ + ((size_t)(row0 + r) * p.H_q + h) * D + 8 * col) =
          *reinterpret_cast<const uint4*>(&Os[TL::off(r, col)]);
  }
}

// ------------------------------------------------------------------ dK, dV, dz
constexpr int DKV_NW = SG / 32;  // waves of a key-stationary workgroup
constexpr int MAXSWEEP = 64;     // most query blocks one key-stationary work item sweeps

// Four waves; wave w serves columns 32 w .. + 31 of the workgroup's SG columns and carries a column through
// the whole step:
//   S = Q K^T + z / scale, dP = dO V^T - D, P = exp2(S c2 - LSE2) (masked in partial mode), dV^T += dO^T P,
//   dS = P o dP, dz += colsum(dS), dK^T += Q^T dS.
// Lane (n, hh) owns column 32 w + n; its accumulators hold channels 32cb + 8gq + 4hh + u.
// Two workgroups of 4 waves share a compute unit at 128 channels (three at 64, one at 256) and drift apart in phase, so
// one computes while the other waits.  What bounds it at 128 channels: of 4140 cycles per 32-row step of a wave (2050 are
// the matrix pipe's for its two waves) 2440 are the products and what they wait for, 580 the change of keys at block
// starts, 460 the issue of copies, 450 the barrier, 220 the copies' arrival -- at a clock that the power limit holds at 1.9
// to 2.1 GHz.  At 256 channels, one wave per SIMD at 2.2 to 2.3 GHz, the products' own latencies count: 3600 of 5800 cycles.
// Registers decide the rest: the accumulators take D, so all of the K fragments and some of V's wait in LDS at 128
// channels (two ring stages instead of three make room) and half of K's at 256; small lane-dependent
// values are formed where they are used (fresh_lane).  Slot sweep / partial lists (as launches of their own), us, with the products in the
// compiler's order, the keys' rows through registers and a wait in every pass of a flush -> now: 16384 tokens x 32 heads
// 1160 / 186 -> 1060 / 168; 2 x 4096 x 16 heads 193 / 81 -> 167 / 66; 16 heads of 256 channels 1775 / 278 -> 1290 / 246;
// packed 65536 x 16 heads of 64 channels 371 / 169 -> 363 / 167.
template <int D> struct DkvShape {
  static constexpr int KS = D / 16, CB = D / 32;
  static constexpr int SUB = 32;                       // query rows per pipeline step
  static constexpr int NS = D == 64 ? 4 : D == 128 ? 2 : 3;  // ring stages
  static constexpr int STILE = SUB * D;
  static constexpr int KL = D == 64 ? 0 : 8;           // contraction steps whose K fragments wait in LDS
  static constexpr int VL = D == 128 ? 2 : 0;          // ... and V fragments
  static constexpr int STR = 8, STC = D == 64 ? 64 : 32;  // flush staging: columns, channels
  static constexpr int LDS_ST = STC + 4;               // padded staging row
};
template <int D> struct DkvShared {
  using S = DkvShape<D>;
  __align__(16) uint16_t ringQ[S::NS * S::STILE];
  __align__(16) uint16_t ringdO[S::NS * S::STILE];
  __align__(16) float meta[S::NS][64];   // per stage: [0,32) LSE * log2 e, [32,64) -D
  __align__(16) int idbuf[2][SG];        // column ids of the current / next block
  __align__(16) int4 binfo[MAXSWEEP + 1];  // block table of this work item's sweep
  __align__(16) float stage_all[DKV_NW * S::STR * S::LDS_ST];  // per wave: [STR columns][STC channels] fp32, flush staging
  __align__(16) bf16x8 vlds[S::VL ? DKV_NW * S::VL * 64 : 1];
  __align__(16) bf16x8 klds[S::KL ? DKV_NW * S::KL * 64 : 1];  // [wave][ks][lane]: K fragments of the first KL steps
  int nblocks;
};
template <int D, bool PARTIAL>
__device__ __forceinline__ void dkv_sweep(const BwdArgs& p, const int wg, DkvShared<D>& sm) {
  using TL = TileLayout<D>;
  using S = DkvShape<D>;
  constexpr int KS = S::KS, CB = S::CB, CPR = D / 8, RPL = 64 / CPR;
  constexpr int SUB = S::SUB, NS = S::NS, STILE = S::STILE, KL = S::KL, VL = S::VL, STR = S::STR, STC = S::STC, LDS_ST = S::LDS_ST;
  constexpr int NSUB = BQ / SUB;          // steps per query block
  constexpr int NWL = 2 * (SUB / RPL);    // 16-byte wave copies per step (Q rows, then dO rows)
  auto& ringQ = sm.ringQ;
  auto& ringdO = sm.ringdO;
  auto& meta = sm.meta;
  auto& idbuf = sm.idbuf;
  auto& binfo = sm.binfo;
  auto& stage_all = sm.stage_all;
  auto& vlds = sm.vlds;
  auto& klds = sm.klds;

  const int ngrp = PARTIAL ? MAXPART / SG : p.kpad / SG;
  const int nchunk = (p.nblk_cap + (PARTIAL ? p.seg_part : p.seg) - 1) / (PARTIAL ? p.seg_part : p.seg);
  int h, item;
  if (!xcd_map(wg, p.H_q, ngrp * nchunk, h, item)) return;
  // Clean mode: the groups of a chunk are neighbours.  Partial mode: group-major, because the high
  // groups of most chunks are empty and workgroups go to the shader engines in turn: with the
  // groups as the fast index all the work would land on the engines that get groups 0 and 1.
  const int chunk = PARTIAL ? item % nchunk : item / ngrp, grp = PARTIAL ? item / nchunk : item - chunk * ngrp;
  const int g = h / (p.H_q / p.H_kv);
  const int tid = thread_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, n = l & 31, hh = l >> 5;
  // The lane number for values that are formed where they are used: kept over the loop they would spill.
  auto fresh_lane = [&] {
    int ln = l;
    asm volatile("" : "+v"(ln));
    return ln;
  };
  const float* zqh = p.zq + (size_t)h * p.T;
  const float* Dh = p.Dws + (size_t)h * p.T;
  const float* L2h = p.L2ws + (size_t)h * p.T;
  const float* c_zero_f = reinterpret_cast<const float*>(p.consts + 260);
  const int32_t* c_m1 = reinterpret_cast<const int32_t*>(p.consts + 264);
  const float* c_pinf = reinterpret_cast<const float*>(p.consts + 268);
  const float scale = *reinterpret_cast<const float*>(p.consts + PLAN_SCALE_OFF);
  const float c2 = *reinterpret_cast<const float*>(p.consts + PLAN_C2_OFF);

  const int seg = PARTIAL ? p.seg_part : p.seg;
  const int bi_begin = chunk * seg, bi_end = min(bi_begin + seg, p.nblk_cap);
  // Block table of this sweep, kept in LDS so that the copy-ring loop issues no ordinary loads:
  // {block index, first row, rows | columns of this group << 16, x} of every block of the chunk in which
  // the group has at least one column (clean mode: slots in use at the block's end, x = the document's
  // first row; partial mode: listed keys, x = first list entry).
  int& nblocks_s = sm.nblocks;
  for (int i = tid; i < MAXSWEEP + 1; i += DKV_NW * 64) binfo[i] = make_int4(-1, 0, 0, 0);
  __syncthreads();
  if (w == 0) {
    int cnt = 0;
    for (int base = bi_begin; base < bi_end; base += 64) {
      const int bi = base + l;
      int4 info = make_int4(-1, 0, 0, 0);
      int nc = 0;
      if (bi < bi_end) {
        info = p.blk[bi];
        if (info.x >= 0) {
          int total;
          if (PARTIAL) {
            const int first = p.pent[(size_t)h * p.nblk_cap + bi];  // the slot sweep has the keys before it
            total = p.pcnt[(size_t)h * p.nblk_cap + bi] - first;
            info.w = first;
          } else {
            total = min(p.k, (p.causal ? info.z : info.y) - info.w);
          }
          nc = max(0, min(SG, total - grp * SG));
        }
      }
      const unsigned long long m = __ballot(nc > 0);
      if (nc > 0) binfo[cnt + __popcll(m & ((1ull << l) - 1ull))] = make_int4(bi, info.y, (info.z - info.y) | nc << 16, info.w);
      cnt += __popcll(m);
    }
    if (l == 0) nblocks_s = cnt;
  }
  __syncthreads();
  const int nblocks = nblocks_s;
  if (nblocks == 0) return;
  const int nsteps = nblocks * NSUB;

  // Block cursor: the table entry of one block of the sweep, held in scalar registers and
  // refreshed only when a stream (producer or consumer) enters the next block.  Past the end of
  // the sweep it is a dummy without columns.
  struct Cursor {
    int bi, row0, row1, ncols, x;
  };
  auto load_cursor = [&](int bl) -> Cursor {
    const int4 info = binfo[min(bl, MAXSWEEP)];
    Cursor c;
    c.bi = __builtin_amdgcn_readfirstlane(info.x);
    c.row0 = __builtin_amdgcn_readfirstlane(info.y);
    const int z = __builtin_amdgcn_readfirstlane(info.z);
    c.row1 = c.row0 + (z & 0xffff);
    c.ncols = z >> 16;
    c.x = __builtin_amdgcn_readfirstlane(info.w);
    return c;
  };

  // ---- producer: copies of step v (32 query rows of Q and dO, their LSE/D, and at a block's first
  // step the block's column ids).  Every wave issues the same number of copies for every step.  Rows past the end of the block (or every row of a block without
  // columns) re-read a valid row: their LSE is +inf and their D is 0, so whatever Q / dO they hold
  // contributes exactly 0.
  constexpr int WLW0 = NWL / DKV_NW;   // copies per issuing wave and step: first half Q rows, second half dO rows
  constexpr int NLO = WLW0 / 2;   // distinct row positions among them
  static_assert(WLW0 == 2 * NLO && NLO >= 1, "copy layout of the key-stationary kernel");
  const uint32_t row_stride = (uint32_t)p.H_q * D * 2;  // bytes between consecutive rows of Q / dO
  // Copy u of a wave takes rows (w + 4 u) * RPL + l / CPR.  Where 4 RPL is a multiple of the swizzle's period of
  // 16 rows, its lane offset is that of copy 0 and the rows between them go into the scalar base.
  constexpr int NOFF = NLO == 1 || DKV_NW * RPL % 16 == 0 ? 1 : NLO;
  auto lane_row = [&](int ln, int u) { return (w + DKV_NW * u) * RPL + ln / CPR; };
  auto lane_chunk = [&](int ln, int u) { return (uint32_t)(((ln % CPR) ^ TL::swz(lane_row(ln, u))) * 16); };
  uint32_t lane_off[NOFF];  // byte offset from the step's first row, for a full step
#pragma unroll
  for (int u = 0; u < NOFF; u++) {
    lane_off[u] = (uint32_t)lane_row(l, u) * row_stride + lane_chunk(l, u);
    settle(lane_off[u]);
  }
  const char* Qh = (const char*)uniform_ptr(reinterpret_cast<const char*>(p.Q) + (size_t)h * D * 2);   // row 0 of this head
  const char* dOh = (const char*)uniform_ptr(reinterpret_cast<const char*>(p.dO) + (size_t)h * D * 2);
  Cursor pc = {-1, 0, 0, 0, 0};
  int issue_st = 0;   // ring stage of the next step to issue (steps are issued in order: v mod NS without a division)
  auto issue = [&](int v) {
    const int qs = v % NSUB;
    if (qs == 0) pc = load_cursor(v / NSUB);
    const int st = issue_st;
    issue_st = issue_st + 1 == NS ? 0 : issue_st + 1;
    const int rowb = pc.row0 + SUB * qs;
    const int left = pc.ncols > 0 ? pc.row1 - rowb : 0;   // rows of the block from this step on (wave-uniform)
    uint16_t* dstQ = ringQ + st * STILE;
    uint16_t* dstdO = ringdO + st * STILE;
    if (left >= SUB) {  // a full step: scalar base of the step's first row + the lane's fixed offset
      const uint32_t boff = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)rowb * row_stride));  // (below 4 GiB: checked on the host)
#pragma unroll
      for (int j = 0; j < WLW0; j++) {
        const int u = j % NLO;
        const uint32_t skip = u < NOFF ? 0u : (uint32_t)(DKV_NW * u * RPL) * row_stride;
        dma16s((j >= NLO ? dOh : Qh) + (boff + skip), lane_off[u < NOFF ? u : 0],
               (j >= NLO ? dstdO : dstQ) + (w + DKV_NW * u) * RPL * D);
      }
      if (w == 0) {
        const int ln = fresh_lane(), n = ln & 31;
        dma4(ln < 32 ? L2h + rowb + n : Dh + rowb + n, &meta[st][0]);
      }
    } else {  // the ragged last step of a block, or a block without columns: rows past the end repeat a valid one
      const int nvalid = max(left, 0);
      const int ln = fresh_lane();
      const uint32_t boff = (uint32_t)(nvalid > 0 ? rowb : 0) * row_stride;
#pragma unroll
      for (int j = 0; j < WLW0; j++) {
        const int u = j % NLO;
        const uint32_t off = (uint32_t)min(lane_row(ln, u), max(nvalid - 1, 0)) * row_stride + lane_chunk(ln, u);
        dma16s((j >= NLO ? dOh : Qh) + boff, off, (j >= NLO ? dstdO : dstQ) + (w + DKV_NW * u) * RPL * D);
      }
      if (w == 0) {
        const int n = ln & 31;
        const bool ok = n < nvalid;
        const float* src = ln < 32 ? (ok ? L2h + rowb + n : c_pinf) : (ok ? Dh + rowb + n : c_zero_f);
        dma4(src, &meta[st][0]);
      }
    }
    if (qs == 0 && w < SG / 64) {
      const int bi = pc.bi;
      const int cl = w * 64 + fresh_lane();
      const int32_t* src = c_m1;
      if (cl < pc.ncols) {
        src = PARTIAL ? p.plist + ((size_t)h * p.nblk_cap + bi) * MAXPART + pc.x + grp * SG + cl
                      : p.slot_tab + ((size_t)h * p.nblk_cap + bi) * p.kpad + grp * SG + cl;
      }
      dma4(src, &idbuf[(v / NSUB) & 1][w * 64]);
    }
  };

  // kj: first row of this lane's key (partial mode also ke: its end row).  A clean-mode column needs the row
  // mask only in the block its key entered in (`entering`: some column of this wave is in that state).
  constexpr int KJ_NONE = PARTIAL ? 0x7fffffff : -1;
  int curid = -1, kj = KJ_NONE, ke = 0;
  bool entering = false;
  float zq = -INFINITY;  // z / scale of this lane's key: the start value of its S accumulator
  bf16x8 kreg[KS > KL ? KS - KL : 1], vreg[KS - VL];  // B-operand fragments of this lane's key: its K row and its V row
  const bf16x8 zero8 = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  bf16x8* kl = klds + w * KL * 64 + l;
  bf16x8* vl = vlds + w * VL * 64 + l;
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    if (ks < VL) vl[64 * ks] = zero8;
    else vreg[ks < VL ? 0 : ks - VL] = zero8;
    if (ks < KL) kl[64 * ks] = zero8;
    else kreg[ks < KL ? 0 : ks - KL] = zero8;
  }
  f32x16 dvacc[CB], dkacc[CB];  // dV^T and dK^T of this lane's column
#pragma unroll
  for (int cb = 0; cb < CB; cb++)
#pragma unroll
    for (int v = 0; v < 16; v++) dvacc[cb][v] = dkacc[cb][v] = 0.f;
  float dzacc = 0.f;

  float* stage = stage_all + w * STR * LDS_ST;
  // Flush the columns whose lanes pass doit = true (wave-uniform call).  The accumulators of up to STR columns at
  // a time are transposed through the wave's LDS staging area, STC channels at a time, so that each atomic
  // instruction adds consecutive channels of one or two keys.
  // Lanes of a wave hand values to each other through LDS (in order, no barrier needed): the compiler must not
  // carry a lane's view of the staging area across.
  auto lanes_exchange = [] { asm volatile("" ::: "memory"); };
  auto flush = [&](bool doit) __attribute__((always_inline)) {
    const int ln = fresh_lane();
    const int n = ln & 31, hh = ln >> 5;
    const float dzt = dzacc + __shfl_xor(dzacc, 32);
    doit = doit && curid >= 0;
    const unsigned fm = (unsigned)__builtin_amdgcn_readfirstlane((int)(__ballot(doit) & 0xffffffffull));
    if (fm == 0) return;
    if (doit && hh == 0) atomicAdd(p.dz + (size_t)h * p.T + curid, dzt);
    int* stage_id = reinterpret_cast<int*>(stage);
    const int nf = __popc(fm), rank = __popc(fm & ((1u << n) - 1u));
    constexpr int NP = 2 * D / STC, CPP = STC / 32;  // passes (dV, then dK), 32-channel blocks per pass
    constexpr int RPI = 64 / STC, U = STR / RPI;     // keys per atomic instruction, instructions per pass
    for (int r0 = 0; r0 < nf; r0 += STR) {
      const int row = rank - r0, cnt = min(STR, nf - r0);
      const bool mine = doit && row >= 0 && row < STR;
      if (mine && hh == 0) stage_id[row * LDS_ST + STC] = curid;  // (in the padding)
      lanes_exchange();
      const int sub = RPI == 2 ? hh : 0;
      size_t off[U];  // element of staging row RPI u + sub this lane adds to, of the first pass of dV and of dK
#pragma unroll
      for (int u = 0; u < U; u++)
        off[u] = ((size_t)stage_id[(RPI * u + (RPI * u + sub < cnt ? sub : 0)) * LDS_ST + STC] * p.H_kv + g) * D + (ln & (STC - 1));
      // A wave's LDS accesses take effect in order: the next pass is written as soon as the reads of the one before it
      // are on their way, and the atomics of a pass follow the reads of the next.
      float x[2][U];
      auto add = [&](int ps) __attribute__((always_inline)) {
        float* dst = ps < NP / 2 ? p.dV32 : p.dK32;
        const int c0 = ps % (NP / 2) * STC;
#pragma unroll
        for (int u = 0; u < U; u++)
          if (RPI * u < cnt) {
            if (RPI * u + sub < cnt) atomicAdd(dst + off[u] + c0, ps < NP / 2 ? x[ps & 1][u] : x[ps & 1][u] * scale);
          }
      };
#pragma unroll
      for (int ps = 0; ps < NP; ps++) {
        if (mine) {
#pragma unroll
          for (int cb = 0; cb < CPP; cb++)
#pragma unroll
            for (int gq = 0; gq < 4; gq++) {
              const f32x16& acc = ps < NP / 2 ? dvacc[ps % (NP / 2) * CPP + cb] : dkacc[ps % (NP / 2) * CPP + cb];
              f32x4 v4;
#pragma unroll
              for (int u = 0; u < 4; u++) v4[u] = acc[4 * gq + u];
              *reinterpret_cast<f32x4*>(&stage[row * LDS_ST + 32 * cb + 8 * gq + 4 * hh]) = v4;
            }
        }
        lanes_exchange();
#pragma unroll
        for (int u = 0; u < U; u++) x[ps & 1][u] = stage[(RPI * u + sub) * LDS_ST + (ln & (STC - 1))];
        lanes_exchange();
        if (ps > 0) add(ps - 1);
      }
      add(NP - 1);
    }
  };

  FragOffsets<D> fo;
  fo.init(l);
  Cursor cc = {-1, 0, 0, 0, 0};
  for (int v = 0; v < NS - 1; v++) issue(v);

  for (int v = 0; v < nsteps; v++) {
    // copies of step v must have landed: at most NS-2 later steps' worth may still be in flight
    // (the occasional id copies and the flush traffic only make this wait more conservative)
    if (w == 0) wait_vmcnt<(NS - 2) * (WLW0 + 1)>();
    else wait_vmcnt<(NS - 2) * WLW0>();
    lds_barrier();  // (and every wave is done with step v - 1, whose stage the next copies take)
    fo.pin();
    issue(v + NS - 1);

    const int qs = v % NSUB;
    if (qs == 0) cc = load_cursor(v / NSUB);
    const int ncols = cc.ncols, row0 = cc.row0, row1 = cc.row1;
    if (qs == 0) {
      const int cl = 32 * w + n;
      int newid = (cl < ncols) ? idbuf[(v / NSUB) & 1][cl] : -1;
      if (!PARTIAL) {
        if (newid < -1) newid = -2 - newid;  // enters inside this block
        // Columns that are new in this block (the first k rows of a document) are not in the table: column
        // c takes the document's key c, unless that key is gone again before the block ends.
        const int col = grp * SG + cl, old = row0 - cc.x;
        if (p.causal && grp * SG + 32 * w + 31 >= old && cl < ncols && col >= old) {
          const int key = cc.x + col;
          if (p.expiry[(size_t)h * p.T + key] >= row1) newid = key;
        }
        entering = p.causal && __any(newid > row0);
        if (newid != curid) kj = newid >= 0 ? newid : KJ_NONE;
      }
      const bool changed = newid != curid;
      if (__any(changed)) {
        // The new keys' rows are requested first and arrive while the finished keys are flushed
        // (the flush reads the accumulators and the old ids only).
        if (changed) {
          if (newid >= 0) {
            const size_t off = ((size_t)newid * p.H_kv + g) * D + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
              if (ks < KL) dma16(p.K + off + 16 * ks, klds + (w * KL + ks) * 64);
              else kreg[ks < KL ? 0 : ks - KL] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p.K + off + 16 * ks));
              if (ks < VL) dma16(p.V + off + 16 * ks, vlds + (w * VL + ks) * 64);
              else vreg[ks < VL ? 0 : ks - VL] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p.V + off + 16 * ks));
            }
            zq = zqh[newid];
            if (PARTIAL) {
              kj = newid;
              ke = p.expiry[(size_t)h * p.T + newid];
            }
          } else {
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
              if (ks < VL) vl[64 * ks] = zero8;
              else vreg[ks < VL ? 0 : ks - VL] = zero8;
              if (ks < KL) kl[64 * ks] = zero8;
              else kreg[ks < KL ? 0 : ks - KL] = zero8;
            }
            zq = -INFINITY;
            if (PARTIAL) {
              kj = KJ_NONE;
              ke = 0;
            }
          }
        }
        flush(changed);  // finished keys out, then re-arm the changed columns
        if (changed) {
#pragma unroll
          for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int vv = 0; vv < 16; vv++) dvacc[cb][vv] = dkacc[cb][vv] = 0.f;
          dzacc = 0.f;
          curid = newid;
        }
        wait_vmcnt<0>();  // the rows that go to LDS (the other loads and the atomics too)
        if (PARTIAL) settle(ke);
        settle(zq);
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
          if (ks >= KL) settle(kreg[ks < KL ? 0 : ks - KL]);
          if (ks >= VL) settle(vreg[ks < VL ? 0 : ks - VL]);
        }
      }
    }
    if (ncols == 0 || row0 + SUB * qs >= row1) continue;  // nothing to do this step
    if (PARTIAL) {
      // none of this wave's keys is active on these rows (the entering keys that do not stay are listed by
      // ascending first row, the expiring ones behind them by ascending end row)
      const int rf = row0 + SUB * qs;
      if (!__any((kj < rf + SUB) & (ke > rf))) continue;
    } else if (entering && !__any((curid >= 0) & (kj < row0 + SUB * qs + SUB))) {
      continue;  // none of this wave's keys has entered yet
    }

    const int st = v % NS;
    const uint16_t* Qs = ringQ + st * STILE;
    const uint16_t* dOs = ringdO + st * STILE;

    // S starts at z / scale, so that scale * S is the biased score (a key that enters in a later step: all of
    // its rows stay at -inf, so P = 0 and dS = 0 exactly; in the step it enters in, the rows before it do)
    f32x16 sacc, dpacc;
    const int rf = row0 + SUB * qs;
    float z0 = zq;
    if (!PARTIAL && entering) z0 = kj >= rf + SUB ? -INFINITY : zq;
    if (!PARTIAL && entering && __any((kj > rf) & (kj < rf + SUB))) {
      const int first = kj - rf - 4 * hh;
#pragma unroll
      for (int vv = 0; vv < 16; vv++) sacc[vv] = 8 * (vv >> 2) + (vv & 3) >= first ? z0 : -INFINITY;
    } else {
#pragma unroll
      for (int vv = 0; vv < 16; vv++) sacc[vv] = z0;
    }
    // The products in a fixed order (S, dP, dV^T, dK^T), each with the LDS reads of the fragments LEAD products ahead and
    // a share of the element-wise work: P under dP and the first products with P, dS under dV and the first with dS.
    // (64 channels: the order is the compiler's; three waves share a SIMD there, and fragments read ahead would spill)
    const float* row_meta = meta[st] + 4 * (fresh_lane() >> 5);
    constexpr int NM = 2 * KS + 4 * CB, LEAD = D == 256 ? 4 : D == 128 ? 2 : 0, EPS = 16 / KS;
    bf16x8 fr[LEAD + 1], fk[KL || VL ? LEAD + 1 : 1], bb[2], db[2];
    f32x4 ls[2];
    auto frag = [&](auto mc) __attribute__((always_inline)) {
      constexpr int m = decltype(mc)::value;
      if constexpr (m < KS) {
        fr[m % (LEAD + 1)] = fo.row_frag(Qs, 0, m);
        if constexpr (m < KL) fk[m % (LEAD + 1)] = kl[64 * m];
      } else if constexpr (m < 2 * KS) {
        fr[m % (LEAD + 1)] = fo.row_frag(dOs, 0, m - KS);
        if constexpr (m - KS < VL) fk[m % (LEAD + 1)] = vl[64 * (m - KS)];
      } else if constexpr (m < 2 * KS + 2 * CB) {
        fr[m % (LEAD + 1)] = fo.tr_frag(dOs, 16 * ((m - 2 * KS) / CB), (m - 2 * KS) % CB);
      } else if constexpr (m < NM) {
        fr[m % (LEAD + 1)] = fo.tr_frag(Qs, 16 * ((m - 2 * KS - 2 * CB) / CB), (m - 2 * KS - 2 * CB) % CB);
      }
    };
    static_for<LEAD>(frag);
    if constexpr (D != 64) __builtin_amdgcn_sched_barrier(0);
    static_for<NM>([&](auto mc) __attribute__((always_inline)) {
      constexpr int m = decltype(mc)::value;
      frag(std::integral_constant<int, m + LEAD>{});
      // dP starts at -D_i of the accumulator's rows: the products then leave dP - D, what dS needs
      if constexpr (m >= KS - 4 && m < KS) {
        constexpr int gq = m - (KS - 4);
        const f32x4 dd = *reinterpret_cast<const f32x4*>(&row_meta[32 + 8 * gq]);
#pragma unroll
        for (int u = 0; u < 4; u++) dpacc[4 * gq + u] = dd[u];
      }
      if constexpr (m < KS) {
        if constexpr (m < KL) sacc = mfma32(fr[m % (LEAD + 1)], fk[m % (LEAD + 1)], sacc);
        else sacc = mfma32(fr[m % (LEAD + 1)], kreg[m - KL], sacc);
      } else if constexpr (m < 2 * KS) {
        if constexpr (m - KS < VL) dpacc = mfma32(fr[m % (LEAD + 1)], fk[m % (LEAD + 1)], dpacc);
        else dpacc = mfma32(fr[m % (LEAD + 1)], vreg[m - KS - VL], dpacc);
      } else if constexpr (m < 2 * KS + 2 * CB) {
        constexpr int i = m - 2 * KS;
        dvacc[i % CB] = mfma32(fr[m % (LEAD + 1)], bb[i / CB], dvacc[i % CB]);
      } else {
        constexpr int i = m - 2 * KS - 2 * CB;
        dkacc[i % CB] = mfma32(fr[m % (LEAD + 1)], db[i / CB], dkacc[i % CB]);
      }
      constexpr int p0 = KS + 1, d0 = 2 * KS + 2;  // first products that P and dS form under
      constexpr int PQ = 4 / EPS;  // products per four elements of P: their LSE is read PQ products ahead
      if constexpr (m >= p0 - PQ && m < p0 + KS - PQ && (m - p0 + PQ) % PQ == 0) {
        constexpr int gq = (m - p0 + PQ) / PQ;
        ls[gq & 1] = *reinterpret_cast<const f32x4*>(&row_meta[8 * gq]);
      }
      if constexpr (m >= p0 && m < p0 + KS) {
#pragma unroll
        for (int vv = (m - p0) * EPS; vv < (m - p0 + 1) * EPS; vv++) {
          float pv = fast_exp2(fmaf(sacc[vv], c2, -ls[(vv >> 2) & 1][vv & 3]));
          if (PARTIAL) {
            const int row = rf + 8 * (vv >> 2) + 4 * hh + (vv & 3);
            pv = ((row >= kj) & (row < ke)) ? pv : 0.f;
          }
          sacc[vv] = pv;
          bb[vv >> 3][vv & 7] = (__bf16)pv;
        }
      }
      if constexpr (m >= d0 && m < d0 + KS) {
#pragma unroll
        for (int vv = (m - d0) * EPS; vv < (m - d0 + 1) * EPS; vv++) {
          const float ds = sacc[vv] * dpacc[vv];
          dzacc += ds;
          db[vv >> 3][vv & 7] = (__bf16)ds;
        }
      }
      if constexpr (D != 64) __builtin_amdgcn_sched_barrier(0);
    });
  }
  wait_vmcnt<0>();
  flush(true);
}

// The slot sweeps' workgroups first, one for every place on the chip, then those of the partial lists: these are short
// and start where sweeps end early (a sweep of 16384 tokens x 32 heads ends between 917 and 1146 us).  One launch against
// two, us: 16384 x 32 heads 1260 -> 1155, 2 x 4096 x 16 heads 238 -> 217, packed 65536 x 16 heads of 64 channels 538 -> 495,
// 16 heads of 256 channels 1523 -> 1443, 300 tokens x 2 heads 53 -> 28.
template <int D>
__global__ __launch_bounds__(DKV_NW * 64, D == 256 ? 1 : D == 64 ? 3 : 2) void dkv_kernel(BwdArgs p) {
  __shared__ DkvShared<D> sm;
  const int wg = wg_id();
  if (wg < (int)p.grid_clean) dkv_sweep<D, false>(p, wg, sm);
  else dkv_sweep<D, true>(p, wg - (int)p.grid_clean, sm);
}

// dK, dV: fp32 accumulators -> bf16 outputs.  HBM-bound (5.8 TB/s).  SPARSE: a row that no q-head of its group ever keeps
// has a zero gradient, and its accumulators are not read.  A workgroup looks the expiries of its rows up once per row and
// head, before its first load (once per float4 before): what that costs where every row is kept after all, with scores
// that rise along the keys, is about one memory latency.  Every row read / random scores / rising scores, us: packed
// 65536 x 16 heads of 64 channels, window 512, 131 / 73 / 134 (before: 99 / 144), the same of 128 channels 311 / 159 / 284
// (194 / 315), 32768 x 2 heads of 128 channels 17.3 / 8.8 / 20.1 (24 / 23), 8192 x 8 heads of 256 channels 31.7 / 14.0 /
// 35.5 (18 / 38).  Workgroups of four times the rows: 78 / 141, 170 / 294, 14.0 / 24.7, 17.7 / 34.6.
struct CvtArgs {
  const float *a, *b;
  uint16_t *oa, *ob;
  const int32_t* expiry;
  int T, H_kv, G;
  size_t n4;
  unsigned nwg;
};
constexpr int CVT_U = 4, CVT_N4 = 256 * CVT_U;  // float4 per thread and per workgroup of the sparse form
__device__ __forceinline__ void cvt_store(uint16_t* out, size_t i, float4 x) {
  bf16x4 o;
  o[0] = (__bf16)x.x; o[1] = (__bf16)x.y; o[2] = (__bf16)x.z; o[3] = (__bf16)x.w;
  reinterpret_cast<bf16x4*>(out)[i] = o;
}
template <int D, bool SPARSE>
__global__ __launch_bounds__(256) void cvt_bf16_kernel(CvtArgs p) {  // (256 threads)
  const float4 *a = reinterpret_cast<const float4*>(p.a), *b = reinterpret_cast<const float4*>(p.b);
  if constexpr (!SPARSE) {
    const size_t st = (size_t)p.nwg * 256;
    for (size_t i = wg_id() * (size_t)256 + thread_id(); i < p.n4; i += st) {
      const float4 x = a[i], y = b[i];
      cvt_store(p.oa, i, x);
      cvt_store(p.ob, i, y);
    }
  } else {
    constexpr int ROW4 = D / 4, ROWS = CVT_N4 / ROW4, QP = 256 / ROWS;  // QP threads share the heads of a row's group
    __shared__ int kept[QP][ROWS];
    const int tid = thread_id();
    const size_t base = (size_t)wg_id() * CVT_N4, row = base / ROW4 + tid % ROWS;
    int any = 0;  // (a row past the end has none)
    if (row < p.n4 / ROW4) {
      const unsigned t = (unsigned)row / (unsigned)p.H_kv, g = (unsigned)row - t * (unsigned)p.H_kv;
      const int32_t* e = p.expiry + (size_t)g * p.G * p.T + t;
      for (int q = tid / ROWS; q < p.G; q += QP) any |= e[(size_t)q * p.T] > (int)t;
    }
    kept[tid / ROWS][tid % ROWS] = any;
    __syncthreads();
    float4 x[CVT_U], y[CVT_U];
#pragma unroll
    for (int u = 0; u < CVT_U; u++) {
      const int j = tid + 256 * u;
      x[u] = y[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      int read = 0;
#pragma unroll
      for (int q = 0; q < QP; q++) read |= kept[q][j / ROW4];
      if (read) {
        x[u] = a[base + j];
        y[u] = b[base + j];
      }
    }
#pragma unroll
    for (int u = 0; u < CVT_U; u++) {
      const size_t i = base + tid + 256 * u;
      if (i < p.n4) {
        cvt_store(p.oa, i, x[u]);
        cvt_store(p.ob, i, y[u]);
      }
    }
  }
}

static unsigned grid_for(size_t n, size_t per_block) {
  size_t g = (n + per_block - 1) / per_block;
  if (g > (1u << 20)) g = 1u << 20;
  return g < 1 ? 1u : (unsigned)g;
}

int launch_bwd(const Ptrs& p, const void* Q, const void* K, const void* V, const void* O, const void* dO,
               const float* LSE, const float* z, const int32_t* expiry, const int32_t* cu, void* dQ, void* dK,
               void* dV, float* dz, const ScoreGrad* sg, char* ws, hipStream_t st) {
  (void)cu;
  (void)z;
  const dma_shape& s = p.s;
  const PlanLayout& L = p.pl;
  const WsLayout wl = ws_layout(s);
  BwdArgs a;
  a.Q = (const uint16_t*)Q; a.K = (const uint16_t*)K; a.V = (const uint16_t*)V;
  a.O = (const uint16_t*)O; a.dO = (const uint16_t*)dO; a.dQ = (uint16_t*)dQ;
  a.zq = (const float*)(p.plan + L.off_zq); a.LSE = LSE; a.expiry = expiry;
  a.Dws = (float*)(ws + wl.off_D); a.L2ws = (float*)(ws + wl.off_L2);
  a.dK32 = (float*)(ws + wl.off_dK); a.dV32 = (float*)(ws + wl.off_dV); a.dz = dz;
  a.blk = (const int4*)(p.plan + L.off_blk);
  a.slot_tab = (const int32_t*)(p.plan + L.off_slot);
  a.pcnt = (const int32_t*)(p.plan + L.off_pcnt);
  a.pent = (const int32_t*)(p.plan + L.off_pent);
  a.plist = (const int32_t*)(p.plan + L.off_plist);
  a.consts = p.plan + L.off_consts;
  a.T = s.T; a.H_q = s.H_q; a.H_kv = s.H_kv; a.k = s.k; a.nblk_cap = L.nblk_cap; a.kpad = L.kpad; a.causal = s.causal;
  {  // Sweep length of a clean-mode work item: as long as possible with an item for every workgroup that fits the
    // chip at once (three per compute unit at 64 channels, two at 128, one at 256) and no second round of a few
    // items.  us of a training step, about 512 items but rather more -> this rule: 65536 packed tokens, d = 64
    // 1740 -> 1690; 16384 tokens x 32 heads, d = 64 1770 -> 1680; 40000 tokens x 8 heads, d = 128, window 100
    // 721 -> 693; 9000 tokens x 16 heads, d = 256 1437 -> 1314.
    const long groups = (long)(L.kpad / SG) * s.H_q, resident = s.d == 64 ? 768 : s.d == 128 ? 512 : 256;
    long seg = ((long)((s.T + BQ - 1) / BQ) * groups + resident - 1) / resident;
    if (seg < 2) seg = 2;
    if (seg > L.nblk_cap) seg = L.nblk_cap;
    if (seg > MAXSWEEP) seg = MAXSWEEP;
    a.seg = (int)seg;
    // Blocks per partial-mode work item: up to 8, which amortises the pipeline fill, but at least about 1024
    // items (most blocks list at most one group of columns, so about as many workgroups have work; 512 fit the
    // chip at once): 16384 tokens x 32 heads 312 us with 256 items, 196 with 1024; 65536 x 16 heads, d = 64: 184 and 180.
    long sp = (long)L.nblk_cap * s.H_q / 1024;
    a.seg_part = sp < 1 ? 1 : sp > 8 ? 8 : (int)sp;
  }

  const size_t nkv = (size_t)s.T * s.H_kv * s.d;
  a.zero_n4 = ((wl.off_dV - wl.off_dK) / 4 + nkv + 3) / 4;  // (the layout pads both buffers to 256 bytes)
  a.dz_n = (size_t)s.H_q * s.T;
  a.dW = sg ? sg->dW : nullptr; a.dA = sg ? sg->dA : nullptr;
  a.dW_n = sg ? s.H_q * s.d : 0; a.dA_n = sg ? s.H_q : 0;
  prof_begin(DMA_STAGE_BWD_ZERO, st);  // (an empty stage: dq_kernel clears the accumulators)
  prof_end(DMA_STAGE_BWD_ZERO, st);
  // dq_kernel: half blocks at 64 channels (three per compute unit), at 256 (four waves with the whole register file each)
  // and, at 128, where every one of them finds a compute unit of its own (us, whole / half blocks: 300 tokens x 2 heads
  // 19.5 / 16.5, 1024 x 32 45 / 38, 4096 x 4 57 / 47; with more of them than compute units 5 x 800 x 8 36 / 45).
  const bool few = 2 * most_blocks(s) <= CUS, halves = s.d != 128 || few;
  const unsigned gq = halves ? xcd_grid(s.H_q, 2l * L.nblk_cap) : xcd_grid(s.H_q, L.nblk_cap);
  a.grid_dq = gq;
  const unsigned gclean = xcd_grid(s.H_q, (long)((L.nblk_cap + a.seg - 1) / a.seg) * (L.kpad / SG));
  const unsigned gpart = xcd_grid(s.H_q, (long)((L.nblk_cap + a.seg_part - 1) / a.seg_part) * (MAXPART / SG));
  prof_begin(DMA_STAGE_BWD_DQ, st);
  if (s.d == 256) dq_kernel<256, 4, 1><<<gq, 256, 0, st>>>(a);
  else if (s.d == 128 && few) dq_kernel<128, 8, 1, 2><<<gq, 512, 0, st>>>(a);
  else if (s.d == 128) dq_kernel<128, 8, 2><<<gq, 512, 0, st>>>(a);
  else dq_kernel<64, 4, 2><<<gq, 256, 0, st>>>(a);
  prof_end(DMA_STAGE_BWD_DQ, st);
  a.grid_clean = gclean;
  prof_begin(DMA_STAGE_BWD_DKV, st);
  if (s.d == 256) dkv_kernel<256><<<gclean + gpart, DKV_NW * 64, 0, st>>>(a);
  else if (s.d == 128) dkv_kernel<128><<<gclean + gpart, DKV_NW * 64, 0, st>>>(a);
  else dkv_kernel<64><<<gclean + gpart, DKV_NW * 64, 0, st>>>(a);
  prof_end(DMA_STAGE_BWD_DKV, st);
  prof_begin(DMA_STAGE_BWD_PART, st);  // (an empty stage: the launch above has the partial lists too)
  prof_end(DMA_STAGE_BWD_PART, st);
  prof_begin(DMA_STAGE_BWD_CVT, st);
  // About how many rows are kept: with random scores a document of n keys keeps k (1 + ln(n / k)) of them at some time.
  const double n = (double)s.T / s.n_docs, share = s.causal && n > s.k ? s.k / n * (1. + std::log(n / s.k)) : 1.;
  // (small calls are all latency: 2048 tokens x 2 heads 6.2 -> 8.1 us)
  const bool sparse = nkv >= 1u << 22 && 1. - std::pow(1. - share, s.H_q / s.H_kv) < 0.6;
  if (sg) {
    const int rc = launch_kv_scores(s, V, *sg, dz, dV, {a.dK32, a.dV32, expiry, (uint16_t*)dK}, sparse, st);
    prof_end(DMA_STAGE_BWD_CVT, st);
    return rc;
  }
  const unsigned gcvt = sparse ? (unsigned)((nkv / 4 + CVT_N4 - 1) / CVT_N4) : grid_for(nkv / 4, 1024);
  const CvtArgs ca = {a.dK32, a.dV32, (uint16_t*)dK, (uint16_t*)dV, expiry, s.T, s.H_kv, s.H_q / s.H_kv, nkv / 4, gcvt};
#define DMA_CVT(DD) (sparse ? cvt_bf16_kernel<DD, true> : cvt_bf16_kernel<DD, false>)<<<gcvt, 256, 0, st>>>(ca)
  if (s.d == 256) DMA_CVT(256);
  else if (s.d == 128) DMA_CVT(128);
  else DMA_CVT(64);
#undef DMA_CVT
  prof_end(DMA_STAGE_BWD_CVT, st);
  return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
}

}  // namespace dma
