// Gradient of the content scores (chain rule of Eq. 3; Section 6: the bias is the differentiable
// path into the score parameters).  Given dz [H_q, T] from the attention backward:
//   x = w_h . v_{g(h), j},  z = exp(A_h softplus(x)),
//   dx = dz z A_h sigmoid(x),  dA_h = sum_j dz z softplus(x),  dW_h = sum_j dx v_{g(h), j},
//   dVz_{j, g} = sum_{h in g} dx_{h, j} w_h.
// HBM-bound: one pass over V (read) and dV (write, plus a read when accumulating), dz read once.
#include "common.h"

#include <algorithm>

namespace dma {

// One workgroup per (TT-token tile, kv-head); TT = 64, or 32 at 256 channels (the V tile is kept in LDS).  (1) every row is held by D / 8 lanes, which reduce
// x = w_h . v for each q-head of the group; (2) one thread per (q-head, row) turns x into dx and
// the dA summand (the transcendental work, 64 different pairs per wave instruction); (3) the row's
// lanes add dx w_h into their 8 channels of the dV row; (4) dW and dA partial sums of the tile
// (from dx and the V tile kept in LDS) are added to the outputs with fp32 atomics (G * D + G per
// workgroup).
template <typename TV, int D, int TT>
__global__ __launch_bounds__(256) void mask_bwd_kernel(const TV* __restrict__ V, const float* __restrict__ W,
                                                       const float* __restrict__ A, const float* __restrict__ dz,
                                                       float* dW, float* dA, TV* dV, int accumulate, int T,
                                                       int H_q, int H_kv, int tiles_per_wg) {
  extern __shared__ float sm[];  // [TT][D] V tile, [G][D] w, [G][D] dW partial, [G][TT] x then dx, [G][TT] dA summands, [G] dA partial
  constexpr int LPR = D / 8, RPP = 256 / LPR, NP = TT / RPP;
  const int g = blockIdx.y, G = H_q / H_kv;
  float* vs = sm;
  float* ws = vs + TT * D;
  float* dws = ws + G * D;
  float* dxs = dws + G * D;
  float* das = dxs + G * TT;
  float* dap = das + G * TT;
  const int tid = threadIdx.x, sub = tid % LPR, rl = tid / LPR;
  for (int i = tid; i < G * D; i += 256) {
    ws[i] = W[(size_t)g * G * D + i];
    dws[i] = 0.f;
  }
  for (int i = tid; i < G; i += 256) dap[i] = 0.f;
  // a workgroup walks tiles_per_wg consecutive TT-token tiles, so that the contended atomics on dW / dA
  // are issued once per workgroup instead of once per tile
  for (int tile = 0; tile < tiles_per_wg; tile++) {
  const int t0 = (blockIdx.x * tiles_per_wg + tile) * TT;
  if (t0 >= T) break;
  __syncthreads();  // the previous tile's readers of vs / dxs / das are done
  float v[NP][8];
#pragma unroll
  for (int pass = 0; pass < NP; pass++) {
    const int r = pass * RPP + rl, t = t0 + r;
#pragma unroll
    for (int e = 0; e < 8; e++) v[pass][e] = 0.f;
    if (t < T) {
      const size_t roff = ((size_t)t * H_kv + g) * D + 8 * sub;
      if constexpr (sizeof(TV) == 2) {
        const uint4 raw = *reinterpret_cast<const uint4*>(V + roff);
        const uint32_t u[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
          v[pass][2 * e] = __uint_as_float(u[e] << 16);
          v[pass][2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
        }
      } else {
        const float4 x0 = *reinterpret_cast<const float4*>(V + roff);
        const float4 x1 = *reinterpret_cast<const float4*>(V + roff + 4);
        v[pass][0] = x0.x; v[pass][1] = x0.y; v[pass][2] = x0.z; v[pass][3] = x0.w;
        v[pass][4] = x1.x; v[pass][5] = x1.y; v[pass][6] = x1.z; v[pass][7] = x1.w;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; e++) vs[r * D + 8 * sub + e] = v[pass][e];
  }
  __syncthreads();
  // (1) x[hh][r]
#pragma unroll
  for (int pass = 0; pass < NP; pass++) {
    const int r = pass * RPP + rl;
    for (int hh = 0; hh < G; hh++) {
      const float* w = ws + hh * D + 8 * sub;
      float x = 0.f;
#pragma unroll
      for (int e = 0; e < 8; e++) x = fmaf(v[pass][e], w[e], x);
      x = group_sum<LPR>(x);
      if (sub == 0) dxs[hh * TT + r] = x;
    }
  }
  __syncthreads();
  // (2) dx and the dA summand, one (q-head, row) pair per thread
  for (int idx = tid; idx < G * TT; idx += 256) {
    const int hh = idx / TT, r = idx % TT, t = t0 + r, h = g * G + hh;
    float dx = 0.f, da = 0.f;
    if (t < T) {
      const float x = dxs[idx], a = A[h];
      const float sp = fmaxf(x, 0.f) + log1pf(expf(-fabsf(x)));
      const float zv = expf(a * sp);
      const float sig = 1.f / (1.f + expf(-x));
      const float dzz = dz[(size_t)h * T + t] * zv;
      dx = dzz * a * sig;
      da = dzz * sp;
    }
    dxs[idx] = dx;
    das[idx] = da;
  }
  __syncthreads();
  // (3) dVz rows
#pragma unroll
  for (int pass = 0; pass < NP; pass++) {
    const int r = pass * RPP + rl, t = t0 + r;
    if (t >= T) continue;  // (no barrier inside this loop)
    float dv[8];
#pragma unroll
    for (int e = 0; e < 8; e++) dv[e] = 0.f;
    for (int hh = 0; hh < G; hh++) {
      const float dx = dxs[hh * TT + r];
      const float* w = ws + hh * D + 8 * sub;
#pragma unroll
      for (int e = 0; e < 8; e++) dv[e] = fmaf(dx, w[e], dv[e]);
    }
    const size_t roff = ((size_t)t * H_kv + g) * D + 8 * sub;
    if constexpr (sizeof(TV) == 2) {
      if (accumulate) {
        const uint4 raw = *reinterpret_cast<const uint4*>(dV + roff);
        const uint32_t u[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
          dv[2 * e] += __uint_as_float(u[e] << 16);
          dv[2 * e + 1] += __uint_as_float(u[e] & 0xffff0000u);
        }
      }
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = (__bf16)dv[e];
      *reinterpret_cast<uint4*>(dV + roff) = __builtin_bit_cast(uint4, o);
    } else {
      float4 o0 = make_float4(dv[0], dv[1], dv[2], dv[3]), o1 = make_float4(dv[4], dv[5], dv[6], dv[7]);
      if (accumulate) {
        const float4 p0 = *reinterpret_cast<const float4*>(dV + roff);
        const float4 p1 = *reinterpret_cast<const float4*>(dV + roff + 4);
        o0.x += p0.x; o0.y += p0.y; o0.z += p0.z; o0.w += p0.w;
        o1.x += p1.x; o1.y += p1.y; o1.z += p1.z; o1.w += p1.w;
      }
      *reinterpret_cast<float4*>(dV + roff) = o0;
      *reinterpret_cast<float4*>(dV + roff + 4) = o1;
    }
  }
  // (4) dW[h, c] += sum_r dx[h, r] V[r, c]: thread per (hh, c); dA[h] += sum_r dz z softplus(x)
  for (int idx = tid; idx < G * D; idx += 256) {
    const int hh = idx / D, c = idx % D;
    float s = 0.f;
#pragma unroll 8
    for (int r = 0; r < TT; r++) s = fmaf(dxs[hh * TT + r], vs[r * D + c], s);
    dws[idx] += s;  // (the same thread owns idx for every tile)
  }
  for (int hh = tid; hh < G; hh += 256) {
    float s = 0.f;
    for (int r = 0; r < TT; r++) s += das[hh * TT + r];
    dap[hh] += s;
  }
  }  // tiles
  for (int idx = tid; idx < G * D; idx += 256) atomicAdd(dW + (size_t)g * G * D + idx, dws[idx]);
  for (int hh = tid; hh < G; hh += 256) atomicAdd(dA + g * G + hh, dap[hh]);
}

// The same for bf16 values and groups of 1, 2, 4 or 8 q-heads, without LDS tiles or barriers: a value row is held
// by D / 8 lanes with the group's weights and dW sums in registers, a wave walks its rows U per lane group at a
// time, and the V, dV and dz of the next rows are requested before the current ones are worked on.  The tile
// kernel above was bound by three dependent round trips to memory and five barriers per tile.  The
// transcendental work of the U * G (row, q-head) pairs of a lane group is dealt out to its lanes.  us, tile
// kernel -> this one: 16384 tokens, 32 / 8 heads, d = 128 65 -> 30 (3.4 TB/s); 65536 tokens, 16 heads, d = 64
// 111 -> 71; 16384 tokens, 16 / 4 heads, d = 256 100 -> 32; 8192 tokens, 16 / 4 heads, d = 128 25 -> 19.
// Groups of 3, 5, 6, 7 and more than 8 q-heads keep the tile kernel (a lane's pairs would belong to several q-heads):
// 16384 tokens, d = 128, 24 / 8 heads 51 us, 28 / 4 heads 67.
//
// FROM: what the rest of dV comes from.  BF16: dV itself, if accumulate.  F32, F32_KEPT: the attention backward's fp32
// accumulators of dK and dV; dK is converted on the way and the sum of both parts of dV rounded once.  F32_KEPT does not
// read a row that no head of the group ever keeps (its accumulators and dz are zero); its expiries are requested two
// trips ahead.
// HBM-bound.  Conversion, fill and this kernel as three launches / one, us: packed 65536 tokens x 16 heads of 64 channels 162 / 118
// (63 % of the rows are not read), 16384 x 32 / 8 heads of 128 63 / 43 (235 MB: 5.4 TB/s), 2 x 4096 x 16 / 4 31 / 21,
// 256 x 2 of 64 14 / 9.  Sums and broadcasts over a row's lanes through registers instead of LDS, us: 8 heads per group, 40000 rows
// of 64 channels 35 -> 19, 100000 of 128 46 -> 35; 16384 x 8 rows of 128, 4 heads 28.8 -> 27.0.
enum { BF16, F32, F32_KEPT };
template <int D, int G, int FROM>
__global__ __launch_bounds__(256) void mask_bwd_rows_kernel(const uint16_t* __restrict__ V, const float* __restrict__ W,
                                                            const float* __restrict__ A, const float* __restrict__ dz,
                                                            float* dW, float* dA, uint16_t* dV, int accumulate, int T,
                                                            int H_kv, int rows_per_wg, KvAccum acc) {
  constexpr int LPR = D / 8, RPW = 64 / LPR, U = 2, STEP = 4 * RPW * U, NR = (U * G + LPR - 1) / LPR;
  static_assert(LPR % G == 0, "a lane's pairs belong to one q-head");
  const int g = blockIdx.y, tid = threadIdx.x, w = tid >> 6, l = tid & 63, sub = l % LPR, rg = l / LPR;
  const int t_begin = blockIdx.x * rows_per_wg, t_end = min(T, t_begin + rows_per_wg);
  const int hi = sub % G;  // q-head of this lane's pairs
  float wr[G][8], dw[G][8], da = 0.f;
#pragma unroll
  for (int h = 0; h < G; h++) {
    const float4* w4 = reinterpret_cast<const float4*>(W + (size_t)(g * G + h) * D + 8 * sub);
    const float4 x0 = w4[0], x1 = w4[1];
    wr[h][0] = x0.x; wr[h][1] = x0.y; wr[h][2] = x0.z; wr[h][3] = x0.w;
    wr[h][4] = x1.x; wr[h][5] = x1.y; wr[h][6] = x1.z; wr[h][7] = x1.w;
#pragma unroll
    for (int e = 0; e < 8; e++) dw[h][e] = 0.f;
  }
  const float a = A[g * G + hi];
  const float* dzh = dz + (size_t)(g * G + hi) * T;
  auto row = [&](int t0, int u) { return t0 + (w * U + u) * RPW + rg; };
  auto offset = [&](int t) { return ((size_t)min(t, t_end - 1) * H_kv + g) * D + 8 * sub; };
  constexpr int NF = FROM == BF16 ? 0 : 2;  // float4 of an accumulator row per lane
  uint4 vn[U], dn[U];
  float4 kn[U][NF + 1], an[U][NF + 1];  // rows of the accumulators of dK and dV
  float zn[NR];
  int en[NR];  // (F32_KEPT) expiries of the trip after the next
  const int32_t* eh = acc.expiry + (size_t)(g * G + hi) * T;
  auto request_expiry = [&](int t0) {
#pragma unroll
    for (int r = 0; r < NR; r++) {
      const int pair = sub + r * LPR, t = row(t0, pair / G);
      en[r] = pair < U * G && t < t_end ? eh[t] : 0;
    }
  };
  auto request = [&](int t0) {
    bool kept[U];
#pragma unroll
    for (int u = 0; u < U; u++) kept[u] = true;
    if constexpr (FROM == F32_KEPT) {
      uint32_t m[NR];  // the lane group's pairs whose head keeps the row
#pragma unroll
      for (int r = 0; r < NR; r++) {
        const int pair = sub + r * LPR;
        const uint64_t all = __ballot(pair < U * G && en[r] > row(t0, pair / G));
        m[r] = (uint32_t)(all >> (rg * LPR)) & (uint32_t)((1ull << LPR) - 1ull);
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        uint32_t any = 0;
#pragma unroll
        for (int i = u * G; i < (u + 1) * G; i++) any |= m[i / LPR] >> (i % LPR) & 1u;
        kept[u] = any != 0;
      }
      request_expiry(t0 + STEP);
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const size_t at = offset(row(t0, u));
      vn[u] = dn[u] = make_uint4(0, 0, 0, 0);
      if (kept[u]) vn[u] = *reinterpret_cast<const uint4*>(V + at);
      if (FROM == BF16 && accumulate) dn[u] = *reinterpret_cast<const uint4*>(dV + at);
#pragma unroll
      for (int i = 0; i < NF; i++) {
        kn[u][i] = an[u][i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (kept[u]) {
          kn[u][i] = *reinterpret_cast<const float4*>(acc.dK32 + at + 4 * i);
          an[u][i] = *reinterpret_cast<const float4*>(acc.dV32 + at + 4 * i);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < NR; r++) {
      const int pair = sub + r * LPR, t = row(t0, pair / G);
      zn[r] = pair < U * G && t < t_end ? dzh[t] : 0.f;
    }
  };
  auto unpack = [](const uint4& raw, float* o) {
    const uint32_t u[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int e = 0; e < 4; e++) {
      o[2 * e] = __uint_as_float(u[e] << 16);
      o[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
    }
  };
  if constexpr (FROM == F32_KEPT) request_expiry(t_begin);
  request(t_begin);
  for (int t0 = t_begin; t0 < t_end; t0 += STEP) {
    uint4 vc[U], dc[U];
    float4 ac[U][NF + 1];
    float zc[NR], x[U][G], dx[NR];
#pragma unroll
    for (int u = 0; u < U; u++) {
      vc[u] = vn[u];
      dc[u] = dn[u];
      if constexpr (NF > 0) {
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < NF; i++) {
          ac[u][i] = an[u][i];
          const float4 x = kn[u][i];
          o[4 * i] = (__bf16)x.x; o[4 * i + 1] = (__bf16)x.y; o[4 * i + 2] = (__bf16)x.z; o[4 * i + 3] = (__bf16)x.w;
        }
        if (row(t0, u) < t_end) *reinterpret_cast<uint4*>(acc.dK + offset(row(t0, u))) = __builtin_bit_cast(uint4, o);
      }
    }
#pragma unroll
    for (int r = 0; r < NR; r++) zc[r] = zn[r];
    if (t0 + STEP < t_end) request(t0 + STEP);
#pragma unroll
    for (int u = 0; u < U; u++) {
      float v[8];
      unpack(vc[u], v);
#pragma unroll
      for (int h = 0; h < G; h++) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) s = fmaf(v[e], wr[h][e], s);
        x[u][h] = group_sum<LPR>(s);
      }
    }
#pragma unroll
    for (int r = 0; r < NR; r++) {
      const int pair = sub + r * LPR;
      // (F32_KEPT: the score of a row that was not read is not known, and a gate above 128 makes that of x = 0 infinite: no
      // gradient, no part in the sums)
      const bool in = pair < U * G && row(t0, pair / G) < t_end && (FROM != F32_KEPT || zc[r] != 0.f);
      float xi = 0.f;
#pragma unroll
      for (int i = r * LPR; i < U * G && i < (r + 1) * LPR; i++) xi = sub == i - r * LPR ? x[i / G][i % G] : xi;
      const float sp = fmaxf(xi, 0.f) + log1pf(expf(-fabsf(xi)));
      const float zv = expf(a * sp);
      const float sig = 1.f / (1.f + expf(-xi));
      const float dzz = zc[r] * zv;
      dx[r] = in ? dzz * a * sig : 0.f;
      da += in ? dzz * sp : 0.f;
    }
    static_for<U>([&](auto uc) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      float v[8], dv[8], old[8];
      unpack(vc[u], v);
      if constexpr (FROM == BF16) {
        unpack(dc[u], old);
      } else {
#pragma unroll
        for (int i = 0; i < NF; i++) {
          old[4 * i] = ac[u][i].x; old[4 * i + 1] = ac[u][i].y; old[4 * i + 2] = ac[u][i].z; old[4 * i + 3] = ac[u][i].w;
        }
      }
#pragma unroll
      for (int e = 0; e < 8; e++) dv[e] = 0.f;
      static_for<G>([&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value, i = u * G + h;
        const float d = group_lane<LPR, i % LPR>(dx[i / LPR]);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          dv[e] = fmaf(d, wr[h][e], dv[e]);
          dw[h][e] = fmaf(d, v[e], dw[h][e]);
        }
      });
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = (__bf16)(dv[e] + old[e]);
      if (row(t0, u) < t_end) *reinterpret_cast<uint4*>(dV + offset(row(t0, u))) = __builtin_bit_cast(uint4, o);
    });
  }
  // sums of the workgroup, then one set of atomics
  __shared__ float sdw[4][G * D];
  __shared__ float sda[256];
#pragma unroll
  for (int h = 0; h < G; h++)
#pragma unroll
    for (int e = 0; e < 8; e++) {
      float s = dw[h][e];
      s = sum_groups<LPR>(s);
      if (rg == 0) sdw[w][h * D + 8 * sub + e] = s;
    }
  sda[tid] = da;
  __syncthreads();
  for (int i = tid; i < G * D; i += 256)
    atomicAdd(dW + (size_t)g * G * D + i, (sdw[0][i] + sdw[1][i]) + (sdw[2][i] + sdw[3][i]));
  if (tid < G) {
    float s = 0.f;
    for (int i = tid; i < 256; i += G) s += sda[i];  // (256 and the lane groups are multiples of G)
    atomicAdd(dA + g * G + tid, s);
  }
}

__global__ void fill_zero_kernel(float* a, size_t na, float* b, size_t nb) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0.f;
  if (i < nb) b[i] = 0.f;
}

// dynamic LDS of one workgroup; beyond 64 KiB (very many q-heads per kv-head) the shape is refused
static size_t mask_bwd_lds_bytes(const dma_shape& s) {
  const size_t G = (size_t)(s.H_q / s.H_kv), TT = s.d == 256 ? 32 : 64;
  return (TT * s.d + 2 * G * s.d + 2 * G * TT + G) * sizeof(float);
}
bool mask_bwd_fits(const dma_shape& s) { return mask_bwd_lds_bytes(s) <= 64 * 1024; }

template <int FROM>
static void launch_rows(const dma_shape& s, const void* V, const float* W, const float* A, const float* dz, float* dW,
                        float* dA, void* dV, int accumulate, const KvAccum& acc, hipStream_t st) {
  const int G = s.H_q / s.H_kv;
  const int step = 4 * (64 / (s.d / 8)) * 2;  // rows of one trip of a workgroup
  // Two workgroups per compute unit: every one ends with contended atomics on dW (1024 instead of 512: 29 us instead of
  // 19 at 8192 tokens x 4 kv-heads), and with rows in flight ahead two are enough.  Up to 512 rows each: beyond
  // that the atomics are few and shorter workgroups even out the end (65536 x 16: 84 us at 2048 rows, 71 at 512).
  // Below 64 rows each the atomics weigh more than idle compute units: one workgroup per unit, half of one where a
  // row is for at most two q-heads (us, 16 or 32 rows -> this: 16384 tokens, one head, d = 128 19.1 -> 13.7; 8192
  // tokens, one head, d = 256 19.1 -> 12.7; 4096 tokens, 16 / 4 heads, d = 128 16.9 -> 14.5).
  const long all_rows = (long)s.T * s.H_kv, wgs = G <= 2 ? 128 : 256;
  long rows = std::max(std::min((all_rows + 511) / 512, 512l), std::min((all_rows + wgs - 1) / wgs, 64l));
  rows = (rows + step - 1) / step * step;
  const dim3 rgrid((unsigned)((s.T + rows - 1) / rows), s.H_kv);
#define DMA_MR(DD, GG) \
  mask_bwd_rows_kernel<DD, GG, FROM><<<rgrid, 256, 0, st>>>((const uint16_t*)V, W, A, dz, dW, dA, (uint16_t*)dV, accumulate, s.T, s.H_kv, (int)rows, acc)
#define DMA_MRG(DD) \
  do { if (G == 1) DMA_MR(DD, 1); else if (G == 2) DMA_MR(DD, 2); else if (G == 4) DMA_MR(DD, 4); else DMA_MR(DD, 8); } while (0)
  if (s.d == 256) DMA_MRG(256);
  else if (s.d == 128) DMA_MRG(128);
  else DMA_MRG(64);
#undef DMA_MRG
#undef DMA_MR
}

bool kv_scores_fit(const dma_shape& s) {
  const int G = s.H_q / s.H_kv;
  return s.dtype == DMA_BF16 && (G == 1 || G == 2 || G == 4 || G == 8);
}

int launch_kv_scores(const dma_shape& s, const void* V, const ScoreGrad& sg, const float* dz, void* dV, const KvAccum& acc,
                     bool sparse, hipStream_t st) {
  if (sparse) launch_rows<F32_KEPT>(s, V, sg.W, sg.A, dz, sg.dW, sg.dA, dV, 1, acc, st);
  else launch_rows<F32>(s, V, sg.W, sg.A, dz, sg.dW, sg.dA, dV, 1, acc, st);
  return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
}

int launch_mask_bwd(const dma_shape& s, const void* V, const float* W, const float* A, const float* dz,
                    float* dW, float* dA, void* dV, int accumulate, hipStream_t st) {
  if (!mask_bwd_fits(s)) return DMA_EUNSUPPORTED;  // (before the first launch)
  const size_t nw = (size_t)s.H_q * s.d;
  fill_zero_kernel<<<(unsigned)((nw + 255) / 256), 256, 0, st>>>(dW, nw, dA, (size_t)s.H_q);
  const int G = s.H_q / s.H_kv;
  // The rows kernel's end (sums over its lane groups, then atomics) outweighs its shorter trips while there are few rows
  // and these are short (us at 64 channels, rows / tile kernel: 256 tokens, 2 / 1 heads 10.5 / 7.2; 8192 tokens, 16 / 4
  // heads 17.8 / 16.1; 16384 tokens, 16 / 4 heads 20.1 / 24.8).
  const bool few_rows = s.d == 64 && G > 1 && (long)s.T * s.H_kv <= 32768;
  if (kv_scores_fit(s) && !few_rows) {
    launch_rows<BF16>(s, V, W, A, dz, dW, dA, dV, accumulate, KvAccum{}, st);
    return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
  }
  const int TT = s.d == 256 ? 32 : 64;  // tokens per tile
  const int ntiles = (s.T + TT - 1) / TT;
  // enough workgroups to fill the chip (about four per CU), as few contended atomics as possible
  int tpw = (int)(((long)ntiles * s.H_kv + 1023) / 1024);
  if (tpw < 1) tpw = 1;
  const dim3 grid((ntiles + tpw - 1) / tpw, s.H_kv);
  const size_t sh = mask_bwd_lds_bytes(s);
#define DMA_MB(TV, DD, TTT) \
  mask_bwd_kernel<TV, DD, TTT><<<grid, 256, sh, st>>>((const TV*)V, W, A, dz, dW, dA, (TV*)dV, accumulate, s.T, s.H_q, s.H_kv, tpw)
  if (s.dtype == DMA_BF16) {
    if (s.d == 256) DMA_MB(uint16_t, 256, 32);
    else if (s.d == 128) DMA_MB(uint16_t, 128, 64);
    else DMA_MB(uint16_t, 64, 64);
  } else {
    if (s.d == 256) DMA_MB(float, 256, 32);
    else if (s.d == 128) DMA_MB(float, 128, 64);
    else DMA_MB(float, 64, 64);
  }
#undef DMA_MB
  return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
}

}  // namespace dma
