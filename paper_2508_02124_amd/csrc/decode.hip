// Decode: one new query row per sequence against its whole KV cache (the case with the paper's
// largest speed-ups, Section 5 "Kernel performance").  The row is the last row of its document, so
// its candidates are all n keys of the document; it keeps the min(k, n) best by (z descending,
// index ascending) (Eq. 4), and attends to them with the bias z (Eq. 5-6).  HBM-bound: z is read a
// few times for the selection, then min(k, n) rows of K and V are gathered.
#include "common.h"
#include "select.h"

#include <algorithm>
#include <type_traits>

namespace dma {

struct float8 {
  float4 a, b;
};

// ---- selection of the kept set of one very long sequence, spread over nsl slices of every (sequence,
// q-head) so that it uses the whole chip: four histogram launches (radix select of the kk-th best score, most
// significant byte first, per-pass histograms accumulated in global memory), one counting launch
// and one ordered-compaction launch.  Every workgroup re-derives the digits already fixed from the
// finished histograms (256 counters per pass), so no launch has to hand state to the next one.
struct DecSel {
  const float* z;
  const int32_t* cu;
  const int32_t* lens;  // nullable: current length of each sequence inside its rows [cu[b], cu[b + 1])
  int32_t* kept;
  uint32_t* hist;  // [4][n_docs * H_q][256], zeroed before the first pass
  uint32_t* cnt;   // [n_docs * H_q][nsl][4 waves][2]: keys better than / equal to the threshold
  int T, H_q, k, nsl;
  int split;       // the sliced launches select for sequences longer than this, decode_select_kernel for the others
};

// Wave 0: the digit of `h256` at which the running count reaches `remaining`; updates prefix / remaining.
__device__ __forceinline__ void dec_pick(const uint32_t* h256, int l, uint32_t& prefix, uint32_t& remaining) {
  uint32_t c4[4], sum = 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    c4[i] = h256[4 * l + i];
    sum += c4[i];
  }
  uint32_t inc = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(inc, off);
    if (l >= off) inc += t;
  }
  uint32_t run = inc - sum, dig = 0, rem = 0;
  bool mine = false;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (!mine && run < remaining && remaining <= run + c4[i]) {
      mine = true;
      dig = 4 * l + i;
      rem = remaining - run;
    }
    run += c4[i];
  }
  const unsigned long long m = __ballot(mine);
  const int src = __ffsll((long long)m) - 1;  // exactly one lane finds it (remaining >= 1 and <= total)
  prefix = (prefix << 8) | (uint32_t)__shfl((int)dig, src);
  remaining = (uint32_t)__shfl((int)rem, src);
}

// length of sequence b: all of its rows, or lens[b] of them (clamped to the rows it owns)
__device__ __forceinline__ int dec_len(const int32_t* __restrict__ cu, const int32_t* __restrict__ lens, int b) {
  const int cap = cu[b + 1] - cu[b];
  return lens ? max(0, min(lens[b], cap)) : cap;
}

struct DecSlice {
  int a, n, kk, j0, j1;  // document start / length, kept count, this wave's key range [j0, j1)
};
__device__ __forceinline__ DecSlice dec_slice(const DecSel& p, int b, int sl, int w) {
  DecSlice s;
  s.a = p.cu[b];
  s.n = dec_len(p.cu, p.lens, b);
  s.kk = p.k < s.n ? p.k : s.n;
  const int slen = ((s.n + p.nsl - 1) / p.nsl + 255) / 256 * 256;
  const int wlen = slen / 4;
  s.j0 = min(s.n, sl * slen + w * wlen);
  s.j1 = min(s.n, sl * slen + (w + 1) * wlen);
  return s;
}

// Threshold state after the passes above `pass` (pass = -1: after all four).
__device__ __forceinline__ void dec_state(const DecSel& p, int bh, int nbh, int pass, int kk, int l, uint32_t* sh2) {
  if (threadIdx.x < 64) {
    uint32_t prefix = 0, remaining = (uint32_t)kk;
    for (int q = 3; q > pass; q--) dec_pick(p.hist + ((size_t)q * nbh + bh) * 256, l, prefix, remaining);
    if (l == 0) {
      sh2[0] = prefix;
      sh2[1] = remaining;
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(256) void decode_hist_kernel(DecSel p, int pass) {
  const int bh = blockIdx.x, b = bh / p.H_q, h = bh % p.H_q, sl = blockIdx.y, nbh = gridDim.x;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const DecSlice s = dec_slice(p, b, sl, w);
  if (s.n <= p.split || s.kk == s.n) return;  // (workgroup-uniform)
  // every digit has 32 sub-counters (one per lane pair), so that the lanes of a wave that hit the
  // same digit (scores share their leading bits) do not serialise on one LDS address
  __shared__ uint32_t hist[256 * 32];
  __shared__ uint32_t st[2];
  for (int i = tid; i < 256 * 32; i += 256) hist[i] = 0;
  dec_state(p, bh, nbh, pass, s.kk, l, st);
  const uint32_t prefix = st[0];
  const float* zh = p.z + (size_t)h * p.T + s.a;
  const int sh = 8 * pass;
  for (int j0 = s.j0; j0 < s.j1; j0 += 8 * 64) {  // eight loads in flight per lane
    float zv[8];
#pragma unroll
    for (int u = 0; u < 8; u++) zv[u] = j0 + u * 64 + l < s.j1 ? zh[j0 + u * 64 + l] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const uint32_t key = desc_key(zv[u]);
      if (j0 + u * 64 + l < s.j1 && (pass == 3 || (key >> (sh + 8)) == prefix))
        atomicAdd(&hist[((key >> sh) & 255u) * 32 + (l & 31)], 1u);
    }
  }
  __syncthreads();
  {
    uint32_t c = 0;
    for (int sc = 0; sc < 32; sc++) c += hist[tid * 32 + ((sc + tid) & 31)];
    if (c) atomicAdd(p.hist + ((size_t)pass * nbh + bh) * 256 + tid, c);
  }
}

__global__ __launch_bounds__(256) void decode_count_kernel(DecSel p) {
  const int bh = blockIdx.x, b = bh / p.H_q, h = bh % p.H_q, sl = blockIdx.y, nbh = gridDim.x;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const DecSlice s = dec_slice(p, b, sl, w);
  uint32_t* out = p.cnt + (((size_t)bh * p.nsl + sl) * 4 + w) * 2;
  if (s.n <= p.split) return;
  if (s.kk == s.n) {  // everything is kept
    if (l == 0) {
      out[0] = (uint32_t)(s.j1 - s.j0);
      out[1] = 0;
    }
    return;
  }
  __shared__ uint32_t st[2];
  dec_state(p, bh, nbh, -1, s.kk, l, st);
  const uint32_t thr = st[0];
  const float* zh = p.z + (size_t)h * p.T + s.a;
  uint32_t cb = 0, ce = 0;
  for (int j0 = s.j0; j0 < s.j1; j0 += 8 * 64) {
    float zv[8];
#pragma unroll
    for (int u = 0; u < 8; u++) zv[u] = j0 + u * 64 + l < s.j1 ? zh[j0 + u * 64 + l] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const bool in = j0 + u * 64 + l < s.j1;
      const uint32_t key = desc_key(zv[u]);
      cb += (uint32_t)__popcll(__ballot(in && key < thr));
      ce += (uint32_t)__popcll(__ballot(in && key == thr));
    }
  }
  if (l == 0) {
    out[0] = cb;
    out[1] = ce;
  }
}

// Ordered compaction: keys better than the threshold, and the first need_eq keys equal to it, in
// ascending index order.
__global__ __launch_bounds__(256) void decode_write_kernel(DecSel p) {
  const int bh = blockIdx.x, b = bh / p.H_q, h = bh % p.H_q, sl = blockIdx.y, nbh = gridDim.x;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const DecSlice s = dec_slice(p, b, sl, w);
  if (s.n <= p.split) return;
  const int kcap = p.k < p.T ? p.k : p.T;
  int32_t* list = p.kept + (size_t)bh * kcap;
  __shared__ uint32_t st[2];
  uint32_t thr = 0xffffffffu, need_eq = 0;  // kk == n: every real key is "better"
  if (s.kk < s.n) {
    dec_state(p, bh, nbh, -1, s.kk, l, st);
    thr = st[0];
    need_eq = st[1];
  }
  // better / equal keys before this wave's range: the counts of all earlier (slice, wave) pairs
  uint32_t rb = 0, re = 0;
  {
    const uint32_t* c = p.cnt + (size_t)bh * p.nsl * 8;
    const int npairs = sl * 4 + w;
    for (int i = l; i < npairs; i += 64) {
      rb += c[2 * i];
      re += c[2 * i + 1];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      rb += __shfl_xor(rb, off);
      re += __shfl_xor(re, off);
    }
  }
  const unsigned long long lt = (1ull << l) - 1ull;
  const float* zh = p.z + (size_t)h * p.T + s.a;
  for (int j0 = s.j0; j0 < s.j1; j0 += 8 * 64) {
    float zv[8];
#pragma unroll
    for (int u = 0; u < 8; u++) zv[u] = j0 + u * 64 + l < s.j1 ? zh[j0 + u * 64 + l] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const int j = j0 + u * 64 + l;
      const uint32_t key = desc_key(zv[u]);
      const bool in = j < s.j1;
      const bool better = in && (s.kk == s.n || key < thr), equal = in && s.kk < s.n && key == thr;
      const unsigned long long bm = __ballot(better), em = __ballot(equal);
      const uint32_t eq_before = re + (uint32_t)__popcll(em & lt);  // equal keys with a lower index
      const uint32_t pos = rb + (uint32_t)__popcll(bm & lt) + min(eq_before, need_eq);
      if (better || (equal && eq_before < need_eq)) list[pos] = s.a + j;
      rb += (uint32_t)__popcll(bm);
      re += (uint32_t)__popcll(em);
    }
  }
}

// ---- selection in one launch: one workgroup per (sequence, q-head).  A wave owns a contiguous run of the
// keys and holds it in registers (R per lane; longer sequences are read again from L2 in every pass).  A
// histogram of 2048 equal bins between the sequence's smallest and largest key finds the bin of the kk-th
// best; that bin's keys (few, unless scores are tied) move to LDS, where they are ranked against each other
// -- or, if they are many, counted digit by digit -- for the exact threshold; the kept keys are then
// counted and written in index order.  (SPLIT: sequences longer than p.split are not this kernel's.)  What bounds it is instruction issue on one compute unit (five passes
// over the registers) and, for short sequences, the chain of barriers between the passes.  The sliced launches
// above pay a launch and a pass over z for every one of those links: whole call, us, sliced -> this, k = 2048,
// 32 heads: one cache of 65536 keys 59 -> 45, 24 caches of 5461 keys on average 213 -> 154.  Past the registers
// every pass reads the scores again, 0.11 us per 1000 keys: still issue, not the loads (32 of them in flight
// instead of 8: 93 -> 89 us for 130000 keys).
// Two workgroups share a compute unit where 64 registers hold what they need (R = 16: 79 without the bound, one workgroup,
// and three rounds of 24 x 32 heads), and sums over a wave run in registers.  Whole call, us, 32 heads: 24 caches of 5461 keys
// 128.2 -> 122.4, 24 of 1000 keys, window 500, 41.1 -> 36.1, 16 of 8192, window 4096, 145.7 -> 141.4; one of 65536 38.7 ->
// 38.3.  (Workgroups of 256 or 512 threads: 30 for 24 of 1000 keys, but 8 of 8192 45 -> 52 / 48, and a sequence far
// above the batch's average, which the host does not see, takes two to four times as long.)
template <int R, bool SPLIT>
__global__ __launch_bounds__(1024, R == 16 ? 8 : 4) void decode_select_kernel(DecSel p) {
  constexpr int NT = 1024, NW = NT / 64, REP = 4, BITS = 11, NDIG = 1 << BITS, DPT = NDIG / NT, CAND = 8192, RANK = 512, STEP = 4;
  constexpr uint32_t NONE = 0xffffffffu;  // behind every key
  const int bh = blockIdx.x, b = bh / p.H_q, h = bh % p.H_q;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int a = p.cu[b], n = dec_len(p.cu, p.lens, b);
  if (n <= 0) return;
  if (SPLIT && n > p.split) {  // left to the sliced launches behind this one: their histograms start at zero
    for (int pass = 0; pass < 4; pass++)
      if (tid < 256) p.hist[((size_t)pass * gridDim.x + bh) * 256 + tid] = 0;
    return;
  }
  const int kk = p.k < n ? p.k : n, kcap = p.k < p.T ? p.k : p.T;
  int32_t* list = p.kept + (size_t)bh * kcap;
  if (kk == n) {  // everything is kept
    for (int j = tid; j < n; j += NT) list[j] = a + j;
    return;
  }
  __shared__ __align__(16) uint32_t hist[NDIG * REP];
  __shared__ __align__(16) uint32_t cand[CAND];
  __shared__ uint32_t wsum[NW][2];
  __shared__ uint32_t st[4];  // digit, rank inside it, its count; [3] number of candidates
  const float* zh = p.z + (size_t)h * p.T + a;
  const int wlen = (n + NW * 64 - 1) / (NW * 64) * 64;  // keys per wave
  const int jw = w * wlen, chunks = wlen / 64, own = min(wlen, n - jw);  // (own <= 0: a wave without keys)
  const bool in_regs = chunks <= R;  // (workgroup-uniform)
  auto sort_key = [](float z) { return min(desc_key(z), NONE - 1); };  // (never NONE, whatever z holds)
  uint32_t key[R];
  // f(key, index) for every key of this wave, 64 consecutive ones at a time, ascending; lanes without a key
  // get NONE (in the first pass: another key of the sequence)
  auto each = [&](auto f) {
    if (in_regs) {
      int ch = chunks;
      asm volatile("" : "+s"(ch));  // (comparisons kept from one pass to the next would spill)
#pragma unroll
      for (int u0 = 0; u0 < R; u0 += STEP)
        if (u0 < ch) {
#pragma unroll
          for (int u = u0; u < u0 + STEP; u++) f(key[u], jw + u * 64 + l);
        }
    } else {
      for (int c0 = 0; c0 < chunks; c0 += 8) {
        float zv[8];
#pragma unroll
        for (int u = 0; u < 8; u++) zv[u] = zh[jw + min((c0 + u) * 64 + l, own - 1)];
#pragma unroll
        for (int u = 0; u < 8; u++) {
          const int jl = (c0 + u) * 64 + l;
          f(jl < own ? sort_key(zv[u]) : NONE, jw + jl);
        }
      }
    }
  };
  uint4* hist4 = reinterpret_cast<uint4*>(hist);
  uint32_t kmin = NONE, kmax = 0;
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < R; u++)
      if (u / STEP * STEP < chunks) key[u] = __float_as_uint(zh[jw + min(u * 64 + l, own - 1)]);
  }
#pragma unroll
  for (int i = 0; i < DPT; i++) hist4[NT * i + tid] = make_uint4(0, 0, 0, 0);
  if (tid == 0) st[3] = 0;
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < R; u++)
      if (u / STEP * STEP < chunks) {
        key[u] = sort_key(__uint_as_float(key[u]));
        kmin = min(kmin, key[u]);
        kmax = max(kmax, key[u]);
      }
    if (own < (chunks + STEP - 1) / STEP * STEP * 64) {
#pragma unroll
      for (int u = 0; u < R; u++)
        if (u * 64 + l >= own) key[u] = NONE;
    }
  } else {
    each([&](uint32_t k32, int) {
      kmin = min(kmin, k32);
      kmax = max(kmax, k32 == NONE ? 0u : k32);
    });
  }
  kmin = last_lane(wave_scan(kmin, NONE, [](uint32_t x, uint32_t y) { return min(x, y); }));
  kmax = last_lane(wave_scan(kmax, 0u, [](uint32_t x, uint32_t y) { return max(x, y); }));
  if (l == 0) {
    wsum[w][0] = kmin;
    wsum[w][1] = kmax;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; i++) {
    kmin = min(kmin, wsum[i][0]);
    kmax = max(kmax, wsum[i][1]);
  }
  kmin = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin);
  const uint32_t range = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kmax - kmin));
  const int sh0 = max(0, 32 - (range ? __clz((int)range) : 32) - BITS);  // (key - kmin) >> sh0 < NDIG
  // The digit at which the running count of the histogram reaches `remaining` (st[0..2]); leaves it cleared.
  auto pick = [&](uint32_t remaining) {
    __syncthreads();
    uint32_t c[DPT], sum = 0;  // this thread's digits
#pragma unroll
    for (int i = 0; i < DPT; i++) {
      const uint4 x = hist4[DPT * tid + i];
      hist4[DPT * tid + i] = make_uint4(0, 0, 0, 0);
      c[i] = x.x + x.y + x.z + x.w;
      sum += c[i];
    }
    const uint32_t inc = wave_scan(sum, 0u, [](uint32_t x, uint32_t y) { return x + y; });
    if (l == 63) wsum[w][0] = inc;
    __syncthreads();
    uint32_t run = inc - sum;
#pragma unroll
    for (int i = 0; i < NW; i++) run += i < w ? wsum[i][0] : 0u;
#pragma unroll
    for (int i = 0; i < DPT; i++) {
      if (run < remaining && remaining <= run + c[i]) {  // exactly one digit of one thread
        st[0] = (uint32_t)(DPT * tid + i);
        st[1] = remaining - run;
        st[2] = c[i];
      }
      run += c[i];
    }
    __syncthreads();
  };
  // (lanes without a key count in the last bin, behind every key of it)
  each([&](uint32_t k32, int) {
    atomicAdd(&hist[min((k32 - kmin) >> sh0, (uint32_t)NDIG - 1) * REP + (l & (REP - 1))], 1u);
  });
  pick((uint32_t)kk);
  const uint32_t base = kmin + (st[0] << sh0);  // first key of the bin
  uint32_t need_eq = st[1], n_eq = st[2], sub = 0;
  if (sh0 > 0) {
    const bool listed = n_eq <= CAND;
    uint32_t ncand = 0;
    if (listed) {
      each([&](uint32_t k32, int) {
        const uint32_t x = k32 - base;
        if ((x >> sh0) == 0 && k32 != NONE) cand[atomicAdd(&st[3], 1u)] = x;
      });
      __syncthreads();
      ncand = st[3];
    }
    if (listed && ncand <= RANK) {  // every candidate counts those before it
      if (tid < (int)ncand) {
        const uint32_t x = cand[tid];
        uint32_t less = 0, equal = 0;
        for (uint32_t i = 0; i < ncand; i += 4) {
          const uint4 c = *reinterpret_cast<const uint4*>(&cand[i]);
          const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
          for (int e = 0; e < 4; e++) {
            less += i + e < ncand && cs[e] < x;
            equal += i + e < ncand && cs[e] == x;
          }
        }
        if (less < need_eq && need_eq <= less + equal) {  // (tied candidates write the same values)
          st[0] = x;
          st[1] = need_eq - less;
          st[2] = equal;
        }
      }
      __syncthreads();
      sub = st[0];
      need_eq = st[1];
      n_eq = st[2];
    } else {
      for (int sh = sh0; sh > 0;) {  // (at most 21 bits are left: two rounds)
        const int bits = min(BITS, sh), s2 = sh - bits;
        auto count = [&](uint32_t x) {
          if ((x >> sh) == sub) atomicAdd(&hist[((x >> s2) & ((1u << bits) - 1u)) * REP + (l & (REP - 1))], 1u);
        };
        if (listed) {
          for (uint32_t i = tid; i < ncand; i += NT) count(cand[i]);
        } else {
          uint32_t from = base;
          asm volatile("" : "+v"(from));
          each([&](uint32_t k32, int) {
            if (k32 != NONE) count(k32 - from);  // (keys below the bin wrap round to the far end: never equal to `sub`)
          });
        }
        pick(need_eq);
        sub = (sub << bits) | st[0];
        need_eq = st[1];
        n_eq = st[2];
        sh = s2;
      }
    }
  }
  const uint32_t thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)(base + sub));
  const bool ties = n_eq != need_eq;  // some keys equal to the threshold are left out: those with the highest indices
  uint32_t rb = 0, re = 0;
  if (!ties) {
    each([&](uint32_t k32, int) { rb += (uint32_t)__popcll(__ballot(k32 <= thr)); });
  } else {
    each([&](uint32_t k32, int) {
      rb += (uint32_t)__popcll(__ballot(k32 < thr));
      re += (uint32_t)__popcll(__ballot(k32 == thr));
    });
  }
  if (l == 0) {
    wsum[w][0] = rb;
    wsum[w][1] = re;
  }
  __syncthreads();
  rb = re = 0;
#pragma unroll
  for (int i = 0; i < NW; i++) {  // better / equal keys of the waves before this one
    rb += i < w ? wsum[i][0] : 0u;
    re += i < w ? wsum[i][1] : 0u;
  }
  rb = (uint32_t)__builtin_amdgcn_readfirstlane((int)rb);
  re = (uint32_t)__builtin_amdgcn_readfirstlane((int)re);
  const unsigned long long lt = (1ull << l) - 1ull;
  uint32_t thr_w = thr;
  asm volatile("" : "+s"(thr_w));  // (as above: the masks of the counting pass are formed again)
  if (!ties) {
    each([&](uint32_t k32, int j) {
      const bool keep = k32 <= thr_w;
      const unsigned long long m = __ballot(keep);
      if (keep) list[rb + (uint32_t)__popcll(m & lt)] = a + j;
      rb += (uint32_t)__popcll(m);
    });
  } else {
    each([&](uint32_t k32, int j) {
      const bool better = k32 < thr_w, equal = k32 == thr_w;
      const unsigned long long bm = __ballot(better), em = __ballot(equal);
      const uint32_t eq_before = re + (uint32_t)__popcll(em & lt);  // equal keys with a lower index
      const uint32_t pos = rb + (uint32_t)__popcll(bm & lt) + min(eq_before, need_eq);
      if (better || (equal && eq_before < need_eq)) list[pos] = a + j;
      rb += (uint32_t)__popcll(bm);
      re += (uint32_t)__popcll(em);
    });
  }
}

__global__ void decode_zero_kernel(uint32_t* p, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---- the kept set carried from one decode step to the next (Eq. 4 as a one-in / one-out update):
// `kept` holds the min(k, n - 1) best of the sequence's first n - 1 keys in ascending index order; the
// new key n - 1 joins while fewer than k are kept, otherwise it replaces the worst kept key if it
// beats it (a tie goes to the lower index, and the new key has the highest).  One workgroup per
// (sequence, head); O(k) work instead of a selection over all n scores.  Three dependent memory latencies and a barrier: the
// new key's score is requested first, and the worst key is found in registers (loop of 16 steps over 8 caches of 8192 keys, 32
// heads, 693 -> 686 us).
__global__ __launch_bounds__(256) void decode_update_kernel(const float* __restrict__ z, const int32_t* __restrict__ cu,
                                                            const int32_t* __restrict__ lens, int32_t* kept, int T,
                                                            int H_q, int k) {
  const int bh = blockIdx.x, b = bh / H_q, h = bh % H_q, tid = threadIdx.x, l = tid & 63, w = tid >> 6;
  const int n = dec_len(cu, lens, b);
  if (n <= 0) return;
  const int kcap = k < T ? k : T, kprev = min(k, n - 1), jn = cu[b] + n - 1;
  int32_t* list = kept + (size_t)bh * kcap;
  if (kprev < k) {  // still filling (kprev < kcap: kprev <= n - 1 < T)
    if (tid == 0) list[kprev] = jn;
    return;
  }
  const float* zh = z + (size_t)h * T;
  const float z_new = zh[jn];
  // worst kept key: largest (descending-score key, index).  Lists of up to
  // 8 * 256 entries stay in registers (all loads of a thread in flight together, and the shift below
  // needs no second pass over memory).
  constexpr int UPD_R = 8;
  const bool in_regs = kprev <= UPD_R * 256;
  int ids[UPD_R];
  unsigned long long worst = 0ull;
  int wpos = -1;
  if (in_regs) {
    float zz[UPD_R];
#pragma unroll
    for (int j = 0; j < UPD_R; j++) ids[j] = tid + 256 * j < kprev ? list[tid + 256 * j] : -1;
#pragma unroll
    for (int j = 0; j < UPD_R; j++) zz[j] = ids[j] >= 0 ? zh[ids[j]] : 0.f;
#pragma unroll
    for (int j = 0; j < UPD_R; j++) {
      const unsigned long long c = ((unsigned long long)desc_key(zz[j]) << 32) | (uint32_t)ids[j];
      if (ids[j] >= 0 && c > worst) worst = c;
    }
  } else {
    for (int i = tid; i < kprev; i += 256) {
      const int id = list[i];
      const unsigned long long c = ((unsigned long long)desc_key(zh[id]) << 32) | (uint32_t)id;
      if (wpos < 0 || c > worst) {
        worst = c;
        wpos = i;
      }
    }
  }
  // (a thread without entries has 0, which no other pair is below)
  const auto most = [](uint32_t x, uint32_t y) { return max(x, y); };
  const uint32_t key = (uint32_t)(worst >> 32), wave_key = last_lane(wave_scan(key, 0u, most));
  const uint32_t wave_id = last_lane(wave_scan(key == wave_key ? (uint32_t)worst : 0u, 0u, most));
  __shared__ unsigned long long sw[4];
  if (l == 0) sw[w] = (unsigned long long)wave_key << 32 | wave_id;
  __syncthreads();
  const unsigned long long mine = worst;
#pragma unroll
  for (int i = 0; i < 4; i++) worst = max(worst, sw[i]);
  const unsigned long long cn = ((unsigned long long)desc_key(z_new) << 32) | (uint32_t)jn;
  if (cn > worst) return;  // the new key does not make it (workgroup-uniform)
  if (in_regs) {  // every entry was read before the barrier above: entries behind the worst one move one place down
#pragma unroll
    for (int j = 0; j < UPD_R; j++) {
      const int i = tid + 256 * j;
      if (i > 0 && ids[j] > (int)(uint32_t)worst) list[i - 1] = ids[j];  // (the list ascends)
    }
    if (tid == 0) list[kprev - 1] = jn;
    return;
  }
  __shared__ int drop;
  if (wpos >= 0 && mine == worst) drop = wpos;
  __syncthreads();
  wpos = drop;
  // drop position wpos: entries behind it move one place down, chunk by chunk (a chunk reads before
  // any thread writes, and a later chunk only overwrites what the earlier one has already read)
  for (int i0 = wpos; i0 < kprev - 1; i0 += 256) {
    const int i = i0 + tid;
    int v = 0;
    if (i < kprev - 1) v = list[i + 1];
    __syncthreads();
    if (i < kprev - 1) list[i] = v;
    __syncthreads();
  }
  if (tid == 0) list[kprev - 1] = jn;
}

// Keys per workgroup of the attention pass.
constexpr int DEC_CHUNK = 256;
// Keys that the registers of one selecting workgroup hold: 16 waves x 64 lanes x 64.
constexpr int DEC_SELECT_MAX = 1 << 16;

// (3) single-row attention over one chunk of DEC_CHUNK kept keys: a key row is held by D / 8
// lanes; every lane group keeps its own running (m, l, o) over the keys it visits, the groups are
// merged through LDS, and the chunk's (o, m, l) goes to `part` for decode_merge_kernel.
// HBM-bound: the chunk's key indices and scores are requested in one go and wait in LDS, then U rows of K and
// of V are in flight per lane group.  The G heads of a kv-group have the same chunk of their lists, which covers
// about the same rows, on one XCD at the same time, so rows that several of them keep come from its L2
// (workgroups are dealt to the 8 XCDs in turn; 24 caches of 5461 keys, 32 / 8 heads, k = 2048:
// step of 65536 cached tokens in 8 caches 58 -> 44 us, 24 caches of 5461 keys 154 -> 133 us a call).  A score is summed over its
// lanes in registers (through LDS: one cache of 65536 keys 38.3 -> 37.5 us, 8 of 8192 45.5 -> 44.8).
template <typename TV, int D>
__global__ __launch_bounds__(256) void decode_attend_kernel(const TV* __restrict__ q, const TV* __restrict__ K,
                                                            const TV* __restrict__ V, const float* __restrict__ z,
                                                            const int32_t* __restrict__ cu,
                                                            const int32_t* __restrict__ lens,
                                                            const int32_t* __restrict__ kept, float* part, int T,
                                                            int n_docs, int H_q, int H_kv, int k, int nsplit, float c2) {
  const unsigned wg = blockIdx.y * gridDim.x + blockIdx.x;  // (a second grid dimension only past 2^22 workgroups)
  const int G = H_q / H_kv, x = wg & 7, idx = (int)(wg >> 3);
  const int unit = (idx / G) * 8 + x, sp = unit / (n_docs * H_kv), bg = unit - sp * (n_docs * H_kv);
  if (sp >= nsplit) return;
  const int b = bg / H_kv, g = bg - b * H_kv, h = g * G + idx % G, bh = b * H_q + h;
  const int n = dec_len(cu, lens, b);
  const int kcap = k < T ? k : T, kk = k < n ? k : n;
  const int32_t* list = kept + (size_t)bh * kcap;
  const int i0 = sp * DEC_CHUNK, cnt = min(DEC_CHUNK, kk - i0);
  if (cnt <= 0) return;  // (decode_merge_kernel reads the chunks that hold keys)
  constexpr int LPR = D / 8, NG = 256 / LPR;
  constexpr int U = sizeof(TV) == 2 ? 8 : 4;  // keys in flight per lane group
  const int tid = threadIdx.x, sub = tid % LPR, grp = tid / LPR;
  float* out = part + ((size_t)bh * nsplit + sp) * (D + 2);
  __shared__ int ids[DEC_CHUNK];
  __shared__ float zs[DEC_CHUNK];  // exp2-domain bias of the key; -inf past the end of the list
  {
    const int id = list[i0 + min(tid, cnt - 1)];
    ids[tid] = id;
    zs[tid] = tid < cnt ? z[(size_t)h * T + id] * LOG2E : -INFINITY;
  }
  using Raw = typename std::conditional<sizeof(TV) == 2, uint4, float8>::type;
  auto unpack = [&](const Raw& r, float* o8) {
    if constexpr (sizeof(TV) == 2) {
      const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
      for (int e = 0; e < 4; e++) {
        o8[2 * e] = __uint_as_float(u[e] << 16);
        o8[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
      }
    } else {
      o8[0] = r.a.x; o8[1] = r.a.y; o8[2] = r.a.z; o8[3] = r.a.w;
      o8[4] = r.b.x; o8[5] = r.b.y; o8[6] = r.b.z; o8[7] = r.b.w;
    }
  };
  float qv[8];
  unpack(*reinterpret_cast<const Raw*>(q + ((size_t)b * H_q + h) * D + 8 * sub), qv);
  float m = -INFINITY, lsum = 0.f, acc[8];
#pragma unroll
  for (int e = 0; e < 8; e++) acc[e] = 0.f;
  __syncthreads();
  for (int i = grp; i < cnt; i += NG * U) {
    Raw kr[U], vr[U];
    float s2[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int ii = min(i + u * NG, DEC_CHUNK - 1);  // (past the end of the list: its last key, with bias -inf)
      const size_t off = ((size_t)ids[ii] * H_kv + g) * D + 8 * sub;
      kr[u] = *reinterpret_cast<const Raw*>(K + off);
      vr[u] = *reinterpret_cast<const Raw*>(V + off);
    }
    float m_new = m;
#pragma unroll
    for (int u = 0; u < U; u++) {
      float kv[8], s = 0.f;
      unpack(kr[u], kv);
#pragma unroll
      for (int e = 0; e < 8; e++) s = fmaf(qv[e], kv[e], s);
      s = group_sum<LPR>(s);
      s2[u] = i + u * NG < cnt ? fmaf(s, c2, zs[i + u * NG]) : -INFINITY;  // exp2 domain
      m_new = fmaxf(m_new, s2[u]);
    }
    const float ref = m_new == -INFINITY ? 0.f : m_new;  // (every score of this group so far is -inf)
    const float alpha = fast_exp2(m - ref);
    m = m_new;
    lsum *= alpha;
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] *= alpha;
    if (i - grp + NG * U > cnt) {  // (workgroup-uniform) past the list's end not even an infinite value may count: 0 * inf
#pragma unroll
      for (int u = 0; u < U; u++)
        if (i + u * NG >= cnt) vr[u] = Raw{};
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      float vv[8];
      unpack(vr[u], vv);
      const float pv = fast_exp2(s2[u] - ref);
      lsum += pv;
#pragma unroll
      for (int e = 0; e < 8; e++) acc[e] = fmaf(pv, vv[e], acc[e]);
    }
  }
  __shared__ float mo[NG][D + 2];
#pragma unroll
  for (int e = 0; e < 8; e++) mo[grp][8 * sub + e] = acc[e];
  if (sub == 0) {
    mo[grp][D] = m;
    mo[grp][D + 1] = lsum;
  }
  __syncthreads();
  if (tid < D) {
    float M = -INFINITY;
    for (int gi = 0; gi < NG; gi++) M = fmaxf(M, mo[gi][D]);
    float num = 0.f, den = 0.f;
    for (int gi = 0; gi < NG; gi++) {
      const float w8 = mo[gi][D] == -INFINITY ? 0.f : fast_exp2(mo[gi][D] - M);  // a group that saw no key
      num = fmaf(mo[gi][tid], w8, num);
      den = fmaf(mo[gi][D + 1], w8, den);
    }
    out[tid] = num;  // un-normalised: sum of exp2(s2 - M) v
    if (tid == 0) {
      out[D] = M;
      out[D + 1] = den;
    }
  }
}

// (4) merge the chunks of one (sequence, head): o = sum_c o_c 2^(M_c - M) / sum_c l_c 2^(M_c - M).  Eight chunks
// are requested at a time: the kernel is the latency of its dependent loads.
template <typename TV, int D>
__global__ __launch_bounds__(D) void decode_merge_kernel(const float* __restrict__ part, const int32_t* __restrict__ cu,
                                                         const int32_t* __restrict__ lens, TV* o, float* lse, int H_q,
                                                         int k, int nsplit) {
  const int bh = blockIdx.x, b = bh / H_q, h = bh % H_q, n_docs = gridDim.x / H_q, c = threadIdx.x;
  const int n = dec_len(cu, lens, b);
  TV* orow = o + (size_t)bh * D;
  if (n <= 0) {  // empty sequence: zero output, LSE = -inf
    orow[c] = TV(0.f);
    if (c == 0) lse[(size_t)h * n_docs + b] = -INFINITY;
    return;
  }
  const int kk = k < n ? k : n, ns = (kk + DEC_CHUNK - 1) / DEC_CHUNK;
  const float* p = part + (size_t)bh * nsplit * (D + 2);
  float M = -INFINITY, num = 0.f, den = 0.f;
  for (int s0 = 0; s0 < ns; s0 += 8) {
    float Ms[8], ls[8], os[8];
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const float* ps = p + (size_t)min(s0 + u, ns - 1) * (D + 2);
      Ms[u] = ps[D];
      ls[u] = ps[D + 1];
      os[u] = ps[c];
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < 8; u++) Mn = fmaxf(Mn, Ms[u]);
    const float ref = Mn == -INFINITY ? 0.f : Mn, alpha = fast_exp2(M - ref);
    M = Mn;
    num *= alpha;
    den *= alpha;
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const bool in = s0 + u < ns;  // (past the end the last chunk is read again and counts for nothing, whatever it holds)
      const float w8 = in ? fast_exp2(Ms[u] - ref) : 0.f;
      num = fmaf(in ? os[u] : 0.f, w8, num);
      den = fmaf(ls[u], w8, den);
    }
  }
  orow[c] = TV(num / den);
  if (c == 0) lse[(size_t)h * n_docs + b] = (M + __builtin_amdgcn_logf(den)) * LN2;
}

// slices per (sequence, head) of the selection: enough workgroups for the chip, slices of >= 1024 keys
int decode_nsl(const dma_shape& s) {
  const long nbh = (long)s.n_docs * s.H_q;
  const int longest = s.max_seqlen > 0 && s.max_seqlen < s.T ? s.max_seqlen : s.T;
  long nsl = (1024 + nbh - 1) / nbh;
  const long cap = (longest + 1023) / 1024;
  if (nsl > cap) nsl = cap;
  if (nsl > 64) nsl = 64;
  if (nsl < 1) nsl = 1;
  return (int)nsl;
}

// scratch after the kept lists: per (sequence, head) and chunk, D + 2 floats of partial output;
// then the selection's histograms and slice counts (as 32-bit words)
size_t decode_part_floats(const dma_shape& s) {
  const size_t kcap = (size_t)(s.k < s.T ? s.k : s.T);
  return (size_t)s.n_docs * s.H_q * ((kcap + DEC_CHUNK - 1) / DEC_CHUNK) * (s.d + 2);
}
size_t decode_sel_words(const dma_shape& s) {
  const size_t nbh = (size_t)s.n_docs * s.H_q;
  return 4 * nbh * 256 + nbh * (size_t)decode_nsl(s) * 8;
}

template <typename TV, int D>
static void launch_decode_t(const dma_shape& s, float c2, const void* q, const void* K, const void* V, const float* z,
                            const int32_t* cu, const int32_t* lens, void* o, float* lse, int32_t* kept, float* part,
                            int nsplit, hipStream_t st) {
  const int nbh = s.n_docs * s.H_q;
  const long wgs = ((long)s.n_docs * s.H_kv * nsplit + 7) / 8 * 8 * (s.H_q / s.H_kv), gx = wgs < (1l << 22) ? wgs : 1l << 22;
  decode_attend_kernel<TV, D><<<dim3((unsigned)gx, (unsigned)((wgs + gx - 1) / gx)), 256, 0, st>>>(
      (const TV*)q, (const TV*)K, (const TV*)V, z, cu, lens, kept, part, s.T, s.n_docs, s.H_q, s.H_kv, s.k, nsplit, c2);
  decode_merge_kernel<TV, D><<<nbh, D, 0, st>>>(part, cu, lens, (TV*)o, lse, s.H_q, s.k, nsplit);
}

// incremental == 0: the kept sets are selected from all scores; otherwise they are carried over from
// the previous step and updated with the newest key of every sequence.
// Scratch of dma_decode_static: the per-chunk partial outputs and the selection's histograms and
// counts of one call, held in the library's own device memory (every GPU the library runs on keeps
// its copy until the process ends).  Host code never passes the array's name to a kernel: the
// device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[DMA_DECODE_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[64] = {};

size_t decode_scratch_bytes(const dma_shape& s) {
  return align_up(decode_part_floats(s) * 4, 256) + align_up(decode_sel_words(s) * 4, 256);
}

int decode_static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DMA_EHIP;
  void* ptr = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return DMA_EHIP;
    __atomic_store_n(&g_scratch_ptr[dev], ptr, __ATOMIC_RELEASE);  // (two first callers store the same address)
  }
  *out = ptr;
  return DMA_OK;
}

// part_and_sel: the scratch region (decode_scratch_bytes): partial outputs, then histograms and counts
int launch_decode(const dma_shape& s, float scale, const void* q, const void* K, const void* V, const float* z,
                  const int32_t* cu, const int32_t* lens, int incremental, void* o, float* lse, int32_t* kept,
                  void* part_and_sel, hipStream_t st) {
  const float c2 = scale * LOG2E;
  const size_t kcap = (size_t)(s.k < s.T ? s.k : s.T);
  const int nsplit = (int)((kcap + DEC_CHUNK - 1) / DEC_CHUNK);
  float* part = reinterpret_cast<float*>(part_and_sel);
  const int nbh = s.n_docs * s.H_q;
  DecSel ds;
  ds.z = z; ds.cu = cu; ds.lens = lens; ds.kept = kept;
  ds.hist = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(part) + align_up(decode_part_floats(s) * 4, 256));
  ds.cnt = ds.hist + 4 * (size_t)nbh * 256;
  ds.T = s.T; ds.H_q = s.H_q; ds.k = s.k; ds.nsl = decode_nsl(s);
  if (incremental) {
    decode_update_kernel<<<nbh, 256, 0, st>>>(z, cu, lens, kept, s.T, s.H_q, s.k);
  } else {
    // One workgroup per (sequence, head) selects alone while its keys fit its registers; the host sees only the
    // caches' total, so a batch is taken at twice its average length.  A sequence that is longer than the registers
    // all the same (where the caller's bound, or without one the total, allows it) is left to the sliced launches if
    // each head has many slices there, 12 or more: at 8 they are slower than one workgroup that reads L2 again (whole
    // call, us, k = 2048, one workgroup / sliced: 130000 and three times 300 keys, 32 heads 98 / 135, 16 heads 94 / 88,
    // 2 heads 90 / 47; 290000 and nine times 500 keys, 8 heads 182 / 149).  Without a bound, an even batch of few heads
    // pays for launches that find nothing to do: eight times 16000 keys, 8 heads 28 -> 38 us (all sliced: 59).
    const long longest = s.max_seqlen > 0 && s.max_seqlen < s.T ? s.max_seqlen : s.T;
    const long typical = std::min(longest, (2l * s.T + s.n_docs - 1) / s.n_docs);
    const bool all_sliced = typical > DEC_SELECT_MAX && ds.nsl > 1;
    const bool long_sliced = !all_sliced && longest > DEC_SELECT_MAX && ds.nsl >= 12;
    ds.split = all_sliced ? 0 : DEC_SELECT_MAX;
    if (all_sliced) {
      const size_t nz = 4 * (size_t)nbh * 256;
      decode_zero_kernel<<<(unsigned)((nz + 255) / 256), 256, 0, st>>>(ds.hist, nz);
    } else if (long_sliced) {
      if (typical > 16 * 1024) decode_select_kernel<64, true><<<nbh, 1024, 0, st>>>(ds);
      else decode_select_kernel<16, true><<<nbh, 1024, 0, st>>>(ds);
    } else {
      if (typical > 16 * 1024) decode_select_kernel<64, false><<<nbh, 1024, 0, st>>>(ds);
      else decode_select_kernel<16, false><<<nbh, 1024, 0, st>>>(ds);
    }
    if (all_sliced || long_sliced) {
      const dim3 sgrid(nbh, ds.nsl);
      for (int pass = 3; pass >= 0; pass--) decode_hist_kernel<<<sgrid, 256, 0, st>>>(ds, pass);
      decode_count_kernel<<<sgrid, 256, 0, st>>>(ds);
      decode_write_kernel<<<sgrid, 256, 0, st>>>(ds);
    }
  }
  if (s.dtype == DMA_BF16) {
    if (s.d == 256) launch_decode_t<__bf16, 256>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
    else if (s.d == 128) launch_decode_t<__bf16, 128>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
    else launch_decode_t<__bf16, 64>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
  } else {
    if (s.d == 256) launch_decode_t<float, 256>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
    else if (s.d == 128) launch_decode_t<float, 128>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
    else launch_decode_t<float, 64>(s, c2, q, K, V, z, cu, lens, o, lse, kept, part, nsplit, st);
  }
  return hipGetLastError() == hipSuccess ? DMA_OK : DMA_EHIP;
}

}  // namespace dma
