// Causal top-k selection (Eq. 4): which key each row evicts.
//
// While a document has more than k rows, every row admits at most one key and evicts the weakest resident, under
// (score descending, index ascending).  evict_kernel writes parent[i] = the key that row i evicts (-1: none, -2: row i's
// own key never enters) and the expiries of keys that no row evicts; the slot kernels add the others.
//
// A block of BQ rows is worked out by itself, from the scores before it: at most BQ residents are evicted inside it, and
// these are among the weakest of the residents at its first row.  A histogram of the scores before the block (Bins,
// select_bins.h) gives the bin of the k-th best and with it how many keys of the block can enter (e); the keys between the
// bins of rank k - e and k, grouped by bin, are ranked against their bin.  A key x then leaves at the row where the c-th of
// the block's keys ranked ahead of x appears, c = the places left behind the residents ahead of x.  Everything is comparison
// of (score bits, index), so the result is the exact kept set.
// Where the bins do not separate the scores (ties, outliers, infinities) the two ranks are narrowed down together, BIN_BITS of
// (score bits, index) at a time.
//
// Long documents: reading everything before every block grows with the square of the length, so checkpoint_kernel
// leaves, every CK_SEG keys, the weakest CK_SEG of the residents (no more can be evicted before the next one), and a
// block reads these and the keys since.
#include "select.h"

namespace dma {

constexpr int RUN = 4;      // keys compared at a time
constexpr int NARROW = 32;  // keys beside a rank that is narrowed down

__device__ __forceinline__ uint64_t ranked(uint32_t key, int i) { return (uint64_t)key << 32 | (uint32_t)i; }

// The scores before a block: m0 of a checkpoint's list (their indices in the document beside them), then nz of the document
// from index c on, both in whole fours.  Threads take four at a time, the first NQ quads of a thread in registers, the others
// read again in every pass.
struct __attribute__((aligned(4))) Quad {  // (16 bytes at 4-byte alignment)
  float v[4];
};
template <int NT, int NQ>
struct Scores {
  const float *list, *z;
  const int32_t* list_idx;
  int c, nq, list_q;
  Quad r[NQ ? NQ : 1];
  __device__ __forceinline__ Quad quad(int t) const {
    Quad q = {};
    if (t < nq) q = *reinterpret_cast<const Quad*>(t < list_q ? list + 4 * t : z + 4 * (t - list_q));
    return q;
  }
  __device__ __forceinline__ void load(const float* list_, const int32_t* list_idx_, int m0, const float* z_, int nz, int c_) {
    list = list_; list_idx = list_idx_; z = z_; c = c_;
    list_q = m0 / 4;
    nq = list_q + nz / 4;
#pragma unroll
    for (int j = 0; j < NQ; j++) {
      r[j] = Quad{};
      if (NT * j < nq) r[j] = quad((int)threadIdx.x + NT * j);
    }
  }
  // index in the document of element e of quad t
  __device__ __forceinline__ int index(int t, int e) const {
    return t < list_q ? list_idx[4 * t + e] : c + 4 * (t - list_q) + e;
  }
  // one of the scores for every thread, over all of them
  __device__ __forceinline__ float sample() const {
    const int i = (int)((uint32_t)(4 * nq) * threadIdx.x / NT);
    return i < 4 * list_q ? list[i] : z[i - 4 * list_q];
  }
  // f(quad, t) for every quad, f(score, t, e) for every element
  template <typename F> __device__ __forceinline__ void each_quad(F&& f) const {
#pragma unroll
    for (int j = 0; j < NQ; j++)
      if (NT * j < nq) {
        const int t = (int)threadIdx.x + NT * j;
        if (t < nq) f(r[j], t);
      }
    quads_again<4>(f, NQ);
  }
  template <int U, typename F> __device__ __forceinline__ void quads_again(F&& f, int j) const {  // U quads in flight
#pragma unroll 1
    for (; NT * j < nq; j += U) {
      Quad q[U];
#pragma unroll
      for (int u = 0; u < U; u++) q[u] = quad((int)threadIdx.x + NT * (j + u));
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int t = (int)threadIdx.x + NT * (j + u);
        if (t < nq) f(q[u], t);
      }
    }
  }
  template <typename F> __device__ __forceinline__ void each(F&& f) const {
    each_quad([&](const Quad& q, int t) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; e++) f(q.v[e], t, e);
    });
  }
  template <typename F> __device__ __forceinline__ void each_again(F&& f) const {  // (where registers are short: two quads)
    quads_again<2>([&](const Quad& q, int t) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; e++) f(q.v[e], t, e);
    }, 0);
  }
};

template <int NT> struct SelShared {
  static constexpr int NW = NT / 64;
  __align__(16) uint64_t cand[CAP + RUN];
  uint32_t wsum[NW];
  uint32_t kmin[NW], kmax[NW];
  uint32_t bin[2], before[2], count[2];
  int fill;
};

// Lane LANE of lo and hi takes a ballot.  The comparison that forms the ballot writes a scalar register, which a vector
// instruction may read as data two wait states later; the compiler keeps this for its own instructions only, so the wait is
// part of the statement.
template <int LANE> __device__ __forceinline__ void write_lane(int& lo, int& hi, uint64_t ballot) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi) : "s"((uint32_t)ballot), "s"((uint32_t)(ballot >> 32)), "n"(LANE));
}

// Exclusive prefix sums of a histogram, in place; seen(bin, count before it, count in it) for every bin.
template <int BITS, int NT, typename F>
__device__ __forceinline__ void scan_bins(SelShared<NT>& sm, uint32_t* hist, F&& seen) {
  constexpr int PER = (1 << BITS) / NT, NW = NT / 64;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  uint32_t v[PER], s = 0;
#pragma unroll
  for (int i = 0; i < PER; i++) {
    v[i] = hist[PER * tid + i];
    s += v[i];
  }
  const uint32_t inc = wave_scan(s, 0, [](uint32_t x, uint32_t y) { return x + y; });
  if (l == 63) sm.wsum[w] = inc;
  __syncthreads();
  uint32_t ex = inc - s;
#pragma unroll
  for (int i = 0; i < NW; i++) ex += i < w ? sm.wsum[i] : 0u;
#pragma unroll
  for (int i = 0; i < PER; i++) {
    hist[PER * tid + i] = ex;
    seen(PER * tid + i, ex, v[i]);
    ex += v[i];
  }
  __syncthreads();
}
// The bin that holds a rank, with the counts before and in it, to place `at`.
template <int NT> __device__ __forceinline__ void note_bin(SelShared<NT>& sm, int at, uint32_t rank, int bin, uint32_t before, uint32_t count) {
  if (rank - before < count) { sm.bin[at] = bin; sm.before[at] = before; sm.count[at] = count; }
}

template <int BITS, int NT> __device__ __forceinline__ void clear_bins(uint32_t* hist) {
  for (int i = threadIdx.x; i < (1 << BITS) / 4; i += NT) reinterpret_cast<uint4*>(hist)[i] = make_uint4(0, 0, 0, 0);
}

// Smallest kmin and largest kmax of all threads.
template <int NT> __device__ __forceinline__ void reduce_range(SelShared<NT>& sm, uint32_t& kmin, uint32_t& kmax) {
  kmin = last_lane(wave_scan(kmin, 0xffffffffu, [](uint32_t x, uint32_t y) { return min(x, y); }));
  kmax = last_lane(wave_scan(kmax, 0u, [](uint32_t x, uint32_t y) { return max(x, y); }));
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sm.kmin[w] = kmin;
    sm.kmax[w] = kmax;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NT / 64; i++) {
    kmin = min(kmin, sm.kmin[i]);
    kmax = max(kmax, sm.kmax[i]);
  }
}
// Best and worst key of a score per thread; zeros and infinities apart (kmin > kmax: there are no others).
template <int NT>
__device__ __forceinline__ void sample_range(SelShared<NT>& sm, float sample, uint32_t& kmin, uint32_t& kmax) {
  const bool takes = sample != 0.f && fabsf(sample) < __builtin_inff();
  kmin = takes ? desc_key(sample) : 0xffffffffu;
  kmax = takes ? desc_key(sample) : 0u;
  reduce_range(sm, kmin, kmax);
}
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// A rank among the scores, and how far it is known: the key with this rank is one of the `count` keys from base to last, with
// `before` keys before these.  Keys are (score, index) as key << ibits | index here.
struct Window {
  uint64_t base, last;
  uint32_t rank, before, count;
  __device__ __forceinline__ void init(uint32_t key0, uint64_t key1, int ibits, uint32_t rank_, uint32_t before_, uint32_t count_) {
    span(key0, key1, ibits);
    rank = uniform(rank_); before = uniform(before_); count = uniform(count_);
  }
  __device__ __forceinline__ void span(uint32_t key0, uint64_t key1, int ibits) {
    base = (uint64_t)uniform(key0) << ibits;
    last = (((uint64_t)uniform((uint32_t)(key1 - 1)) + 1) << ibits) - 1;
  }
  template <int BITS> __device__ __forceinline__ int shift() const {
    return max(0, 64 - (int)__clzll((long long)(last - base)) - BITS);
  }
  template <int NT> __device__ __forceinline__ void take(const SelShared<NT>& sm, int at, int shift) {
    const uint32_t ahead = uniform(sm.before[at]);
    base += (uint64_t)uniform(sm.bin[at]) << shift;
    last = base + ((1ull << shift) - 1);
    before += ahead;
    rank -= ahead;
    count = uniform(sm.count[at]);
  }
  __device__ __forceinline__ bool holds(uint64_t c) const { return c >= base && c <= last; }
};
__device__ __forceinline__ uint64_t composite(uint32_t key, int i, int ibits) { return (uint64_t)key << ibits | (uint32_t)i; }
// (with ties the lanes mostly agree: one addition for all that agree with the first)
template <int BITS> __device__ __forceinline__ void count_agreeing(uint32_t* hist, uint64_t bin) {
  if (bin >> BITS) return;
  const uint32_t b = (uint32_t)bin, b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
  const uint64_t same = __ballot(b == b0);
  if (b != b0) atomicAdd(&hist[b], 1u);
  else if ((same & ((1ull << (threadIdx.x & 63)) - 1ull)) == 0) atomicAdd(&hist[b], (uint32_t)__popcll(same));
}
// The histogram of all scores; true if one of the thread's is not a number.  Each wave looks at one per lane first: where many lanes
// agree, additions to one counter would wait for each other (evict_kernel, 16384 x 32, nearly all scores in one bin: 166 -> 119
// us).  CUT: without what is behind the bins' range.
template <bool CUT, int BITS, int NT, int NQ>
__device__ __forceinline__ bool count_all(uint32_t* hist, const Scores<NT, NQ>& s, const Bins<BITS>& bins, float sample) {
  if (NQ > 0) sample = s.r[0].v[0];  // (with its neighbours, whose order may be that of the scores)
  const uint32_t b = bins.of(sample);
  bool bad = false;
  if (__popcll(__ballot(b == (uint32_t)__builtin_amdgcn_readfirstlane((int)b) && !(CUT && bins.behind(sample)))) < 16)
    s.each([&](float z, int, int) {
      bad |= z != z;
      if (!CUT || !bins.behind(z)) atomicAdd(&hist[bins.of(z)], 1u);
    });
  else
    s.each_again([&](float z, int, int) {
      bad |= z != z;
      if (!CUT || !bins.behind(z)) count_agreeing<BITS>(hist, bins.of(z));
    });
  return bad;
}
// The windows of two ranks that are known to their bins.
template <int BITS>
__device__ __forceinline__ void windows_of_bins(const Bins<BITS>& bins, bool cut, int bin0, int bin1, int ibits, uint32_t rank0, uint32_t before0,
                                                uint32_t count0, uint32_t rank1, uint32_t before1, uint32_t count1, Window& w0,
                                                Window& w1) {
  const int l = threadIdx.x & 63;
  const int ends = (int)bins.bound((uint32_t)((l & 2 ? bin1 : bin0) + (l & 1)), cut);  // lanes 0 to 3
  const auto end = [&](int lane) { return (uint32_t)__builtin_amdgcn_readlane(ends, lane); };
  w0.init(end(0), end(1), ibits, rank0 - before0, before0, count0);
  w1.init(end(2), end(3), ibits, rank1 - before1, before1, count1);
}
// Limits two windows to the scores that there are.
template <int NT, int NQ>
__device__ __forceinline__ void tighten(SelShared<NT>& sm, const Scores<NT, NQ>& s, int ibits, Window& w0, Window& w1) {
  const uint32_t a0 = (uint32_t)(w0.base >> ibits), b0 = (uint32_t)(w0.last >> ibits);
  const uint32_t a1 = (uint32_t)(w1.base >> ibits), b1 = (uint32_t)(w1.last >> ibits);
  uint32_t min0 = 0xffffffffu, max0 = 0, min1 = 0xffffffffu, max1 = 0;
  s.each_again([&](float z, int, int) {
    const uint32_t key = desc_key(z);
    const bool in0 = key >= a0 && key <= b0, in1 = key >= a1 && key <= b1;
    min0 = min(min0, in0 ? key : 0xffffffffu);
    max0 = max(max0, in0 ? key : 0u);
    min1 = min(min1, in1 ? key : 0xffffffffu);
    max1 = max(max1, in1 ? key : 0u);
  });
  __syncthreads();
  reduce_range(sm, min0, max0);
  __syncthreads();
  reduce_range(sm, min1, max1);
  if (w0.count > 0) w0.span(min0, (uint64_t)max0 + 1, ibits);
  if (w1.count > 0) w1.span(min1, (uint64_t)max1 + 1, ibits);
}
// Narrows two windows until neither holds more than `limit` keys, both in the same passes over the scores, BITS of what is left at
// a time (with ties, of the indices alone: tighten has left one score).  Scores of sixteen different values, whole dma_mask_gen, us, a
// sort / a search of its own for each rank / this: 16384 x 32 114 / 169 / 117, packed 65536 x 16 157 / 117 / 104, 65536 x 32, window
// 16384, 487 / 637 / 548.
template <int BITS, int NT, int NQ>
__device__ __forceinline__ void narrow(SelShared<NT>& sm, uint32_t* hist0, uint32_t* hist1, const Scores<NT, NQ>& s, int ibits,
                                       Window& w0, Window& w1, uint32_t limit) {
#pragma unroll 1
  for (;;) {
    const bool go0 = w0.count > limit && w0.base < w0.last, go1 = w1.count > limit && w1.base < w1.last;
    const bool one = go0 && go1 && w0.base == w1.base && w0.last == w1.last;
    if (!go0 && !go1) return;
    const int shift0 = w0.shift<BITS>(), shift1 = w1.shift<BITS>();
    __syncthreads();
    clear_bins<BITS, NT>(hist0);
    clear_bins<BITS, NT>(hist1);
    __syncthreads();
    s.each_again([&](float z, int t, int e) {
      const uint64_t c = composite(desc_key(z), s.index(t, e), ibits);
      if (go0) count_agreeing<BITS>(hist0, (c - w0.base) >> shift0);
      if (go1 && !one) count_agreeing<BITS>(hist1, (c - w1.base) >> shift1);
    });
    __syncthreads();
    if (go0)
      scan_bins<BITS>(sm, hist0, [&](int bin, uint32_t before, uint32_t count) {
        note_bin(sm, 0, w0.rank, bin, before, count);
        if (one) note_bin(sm, 1, w1.rank, bin, before, count);
      });
    if (go1 && !one)
      scan_bins<BITS>(sm, hist1, [&](int bin, uint32_t before, uint32_t count) { note_bin(sm, 1, w1.rank, bin, before, count); });
    if (go0) w0.take(sm, 0, shift0);
    if (go1) w1.take(sm, 1, shift1);
  }
}

// ------------------------------------------------------------------ checkpoints
// One workgroup per (checkpoint, head).
// What bounds it: instruction issue over the N scores, three passes of loads of 16 bytes per lane: 65536 tokens x
// 32 heads 43 us (window 16384: 52).
constexpr int CK_NT = 1024, CK_NQ = 0;
__global__ __launch_bounds__(CK_NT, 8) void checkpoint_kernel(SelectArgs p) {
  __shared__ SelShared<CK_NT> sm;
  __shared__ __align__(16) uint32_t hist[1 << CK_BIN_BITS], exact_hist[1 << CK_BIN_BITS];
  __shared__ uint64_t cand1[CAP], found[2];
  __shared__ int fill[2];
  const int slot = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int d = piece_doc<CK_SEG>(p.cu, p.n_docs, slot);
  const int a = p.cu[d], n = p.cu[d + 1] - a;
  const int c = CK_SEG * (slot - piece_slot<CK_SEG>(a, d, 0) + 1);
  if (n <= p.ck_min || n <= p.k || c >= n) return;
  Scores<CK_NT, CK_NQ> s;
  s.load(p.z, p.ck_idx, 0, p.z + (size_t)h * p.T + a, c, 0);
  const int m0 = ck_keys(p.k), kept = max(m0, min(p.k, c));
  uint64_t from = 0, to = ~0ull;  // the weakest m0 of the kept: ranks kept - m0 .. kept - 1
  if (kept < c || m0 < kept) {
    uint32_t kmin, kmax;
    const float sample = s.sample();
    clear_bins<CK_BIN_BITS, CK_NT>(hist);
    sample_range(sm, sample, kmin, kmax);
    Bins<CK_BIN_BITS> bins;
    bins.init(kmin, kmax);
    const uint32_t rank0 = kept - m0, rank1 = kept - 1;
    const bool cut0 = rank0 > 0, cut1 = kept < c;  // (otherwise nothing is left out on that side)
    if (bins.ok) {
      bins.ok = !__syncthreads_or(count_all<false>(hist, s, bins, sample));
      scan_bins<CK_BIN_BITS>(sm, hist, [&](int bin, uint32_t before, uint32_t count) {
        note_bin(sm, 0, rank0, bin, before, count);
        note_bin(sm, 1, rank1, bin, before, count);
      });
    }
    const uint32_t bin0 = sm.bin[0], before0 = sm.before[0], count0 = sm.count[0];
    const uint32_t bin1 = sm.bin[1], before1 = sm.before[1], count1 = sm.count[1];
    const int ibits = 32 - __clz(n);
    const bool by_bin = bins.ok && !(cut0 && count0 > CAP) && !(cut1 && count1 > CAP);
    Window w0 = {0, 0, rank0, before0, count0}, w1 = {0, 0, rank1, before1, count1};
    if (!by_bin) {
      if (bins.ok) {
        windows_of_bins(bins, false, bin0, bin1, ibits, rank0, before0, cut0 ? count0 : 0, rank1, before1, cut1 ? count1 : 0, w0, w1);
      } else {
        w0.init(0, 1ull << 32, ibits, rank0, 0, cut0 ? c : 0);
        w1.init(0, 1ull << 32, ibits, rank1, 0, cut1 ? c : 0);
      }
      tighten(sm, s, ibits, w0, w1);
      narrow<CK_BIN_BITS>(sm, hist, exact_hist, s, ibits, w0, w1, CAP);
    }
    __syncthreads();
    if (tid < 2) fill[tid] = 0;
    __syncthreads();
    if (by_bin) {
      s.each([&](float z, int t, int e) {
        const uint32_t b = bins.of(z);
        if (b == bin0 && cut0) sm.cand[atomicAdd(&fill[0], 1)] = ranked(desc_key(z), s.index(t, e));
        if (b == bin1 && cut1) cand1[atomicAdd(&fill[1], 1)] = ranked(desc_key(z), s.index(t, e));
      });
    } else {
      s.each_again([&](float z, int t, int e) {
        const int i = s.index(t, e);
        const uint64_t c2 = composite(desc_key(z), i, ibits);
        if (cut0 && w0.holds(c2)) sm.cand[atomicAdd(&fill[0], 1)] = ranked(desc_key(z), i);
        if (cut1 && w1.holds(c2)) cand1[atomicAdd(&fill[1], 1)] = ranked(desc_key(z), i);
      });
    }
    __syncthreads();
    const auto find = [&](const uint64_t* cand, uint32_t count, uint32_t rank, uint64_t& found) __attribute__((always_inline)) {
      if (tid >= (int)count) return;
      const uint64_t mine = cand[tid];
      uint32_t ahead = 0;
      for (uint32_t j = 0; j < count; j++) ahead += cand[j] < mine;
      if (ahead == rank) found = mine;
    };
    if (cut0) find(sm.cand, w0.count, rank0 - w0.before, found[0]);
    if (cut1) find(cand1, w1.count, rank1 - w1.before, found[1]);
    __syncthreads();
    if (cut0) from = found[0];
    if (cut1) to = found[1];
  }
  const size_t out = (size_t)h * p.T + a + (c - CK_SEG);
  __syncthreads();
  if (tid == 0) fill[0] = kept < c ? 1 : 0;
  __syncthreads();
  s.each([&](float z, int t, int e) {
    const int i = s.index(t, e);
    const uint64_t r = ranked(desc_key(z), i);
    if (r >= from && r <= to) {
      const int at = r == to ? 0 : atomicAdd(&fill[0], 1);  // (the last kept key stands first)
      p.ck_z[out + at] = z;
      p.ck_idx[out + at] = i;
    }
  });
}

// ------------------------------------------------------------------ evictions of one block
// One workgroup per (block, head).  What bounds it: instruction issue; its twelve short phases between barriers take about 14000
// cycles with 1024 older scores (what a score costs is about 15 instructions in all).  (Registers for eight workgroups per compute unit
// instead of seven: 65536 x 32 of window 1024 50 -> 48 us, 16384 x 32 31 -> 33.)
// Whole selection, us, against a radix sort and wavelet matrix per 4096 or 16384 keys and a range query per key: 256
// tokens x 2 heads 25 -> 7, 2 x 4096 x 16 52 -> 12, 16384 x 32 76 -> 29, packed 65536 x 16 121 -> 32, 65536 x 32 of
// window 1024 241 -> 94.
template <int NT, int NQ>
__global__ __launch_bounds__(NT, 7) void evict_kernel(SelectArgs p) {
  constexpr int NW = NT / 64, BINS = 1 << BIN_BITS;
  constexpr int XT = (CAP + BQ + NT - 1) / NT;  // keys ranked per thread
  static_assert(NT >= BQ, "one thread per row of the block");
  __shared__ SelShared<NT> sm;
  __shared__ __align__(16) uint32_t hists[2 * BINS];  // of the older scores, of those of the block that can enter; then the sets below
  uint32_t *const hist = hists, *const new_hist = hists + BINS;
  __shared__ __align__(16) uint64_t newc[BQ];      // the block's keys that can enter, in index order
  __shared__ __align__(16) uint64_t new_run[BQ + RUN];  // ... grouped by bin
  __shared__ int new_rank[BQ];                     // ... how many of them are ahead of each
  __shared__ int out[BQ];
  const int bi = p.nblk_cap - 1 - (int)blockIdx.x, h = blockIdx.y;  // long prefixes first
  const int4 info = p.blk[bi];
  if (info.x < 0) return;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int a = info.w, lo = info.y - a, nb = info.z - info.y, n = p.cu[info.x + 1] - a, k = p.k;
  int32_t* par = p.parent + (size_t)h * p.T + info.y;
  int32_t* ex = p.expiry + (size_t)h * p.T + info.y;
  auto store = [&](int evicted) __attribute__((always_inline)) {
    if (tid < nb) {
      par[tid] = evicted;
      ex[tid] = evicted == -2 ? info.y + tid : a + n;
    }
  };
  if (n <= k || lo + nb <= k) {  // nothing is evicted here
    store(-1);
    return;
  }
  const float* zd = p.z + (size_t)h * p.T + a;
  int c = 0, m0 = 0, cap = k;  // list of the last checkpoint, if there is one; places for its keys and those since
  if (n > p.ck_min && lo >= CK_SEG) {
    c = lo & ~(CK_SEG - 1);
    m0 = ck_keys(k);
    cap = k - max(0, min(k, c) - m0);
  }
  const int N = m0 + lo - c, kept = min(cap, N);
  const size_t ck = m0 ? (size_t)h * p.T + a + (c - CK_SEG) : 0;
  const float zn = zd[lo + min(tid, nb - 1)];
  const uint32_t kn = desc_key(zn);
  Scores<NT, NQ> s;
  s.load(p.ck_z + ck, p.ck_idx + ck, m0, zd + c, lo - c, c);

  // Which older keys take part (nl of them, in sm.cand), how many residents are ahead of all of these, and which of the
  // block's keys can enter.
  int strong = 0, nl = 0;
  bool enters = tid < nb;
  int b1 = BINS - 1, b2 = 0;     // bins of the last resident and of the first that takes part
  int end_before = 0, end = N;   // keys before b1 and up to its end
  int first = 0;  // rank of the first that takes part
  Bins<BIN_BITS> bins;
  clear_bins<BIN_BITS, NT>(hist);
  clear_bins<BIN_BITS, NT>(new_hist);
  if (tid == 0) sm.bin[1] = sm.before[1] = 0;  // (what is left without older keys)
  // (a full checkpoint: what is behind its last key is not kept, nor counted; the bins end there)
  const bool full = m0 > 0 && c > max(m0, k);
  const uint32_t worst = full ? desc_key(s.list[0]) : 0;
  const float sample = N > 0 ? s.sample() : zn;
  uint32_t kmin, kmax;
  sample_range(sm, sample, kmin, kmax);
  bins.init(kmin, full ? worst : kmax);
  bool by_bin = bins.ok;
  // the bin of a rank among the older keys, and the count before it
  auto find_bin = [&](int rank) __attribute__((always_inline)) {
    constexpr int PER = BINS / NT;
    int begin[PER + 1];
#pragma unroll
    for (int i = 0; i < PER; i++) begin[i] = hist[PER * tid + i];
    begin[PER] = tid + 1 < NT ? (int)hist[PER * (tid + 1)] : N;
#pragma unroll
    for (int i = 0; i < PER; i++)
      if (begin[i] <= rank && rank < begin[i + 1]) {
        sm.bin[1] = PER * tid + i;
        sm.before[1] = begin[i];
        sm.count[1] = begin[i + 1] - begin[i];
      }
    __syncthreads();
  };
  if (by_bin) {
    bool bad = zn != zn;
    if (full) bad |= count_all<true>(hist, s, bins, sample);
    else bad |= count_all<false>(hist, s, bins, sample);
    by_bin = bins.ok = !__syncthreads_or(bad);
  }
  if (by_bin) {
    const int bn = bins.of(zn);
    scan_bins<BIN_BITS>(sm, hist, [&](int bin, uint32_t before, uint32_t count) {
      note_bin(sm, 0, (uint32_t)(kept - 1), bin, before, count);
    });
    // (kept == N: every older key is still there, whatever its rank)
    if (kept < N) {
      b1 = sm.bin[0];
      end_before = sm.before[0];
      end = end_before + sm.count[0];
    }
    enters = tid < nb && bn <= b1 && (!full || kn < worst);
    const int e = __syncthreads_count(enters);
    if (e == 0) {
      store(-2);
      return;
    }
    if (enters) atomicAdd(&new_hist[bn], 1u);
    // (a row evicts nothing before the places are taken)
    first = max(0, kept - min(e, lo + nb - k));
    find_bin(first);
    b2 = sm.bin[1];
    strong = sm.before[1];
    nl = end - strong;
    by_bin = nl - (kept - first) <= NEAR;
    if (by_bin) {
      const float most = bins.most(b2), least = fmaxf(bins.least(b1), full ? bits_float(bins.last) : -__builtin_inff());
      s.each([&](float z, int t, int e2) {
        const float y = z + bins.add;
        if (y <= most && y >= least) sm.cand[atomicAdd(&hist[bins.of(z)], 1u) - strong] = ranked(desc_key(z), s.index(t, e2));
      });
      scan_bins<BIN_BITS>(sm, new_hist, [](int, uint32_t, uint32_t) {});
      if (enters) new_run[atomicAdd(&new_hist[bn], 1u)] = ranked(kn, lo + tid);
    }
  }
  if (!by_bin && N > 0) {
    const int ibits = 32 - __clz(n);
    Window w0, w1;  // of the first that takes part and of the last resident
    if (bins.ok) {
      windows_of_bins(bins, full, b2, b1, ibits, first, strong, sm.count[1], kept - 1, end_before, end - end_before, w0, w1);
      if (kept == N) w1.count = 0;  // (every older key is still there)
      tighten(sm, s, ibits, w0, w1);
    } else {
      w0.init(0, 1ull << 32, ibits, 0, 0, N);
      w1 = w0;
      tighten(sm, s, ibits, w0, w1);
      // (with no place left, a key has to be ahead of the last older one to enter)
      enters = tid < nb && (cap > N || kn < (uint32_t)(w0.last >> ibits));
      const int e = __syncthreads_count(enters);
      if (e == 0) {
        store(-2);
        return;
      }
      w0.rank = uniform(max(0, kept - min(e, lo + nb - k)));
      w1.rank = uniform(kept - 1);
      if (kept == N) w1.count = 0;
    }
    narrow<BIN_BITS>(sm, hist, new_hist, s, ibits, w0, w1, NARROW);
    if (kept < N) enters = enters && composite(kn, lo + tid, ibits) <= w1.last;
    if (__syncthreads_count(enters) == 0) {
      store(-2);
      return;
    }
    strong = w0.before;
    if (tid == 0) sm.fill = 0;
    __syncthreads();
    s.each_again([&](float z, int t, int e2) {
      const uint64_t c2 = composite(desc_key(z), s.index(t, e2), ibits);
      if (c2 >= w0.base && (kept == N || c2 <= w1.last)) sm.cand[atomicAdd(&sm.fill, 1)] = ranked(desc_key(z), s.index(t, e2));
    });
    __syncthreads();
    nl = sm.fill;
  }
  const int places = cap - strong;  // for the nl older keys and the new ones
  const uint64_t em = __ballot(enters);
  if (l == 0) sm.wsum[w] = __popcll(em);
  if (tid < BQ) out[tid] = enters ? -1 : -2;
  __syncthreads();  // (sm.cand is complete too)
  int ne = 0, nbase = 0;
#pragma unroll
  for (int i = 0; i < BQ / 64; i++) {
    nbase += i < w ? sm.wsum[i] : 0u;
    ne += sm.wsum[i];
  }
  if (enters) {
    const int i = nbase + __popcll(em & ((1ull << l) - 1ull));
    newc[i] = ranked(kn, lo + tid);
    if (!by_bin) new_run[i] = ranked(kn, lo + tid);
  }
  __syncthreads();
  // Key x leaves at the row of the left-th new key (in index order) among those ahead of it: `left` from the older keys
  // ahead of it, and how many new ones are ahead of it in all, ...
  uint64_t cx[XT];
  int left[XT], ahead[XT];
#pragma unroll
  for (int u = 0; u < XT; u++) {
    const int x = tid + NT * u;
    left[u] = ahead[u] = 0;
    cx[u] = 0;
    if (x >= nl + ne) continue;
    cx[u] = x < nl ? sm.cand[x] : newc[x - nl];
    int r0 = 0, r1 = nl, n0 = 0, n1 = ne;  // the older and the new keys of its bin, or all of them
    if (by_bin) {
      const int b = bins.of(key_value((uint32_t)(cx[u] >> 32)));
      r0 = b > b2 ? (int)hist[b - 1] - strong : 0;  // (the counters stand at their bins' ends now)
      r1 = b >= b2 ? (int)hist[b] - strong : 0;
      n0 = b > 0 ? (int)new_hist[b - 1] : 0;
      n1 = new_hist[b];
    }
    auto rank_in = [&](const uint64_t* run, int i0, int i1) __attribute__((always_inline)) {
      int r = i0, i = i0;
#pragma unroll 1
      for (; i + RUN <= i1; i += RUN) {
#pragma unroll
        for (int j = 0; j < RUN; j++) r += run[i + j] < cx[u];
      }
#pragma unroll
      for (int j = 0; j < RUN - 1; j++) r += (i + j < i1) & (run[i + j] < cx[u]);
      return r;
    };
    left[u] = places - rank_in(sm.cand, r0, r1);
    ahead[u] = rank_in(new_run, n0, n1);
    if (x >= nl) new_rank[x - nl] = ahead[u];
  }
  __syncthreads();
  // ... then by the set of the first r new keys in rank order, as bits in index order, for every r.
  uint64_t* sets = reinterpret_cast<uint64_t*>(hists);  // [r - 1][BQ / 64]
  static_assert(BQ * (BQ / 64) * 8 <= 2 * BINS * 4, "the sets take the histograms' place");
  {
    const int words = ne <= 64 ? 1 : ne <= 128 ? 2 : 4, wd = w % words;
    const int mine = 64 * wd + l < ne ? new_rank[64 * wd + l] : BQ;
    for (int r0 = w / words * 64; r0 < ne; r0 += NW / words * 64) {
      int lo32 = 0, hi32 = 0;  // lane i: the set of r0 + i + 1
      static_for<64>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        write_lane<i>(lo32, hi32, __ballot(mine <= r0 + i));
      });
      if (r0 + l < ne) sets[(r0 + l) * (BQ / 64) + wd] = (uint64_t)(uint32_t)hi32 << 32 | (uint32_t)lo32;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < XT; u++) {
    const int x = tid + NT * u;
    if (x >= nl + ne) continue;
    const int key = a + (int)(uint32_t)cx[u];
    int y = -1;  // the new key at whose row it leaves
    if (left[u] > 0 && left[u] <= ahead[u]) {
      const uint64_t* set = sets + (ahead[u] - 1) * (BQ / 64);
      int r = left[u];
      uint64_t m = 0;
#pragma unroll
      for (int i = 0; i < BQ / 64; i++)
        if (64 * i < ne && y < 0) {
          m = set[i];
          const int cnt = __popcll(m);
          if (r <= cnt) y = 64 * i; else r -= cnt;
        }
      uint32_t v = (uint32_t)m;
      const int low = __popc(v);
      if (r > low) { r -= low; y += 32; v = (uint32_t)(m >> 32); }
#pragma unroll
      for (int b = 16; b > 0; b >>= 1) {
        const int cnt = __popc(v & ((1u << b) - 1u));
        if (r > cnt) { r -= cnt; y += b; v >>= b; }
      }
    }
    const int row = y >= 0 ? (int)(uint32_t)newc[y] - lo : -1;
    if (x < nl) {
      if (y >= 0) out[row] = key;
    } else if (left[u] <= 0 || (y >= 0 && y < x - nl)) {
      out[key - a - lo] = -2;  // it never enters
    } else if (y >= 0) {
      out[row] = key;
    }
  }
  __syncthreads();
  store(out[min(tid, BQ - 1)]);
}

void launch_evictions(const SelectArgs& a, int longest, int H_q, hipStream_t st) {
  if (a.ck_min < longest)
    checkpoint_kernel<<<dim3(a.T / CK_SEG + a.n_docs, H_q), CK_NT, 0, st>>>(a);
  evict_kernel<256, 4><<<dim3(a.nblk_cap, H_q), 256, 0, st>>>(a);
}

}  // namespace dma
