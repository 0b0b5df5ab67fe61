// Top-k pages of one stream by one workgroup: shared by the stand-alone selection kernel and
// by the attention kernel whose workgroups select their own pages.
#pragma once
#include "stc_common.hpp"

namespace stc {

__device__ __forceinline__ int wave_incl_scan(int v, int /*lane*/) {
  return (int)wave_scan((uint32_t)v, OpAdd{}, 0u);
}

// Exclusive scan over the block (thread order); *total = block sum.
__device__ __forceinline__ int block_exscan(int v, int* lds_waves, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  const int inc = wave_incl_scan(v, lane);
  if (lane == 63) lds_waves[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const int x = lds_waves[w];
    if (w < wave) base += x;
    tot += x;
  }
  *total = tot;
  __syncthreads();
  return base + inc - v;
}

// The same scan for callers that keep two buffers of per-wavefront sums and alternate
// between them: a buffer is written again two barriers after it was last read at the
// earliest, so the barrier behind the reads can go.
template <int NW>
__device__ __forceinline__ uint32_t block_exscan_once(uint32_t v, uint32_t* lds_waves,
                                                      uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_scan(v, OpAdd{}, 0u);
  if (lane == 63) lds_waves[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t x = lds_waves[w];
    if (w < wave) base += x;
    tot += x;
  }
  *total = tot;
  return base + inc - v;
}

constexpr int kTopkBins = 1024;  // bins of the first histogram, of bf16 resolution, used in a circle
constexpr int kTopkFine = 256;   // bins of the second one, between the first threshold and the maximum

// Shared memory of a selection by THREADS threads (512 at most) with IPT keys each.
template <int IPT, int THREADS>
struct TopkLds {
  // keys above the first threshold that a wavefront can hold: all of its own up to 8 per thread
  static constexpr int OWN = IPT > 2 ? (IPT < 8 ? IPT : 8) * 64 : 1;
  alignas(16) int hist[kTopkBins];
  alignas(16) int fine[kTopkFine];
  alignas(16) uint32_t wmin[8], wmax[8];
  int tot[8];
  int cand[64];
  int gt[64], ge[64];
  int ncand, full;
  int key[THREADS / 64][OWN];
  uint16_t page[THREADS / 64][OWN];
};

__device__ __forceinline__ int lanes_below(uint64_t m) {  // set bits of m below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Of the 256 counts whose largest bins lane l holds four of (h4, lane 0 the topmost): the bin that holds
// the key of rank `rank`, if it is among them (uniform over the wavefront).  `above` = counts in front
// of it (of all, if it is not there), `cnt` = its own; returns its offset from the top or -1.
__device__ __forceinline__ int rank_bin(int4 h4, int rank, int& above, int& cnt) {
  const int cd[4] = {h4.w, h4.z, h4.y, h4.x};
  const int mine = (h4.w + h4.z) + (h4.y + h4.x);
  const int incl = (int)wave_scan((uint32_t)mine, OpAdd{}, 0u);
  int at = above + incl - mine, f_bin = 0, f_above = 0, f_cnt = 0;
  const uint64_t hit = __ballot(at < rank && rank <= at + mine);
  if (hit == 0) {
    above += __builtin_amdgcn_readlane(incl, 63);
    return -1;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (at < rank) f_bin = j, f_above = at, f_cnt = cd[j];
    at += cd[j];
  }
  const int src = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
  above = __builtin_amdgcn_readlane(f_above, src);
  cnt = __builtin_amdgcn_readlane(f_cnt, src);
  return 4 * src + __builtin_amdgcn_readlane(f_bin, src);
}

// Top-k pages of a stream by one workgroup of THREADS threads, NP <= THREADS * IPT pages.
// The selected pages are handed to emit(position in the ascending list, page).  Returns false,
// with nothing emitted, if the scores are not of the kind that it is made for (below).
//
// Bound by latency: a chain of barriers and of dependent instructions, in which a step over all keys
// of a thread, or a branch per key, costs as much as a barrier.  So no phase goes through a thread's
// keys one by one, and few keys are left after the first:
//  - Scores are compared as the integers that their bits are, which is their order wherever
//    they are positive.
//  - The digits of the first histogram are the upper 16 bits (bf16 resolution, 128 bins per
//    octave), taken in a circle of 1024 bins, so that the range of the keys need not be known
//    before they are counted.
//  - Up to 2 keys per thread: all of them are counted, and the bin of the k-th largest is found.
//  - More: only the maxima of groups of 4 adjacent keys are counted.  k maxima at or above a bin's
//    lower edge are k keys at or above it, so the pages below it are out.  Every wavefront gathers
//    those that are left of its own, few more than k in all, and only these are counted in finer
//    bins between that edge and the maximum.
//  - The keys of the wanted bin are ranked one by one, and positions come from ballots.
// Many keys in the wanted bin get further bins between the smallest and the largest of them, equal ones
// are taken in page order.  Made for streams whose k-th largest score is positive and within 8
// octaves of the maximum; NaN and infinities are outside.
// Time from the scores' arrival to the list, inside the attention launch, against topk_any: 8192 keys of
// which 256 are kept 5.3 -> 3.6 us, 2048 of which 128 are kept 3.0 -> 2.4 (a step over 28 caches of
// 131072 tokens 604 -> 543 us, over 64 streams of 2048 pages 30.4 -> 30.0).  Scores that it gives up
// on cost its first phases on top, 0.3 to 1.5 us.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ bool topk_positive(const float* __restrict__ sc, int NP, int k,
                                              TopkLds<IPT, THREADS>& S, Emit emit) {
  constexpr int NW = THREADS / 64;
  constexpr bool ALL = IPT <= 2;
  constexpr int VEC = IPT < 4 ? IPT : 4, NQ = IPT / VEC;
  constexpr int NE = ALL ? VEC : TopkLds<IPT, THREADS>::OWN / 64;  // keys per lane that are left, at most
  typedef int keyvec __attribute__((ext_vector_type(VEC == 1 ? 2 : VEC), aligned(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (NP < VEC || (!ALL && k > (NP / VEC) / 8 * 7)) return false;

  // A wavefront owns 64 * IPT adjacent pages, a lane VEC adjacent ones of each of their NQ parts:
  // key[q * VEC + i] is page first(q) + i.  The lanes behind the last page read the last VEC pages,
  // of which they own those from their own first page on.
  int key[NQ * VEC];
  auto own = [&](int q) { return ((wave * NQ + q) * 64 + lane) * VEC; };
  auto first = [&](int q) { return min(own(q), NP - VEC); };
  static_for<0, NQ>([&](auto q) {
    const float* p = sc + first(q);
    if constexpr (VEC == 1) {
      key[q] = __float_as_int(*p);
    } else {
      const keyvec v = *(const keyvec*)p;
      static_for<0, VEC>([&](auto i) { key[q * VEC + i] = v[(int)i]; });
    }
  });
  for (int i = tid; i < kTopkBins / 4; i += THREADS) ((int4*)S.hist)[i] = int4{0, 0, 0, 0};
  if (!ALL && tid < kTopkFine / 4) ((int4*)S.fine)[tid] = int4{0, 0, 0, 0};
  if (tid == 0) S.ncand = 0, S.full = 0;
  __syncthreads();
  if ((wave + 1) * 64 * IPT > NP)
    static_for<0, NQ>([&](auto q) {
      static_for<0, VEC>([&](auto i) {
        if (first(q) + i < own(q)) key[q * VEC + i] = INT32_MIN;
      });
    });

  // What is counted, and the range of it.
  uint32_t vmax = 0u, vmin = 0xffffffffu;
  auto count = [&](int v) {
    if (v > 0) atomicAdd(&S.hist[(v >> 16) & (kTopkBins - 1)], 1);
    vmax = max(vmax, (uint32_t)max(v, 0));
    vmin = min(vmin, v > 0 ? (uint32_t)v : 0xffffffffu);
  };
  static_for<0, NQ>([&](auto q) {
    if constexpr (ALL) {
      static_for<0, VEC>([&](auto i) { count(key[i]); });
    } else {
      count(max(max(key[4 * q], key[4 * q + 1]), max(key[4 * q + 2], key[4 * q + 3])));
    }
  });
  vmax = wave_reduce(vmax, OpMax{}, 0u);
  vmin = wave_reduce(vmin, OpMin{}, 0xffffffffu);
  if (lane == 0) S.wmax[wave] = vmax, S.wmin[wave] = vmin;
  __syncthreads();

  // The bin in which the count from above reaches k; every wavefront finds it for itself.
#pragma unroll
  for (int w = 0; w < NW; ++w) vmax = max(vmax, S.wmax[w]), vmin = min(vmin, S.wmin[w]);
  if (vmax == 0u) return false;
  const int top = (int)(vmax >> 16) | 3, bins = top - (int)(vmin >> 16) + 1;
  if (bins > kTopkBins) return false;
  int above = 0, cnt = 0, bin = -1;
  for (int c0 = 0; bin < 0; c0 += 256) {
    if (c0 >= bins) return false;  // fewer than k of them are positive
    const int o = rank_bin(*(const int4*)&S.hist[(top - 3 - c0 - 4 * lane) & (kTopkBins - 1)], k,
                           above, cnt);
    if (o >= 0) bin = top - c0 - o;
  }
  if (bin <= 0) return false;  // zeros would lie in it, which are not counted
  int edge = bin << 16;        // of the wanted bin, which has `cnt` keys

  // left[e], page[e]: the keys at or above the edge that this wavefront gathers from its own, in page
  // order: number 64*e + lane.  (ALL: its own keys, number 64*e + lane is key e of the lane.)
  int left[NE], page[NE];
  int n = 64;  // their number in this wavefront
  auto each = [&](auto f) {  // more than one per lane are rare
    f(IC<0>{});
    if constexpr (NE > 1) {
      if (ALL || n > 64)
        static_for<1, NE>([&](auto e) {
          if (ALL || 64 * e < n) f(e);
        });
    }
  };
  int shift = 16;  // binary digits of the keys below those of the bin
  if constexpr (ALL) {
    static_for<0, NE>([&](auto e) { left[e] = key[e], page[e] = first(0) + e; });
  } else {
    uint32_t has = 0u;
    static_for<0, IPT>([&](auto j) { has |= key[j] >= edge ? 1u << j : 0u; });
    int start[NQ];
    n = 0;
    static_for<0, (NQ + 1) / 2>([&](auto h) {  // counts of two parts in the halves of a word
      const uint32_t c = (uint32_t)__popc(has >> (8 * h) & 0xfu) |
                         (uint32_t)__popc(has >> (8 * h) & 0xf0u) << 16;
      const uint32_t incl = wave_scan(c, OpAdd{}, 0u);
      const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      start[2 * h] = n + (int)((incl - c) & 0xffffu);
      n += (int)(all & 0xffffu);
      if constexpr (2 * h + 1 < NQ) {
        start[2 * h + 1] = n + (int)((incl - c) >> 16);
        n += (int)(all >> 16);
      }
    });
    if (n <= TopkLds<IPT, THREADS>::OWN) {
      for (uint32_t m = has; m; m &= m - 1u) {
        const int j = __ffs((int)m) - 1, q = j >> 2;
        const int at = pick_of(start, q) + __popc(has & (0xfu << (4 * q)) & ((1u << j) - 1u));
        S.key[wave][at] = pick_of(key, j);
        S.page[wave][at] = (uint16_t)(first(q) + (j & 3));
      }
    } else {
      n = 0;
      S.full = 1;
    }
    wave_lds_sync();
    shift = max(0, 24 - __clz((int)(vmax - (uint32_t)edge) | 1));
    each([&](auto e) {
      const int at = max(min(64 * e + lane, n - 1), 0);
      const int v = S.key[wave][at];
      page[e] = S.page[wave][at];
      left[e] = 64 * e + lane < n ? v : INT32_MIN;
      if (64 * e + lane < n) atomicAdd(&S.fine[(v - edge) >> shift], 1);
    });
    __syncthreads();
    if (S.full) return false;  // a wavefront has more than it can hold
    above = 0;
    const int o = rank_bin(*(const int4*)&S.fine[kTopkFine - 4 - 4 * lane], k, above, cnt);
    edge += (kTopkFine - 1 - o) << shift;
  }

  // The least key that is taken: the edge, or a key of the wanted bin.
  int least = edge;
  int rank = k - above;  // in the wanted bin
  int equal = 0;         // > 0: that many keys are the least one, and not all of them are taken
  // Too many to rank one by one: bins between the smallest and the largest of them, unless all are equal.
  while (rank < cnt && cnt > 64) {
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    auto in_bin = [&](int v) { return ((uint32_t)v - (uint32_t)edge) >> shift == 0u; };
    each([&](auto e) {
      if (in_bin(left[e])) kmin = min(kmin, (uint32_t)left[e]), kmax = max(kmax, (uint32_t)left[e]);
    });
    kmin = wave_reduce(kmin, OpMin{}, 0xffffffffu);
    kmax = wave_reduce(kmax, OpMax{}, 0u);
    __syncthreads();  // the bins and the range of the round before have been read
    if (lane == 0) S.wmax[wave] = kmax, S.wmin[wave] = kmin;
    if (tid < kTopkFine / 4) ((int4*)S.fine)[tid] = int4{0, 0, 0, 0};
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) kmax = max(kmax, S.wmax[w]), kmin = min(kmin, S.wmin[w]);
    if (kmin == kmax) {
      least = (int)kmin, equal = cnt;
      break;
    }
    const int finer = max(0, 24 - __clz((int)(kmax - kmin) | 1));
    each([&](auto e) {
      if (in_bin(left[e])) atomicAdd(&S.fine[(left[e] - (int)kmin) >> finer], 1);
    });
    __syncthreads();
    int front = 0;
    const int o = rank_bin(*(const int4*)&S.fine[kTopkFine - 4 - 4 * lane], rank, front, cnt);
    rank -= front;
    shift = finer;
    edge = (int)kmin + ((kTopkFine - 1 - o) << finer);
    least = edge;
  }
  if (rank < cnt && equal == 0) {
    each([&](auto e) {
      if (((uint32_t)left[e] - (uint32_t)edge) >> shift == 0u) S.cand[atomicAdd(&S.ncand, 1)] = left[e];
    });
    __syncthreads();
    const int mine = lane < cnt ? S.cand[lane] : INT32_MIN;
    int gt = 0;
    for (int i = 0; i < cnt; ++i) gt += __builtin_amdgcn_readlane(mine, i) > mine;
    int larger = rank - 1;  // keys of the bin above the wanted one
    uint64_t eq;            // the candidates with its value
    while ((eq = __ballot(lane < cnt && gt == larger)) == 0) --larger;
    least = __builtin_amdgcn_readlane(
        mine, __builtin_amdgcn_readfirstlane(__ffsll((long long)eq) - 1));
    rank -= larger;
    if (rank < __popcll(eq)) equal = __popcll(eq);
  }
  if (equal > 0) {  // of the equal keys the first `rank` are taken; the others are out
    uint64_t same[NE] = {};
    int sum = 0;
    each([&](auto e) {
      same[e] = __ballot(left[e] == least);
      sum += __popcll(same[e]);
    });
    if (lane == 0) S.gt[wave] = sum;
    __syncthreads();
    const uint32_t t = lane < NW ? (uint32_t)S.gt[lane] : 0u;
    int at = __builtin_amdgcn_readlane((int)(wave_scan(t, OpAdd{}, 0u) - t), wave);
    if constexpr (ALL) static_for<0, NE>([&](auto e) { at += lanes_below(same[e]); });
    each([&](auto e) {
      if (left[e] == least && (ALL ? at++ : at + lanes_below(same[e])) >= rank)
        left[e] = INT32_MIN;
      if (!ALL) at += __popcll(same[e]);
    });
  }

  // Positions: a count per wavefront, and the wavefronts in front of it.
  uint64_t taken[NE] = {};
  int sum = 0;
  each([&](auto e) {
    taken[e] = __ballot(left[e] >= least);
    sum += __popcll(taken[e]);
  });
  if (lane == 0) S.tot[wave] = sum;
  __syncthreads();
  const uint32_t t = lane < NW ? (uint32_t)S.tot[lane] : 0u;
  int pos = __builtin_amdgcn_readlane((int)(wave_scan(t, OpAdd{}, 0u) - t), wave);
  if constexpr (ALL) {
    static_for<0, NE>([&](auto e) { pos += lanes_below(taken[e]); });
    static_for<0, NE>([&](auto e) {
      if (left[e] >= least) emit(pos++, page[e]);
    });
  } else {
    each([&](auto e) {
      if (left[e] >= least) emit(pos + lanes_below(taken[e]), page[e]);
      pos += __popcll(taken[e]);
    });
  }
  return true;
}

// The same for any scores, by radix select: thread t owns the IPT adjacent pages t*IPT .. and holds
// their keys in registers.  Each radix pass is a shared-memory histogram of one key digit, which
// every wavefront then scans for itself (digits in descending order) to find the digit that holds
// the k-th largest key: no broadcast and no second barrier.  The usual case (one pass, then at
// most 64 candidates ranked directly) crosses five workgroup barriers.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_any(const float* __restrict__ sc, int NP, int k,
                                         TopkLds<IPT, THREADS>& S, Emit emit) {
  constexpr int NW = THREADS / 64;
  // Digit width: 8 bits, 10 from 4096 keys on, where a digit of 8 bits leaves more keys beside
  // the k-th than are ranked directly, which costs a second pass.
  constexpr int HB = THREADS * IPT > 2048 ? 10 : 8;
  constexpr int BINS = 1 << HB, PER = BINS / 64;  // digits per lane of a wavefront's scan
  int* const hist = S.hist;
  uint32_t* const waves = (uint32_t*)S.tot;  // per-wavefront sums of the final scan
  uint32_t *const s_min = S.wmin, *const s_max = S.wmax;
  int& s_ncand = S.ncand;
  uint32_t* const cand = (uint32_t*)S.cand;
  int *const s_gt = S.gt, *const s_ge = S.ge;  // per candidate: candidates above it / not below it
  static_assert(BINS <= kTopkBins && NW <= 8, "shared memory");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int i0 = tid * IPT;

  // keys of absent pages (index >= NP) are 0, below the key of any finite float
  uint32_t key[IPT];
  if constexpr (IPT >= 4) {
    if (i0 + IPT <= NP && (NP % 4) == 0) {
#pragma unroll
      for (int j = 0; j < IPT; j += 4) {
        const float4 v = *(const float4*)(sc + i0 + j);
        key[j] = float_key(v.x), key[j + 1] = float_key(v.y);
        key[j + 2] = float_key(v.z), key[j + 3] = float_key(v.w);
      }
    } else {
#pragma unroll
      for (int j = 0; j < IPT; ++j) key[j] = i0 + j < NP ? float_key(sc[i0 + j]) : 0u;
    }
  } else {
#pragma unroll
    for (int j = 0; j < IPT; ++j) key[j] = i0 + j < NP ? float_key(sc[i0 + j]) : 0u;
  }
  for (int i = tid; i < BINS; i += THREADS) hist[i] = 0;
  if (tid < 64) s_gt[tid] = 0, s_ge[tid] = 0;
  if (tid == 0) s_ncand = 0;

  // Bits above the highest bit in which two keys differ are common to all keys and
  // need no pass; starting at that bit also spreads the first histogram over many
  // bins (page scores share their sign and most exponent bits).
  uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (i0 + j < NP) kmin = min(kmin, key[j]), kmax = max(kmax, key[j]);
  kmin = wave_reduce(kmin, OpMin{}, 0xffffffffu);
  kmax = wave_reduce(kmax, OpMax{}, 0u);
  if ((tid & 63) == 0) s_min[tid >> 6] = kmin, s_max[tid >> 6] = kmax;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) kmin = min(kmin, s_min[w]), kmax = max(kmax, s_max[w]);
  const uint32_t diff = kmin ^ kmax;
  const int top = diff ? 31 - __clz(diff) : 0;  // highest differing bit
  int shift = max(top - (HB - 1), 0);
  uint32_t decided = shift + HB < 32 ? ~((1u << (shift + HB)) - 1u) : 0u;  // key bits fixed so far
  uint32_t prefix = kmax & decided;
  int remaining = k;  // rank of the k-th largest key among the keys sharing the prefix
  // The last window may overlap bits that are already fixed; keys are filtered on all
  // fixed bits, so the digit found repeats them.  The histogram is zero on entry to every
  // pass.
  for (;; shift = max(shift - HB, 0)) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool in = (key[j] & decided) == prefix;
      if (in && i0 + j < NP) atomicAdd(&hist[(key[j] >> shift) & (BINS - 1u)], 1);
    }
    __syncthreads();
    // Every wavefront finds the digit for itself (no broadcast, no second barrier): lane l
    // looks at PER adjacent digits in descending order, a wavefront scan gives the keys with a
    // larger digit.
    int cd[PER], mine = 0;
#pragma unroll
    for (int j = 0; j < PER; j += 4) {
      const int4 h4 = *(const int4*)&hist[BINS - 4 - j - PER * lane];
      cd[j] = h4.w, cd[j + 1] = h4.z, cd[j + 2] = h4.y, cd[j + 3] = h4.x;
      mine += (h4.w + h4.z) + (h4.y + h4.x);
    }
    int above = (int)wave_scan((uint32_t)mine, OpAdd{}, 0u) - mine;
    int f_digit = 0, f_above = 0, f_cnt = 0;
    bool found = false;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool hit = above < remaining && remaining <= above + cd[j];
      if (hit) f_digit = BINS - 1 - PER * lane - j, f_above = above, f_cnt = cd[j];
      found |= hit;
      above += cd[j];
    }
    const int src = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(found)) - 1);
    const int digit = __builtin_amdgcn_readlane(f_digit, src);
    const int c = __builtin_amdgcn_readlane(f_cnt, src);  // keys that share the new prefix
    remaining -= __builtin_amdgcn_readlane(f_above, src);
    prefix = (prefix & ~((BINS - 1u) << shift)) | ((uint32_t)digit << shift);
    decided = ~((1u << shift) - 1u);
    if (shift == 0) break;
    if (c <= 64) {
      // Few keys are left: list them and rank them directly.
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if (i0 + j < NP && (key[j] & decided) == prefix) cand[atomicAdd(&s_ncand, 1)] = key[j];
      __syncthreads();
      // rank of every candidate among the candidates: wavefront w compares all of them with
      // its share of the list, the partial counts meet in shared memory
      {
        constexpr int PER = (64 + NW - 1) / NW;
        const int ci = tid & 63, j0 = (tid >> 6) * PER;
        if (ci < c && j0 < c) {
          const uint32_t mine = cand[ci];
          int gt = 0, ge = 0;
#pragma unroll
          for (int j = 0; j < PER; ++j) {
            const uint32_t o = cand[min(j0 + j, 63)];
            const bool in = j0 + j < c;
            gt += in && o > mine;
            ge += in && o >= mine;
          }
          if (gt) atomicAdd(&s_gt[ci], gt);
          if (ge) atomicAdd(&s_ge[ci], ge);
        }
      }
      __syncthreads();
      {  // every wavefront picks the k-th key itself: lane i looks at candidate i
        const int ci = min(lane, c - 1);
        const int gt = s_gt[ci], ge = s_ge[ci];
        const uint32_t mine = cand[ci];
        const bool kth = gt < remaining && remaining <= ge;  // equal keys agree
        const int s2 = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(kth)) - 1);
        prefix = (uint32_t)__builtin_amdgcn_readlane((int)mine, s2);
        remaining -= __builtin_amdgcn_readlane(gt, s2);
      }
      break;
    }
    // another pass: the histogram is cleared once every wavefront has read it
    __syncthreads();
    for (int i = tid; i < BINS; i += THREADS) hist[i] = 0;
    __syncthreads();
  }
  // prefix = key of the k-th largest score; `remaining` of the pages equal to it are
  // taken, lowest page index first.  One scan carries both counts of a thread: pages above
  // the key in the low half, pages equal to it in the high half.
  uint32_t both = 0;
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (i0 + j < NP) both += (key[j] > prefix ? 1u : 0u) + (key[j] == prefix ? 0x10000u : 0u);
  uint32_t tot;
  const uint32_t before = block_exscan_once<NW>(both, waves, &tot);
  int e = (int)(before >> 16);                           // equal pages in front of this thread
  int pos = (int)(before & 0xffffu) + min(e, remaining);  // selected pages in front of it
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    if (i0 + j < NP) {
      bool t = key[j] > prefix;
      if (key[j] == prefix) t = e++ < remaining;
      if (t && pos < k) emit(pos++, i0 + j);
    }
  }
}

// The same for any scores of at most 128 pages (64 with fewer than 8 wavefronts): a page's place is the
// number of pages in front of it, which every wavefront counts over its share of the pages.  One
// barrier, where the forms above cross four: 8 streams of 64 pages, 16 kept, 5.9 us per step for 6.3.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_few(const float* __restrict__ sc, int NP, int k,
                                         TopkLds<IPT, THREADS>& S, Emit emit) {
  constexpr int NW = THREADS / 64, E = NW < 8 ? 1 : 2;  // pages per lane
  static_assert(NW * E * 64 <= kTopkBins, "counts of all wavefronts");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t key[E];
  int ahead[E];
  static_for<0, E>([&](auto e) {
    key[e] = float_key(sc[min(e * 64 + lane, NP - 1)]);
    ahead[e] = 0;
  });
  const int share = (NP + NW - 1) / NW, j1 = min((wave + 1) * share, NP);
  for (int j = wave * share; j < j1; ++j) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)(j < 64 ? key[0] : key[E - 1]), j & 63);
    static_for<0, E>([&](auto e) {
      ahead[e] += (o > key[e]) | ((o == key[e]) & (j < e * 64 + lane));
    });
  }
  static_for<0, E>([&](auto e) { S.hist[(wave * E + e) * 64 + lane] = ahead[e]; });
  __syncthreads();
  int pos = 0;
  static_for<0, E>([&](auto e) {
    int place = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) place += S.hist[(w * E + e) * 64 + lane];
    const bool t = e * 64 + lane < NP && place < k;
    const uint64_t m = __ballot(t);
    if (wave == e && t) emit(pos + lanes_below(m), e * 64 + lane);
    pos += __popcll(m);
  });
}

// Top-k pages of a stream by one workgroup of THREADS threads, NP <= THREADS * IPT <= 65535: ties to
// the lowest page, emit(position in the ascending list, page) for every selected one.  `sc` must not
// lie in `S`.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_block(const float* __restrict__ sc, int NP, int k,
                                           TopkLds<IPT, THREADS>& S, Emit emit) {
  if constexpr (IPT <= 2) {
    if (NP <= (THREADS < 512 ? 64 : 128)) {
      topk_few<IPT, THREADS>(sc, NP, k, S, emit);
      return;
    }
  }
  if (topk_positive<IPT, THREADS>(sc, NP, k, S, emit)) return;
  __syncthreads();
  topk_any<IPT, THREADS>(sc, NP, k, S, emit);
}

}  // namespace stc
