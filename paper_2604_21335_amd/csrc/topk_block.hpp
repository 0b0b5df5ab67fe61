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

constexpr int kTopkBits = 8, kTopkBins = 1 << kTopkBits;  // bins of a histogram
constexpr int kTopkRanked = 16;  // keys that are ranked one by one at most

// Shared memory of a selection by THREADS threads (512 at most) with IPT keys each.
template <int IPT, int THREADS>
struct TopkLds {
  static constexpr int OWN = IPT > 2 ? 64 * IPT : 1;  // keys that a wavefront may have to list
  alignas(16) int hist[4][kTopkBins];
  alignas(16) uint32_t wmin[8], wmax[8], rmin[8], rmax[8], tot[8];
  int npos[8], np[8], cand[kTopkRanked], ncand;
  int key[THREADS / 64][OWN];
  uint16_t page[THREADS / 64][OWN];
};

__device__ __forceinline__ int lanes_below(uint64_t m) {  // set bits of m below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// What is rare lies out of the way: the code of a launch is fetched while it runs, and what has to be
// jumped over costs more than the test for it (0.2 us of a step of 17 when all of it lay in line).
__device__ __forceinline__ bool topk_rare(bool x) { return __builtin_expect(x, false); }

// Of the 256 counts of which lane l holds the four from bin 4*l on, behind `above` others: the bin that holds
// the key of rank `rank`, which is among them (uniform over the wavefront).  `above` = counts in front of
// it, `cnt` = its own.
__device__ __forceinline__ int rank_bin(int4 h4, int rank, int& above, int& cnt) {
  const int cd[4] = {h4.x, h4.y, h4.z, h4.w};
  const int mine = (h4.x + h4.y) + (h4.z + h4.w);
  const int incl = (int)wave_scan((uint32_t)mine, OpAdd{}, 0u);
  int at = above + incl - mine, f_bin = 0, f_above = 0, f_cnt = 0;
  const uint64_t hit = __ballot(at < rank && rank <= at + mine);
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

// Keys lo .. hi: bin `bin` of those of 2^shift keys each that are counted downwards from `top`, as far as
// it lies at or above `bottom`.
struct TopkBin {
  int lo, hi;
  __device__ __forceinline__ TopkBin(int top, int bottom, int shift, int bin) {
    hi = (int)((uint32_t)top - ((uint32_t)bin << shift));
    const uint32_t width = (1u << shift) - 1u;
    lo = (uint32_t)hi - (uint32_t)bottom < width ? bottom : (int)((uint32_t)hi - width);
  }
  __device__ __forceinline__ bool holds(int v) const { return lo <= v && v <= hi; }
};
// Shift with which the keys lo .. hi fall into the bins of a histogram.
__device__ __forceinline__ int topk_shift(int hi, int lo) {
  return max(0, 32 - kTopkBits - __clz((int)(((uint32_t)hi - (uint32_t)lo) | 1u)));
}

// Top-k pages of a stream by one workgroup of THREADS threads, 4 <= NP <= THREADS * IPT pages.
// The selected pages are handed to emit(position in the ascending list, page).
//
// Bound by latency: a chain of barriers and of dependent instructions, in which a step over all keys
// of a thread, or a branch per key, costs as much as a barrier.  So no phase goes through a thread's
// keys one by one, and few keys are left after the first:
//  - Positive scores are compared as the integers that their bits are, which is their order.  Those of
//    negative ones are turned round where they come into it.
//  - A histogram has 256 bins between the smallest and the largest key: one scan by a wavefront, and
//    few keys in the wanted bin, whether the scores lie close together or octaves apart.
//  - Up to 2 keys per thread: all positive ones are counted, and the bin of the k-th largest is found.
//  - More, and k not too large for it: only the maxima of groups of 4 adjacent keys are counted.  k
//    maxima at or above a bin's lower edge are k keys at or above it, so the pages below it are out.
//    Every wavefront lists those that are left of its own, few more than k in all, and only these are
//    counted in bins between that edge and the maximum.
//  - Fewer than k positive keys: the others are counted (with maxima perhaps the positive ones after all).
//  - Up to 16 keys of the wanted bin are ranked one by one, more of them get bins between the smallest
//    and the largest of them, and equal ones are taken in page order.  Positions come from ballots.
// us per step, with a radix select of the keys' differing bits / with that one behind a form for positive
// scores within 8 octaves of the maximum, up to 64 keys of a bin of 1/128 octave ranked / now:
//   pages, kept (streams)      8192, 256 (4)        2048, 128 (64)       500, 40 (192)
//     positive, spread      19.4 / 16.9 / 15.9   29.9 / 28.1 / 28.0   22.3 / 21.4 / 21.4
//     both signs            20.9 / 19.6 / 15.3   30.5 / 29.4 / 27.9   22.9 / 22.4 / 21.4
//     negative              19.7 / 18.5 / 18.0   30.2 / 28.5 / 28.8   22.2 / 22.0 / 21.7
//     within 1 %            24.8 / 25.6 / 18.0   31.5 / 31.0 / 28.3   23.1 / 24.3 / 21.5
//     all equal             24.2 / 25.4 / 18.1   31.0 / 31.6 / 28.0
//     3 % positive, zeros   47.2 / 46.2 / 19.2   42.0 / 40.0 / 28.0   24.5 / 24.3 / 20.8
//     rising with the page  19.7 / 20.0 / 20.0   30.0 / 28.6 / 29.7   21.9 / 21.1 / 21.1
// (rising: all kept pages are one wavefront's.)  With four channels of the keys eight times the others, as the
// benchmark's are, ordinary steps pay 0.5 to 1 % for the range of the keys, without which the second of the
// three counted at once: 64 streams of 2048 pages, 28 heads 28.0 / 28.2; one layer of 4 streams of 8192 15.39 /
// 15.53; 40 of 751 with a tail 16.5 / 16.7.  Measured and left out: counting a bin that many lanes share
// by ballots (20.0 -> 21.9 with rising scores), lists of 128 to 256 keys with a walk over the keys in
// registers where they do not fit (17.4 there, but 2 to 4 % more in every ordinary step: its code).
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_keys(const float* __restrict__ sc, int NP, int k,
                                          TopkLds<IPT, THREADS>& S, Emit emit) {
  constexpr int NW = THREADS / 64;
  constexpr bool ALL = IPT <= 2;
  constexpr int VEC = IPT < 4 ? IPT : 4, NQ = IPT / VEC;
  constexpr int NE = IPT;
  typedef int keyvec __attribute__((ext_vector_type(VEC == 1 ? 2 : VEC), aligned(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto ordered = [](int v) { return (uint32_t)v ^ 0x80000000u; };  // signed order as unsigned
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };

  // A wavefront owns 64 * IPT adjacent pages, a lane VEC adjacent ones of each of their NQ parts:
  // key[q * VEC + i] is page first(q) + i.  The lanes behind the last page read the last VEC pages,
  // of which they own those from their own first page on; the others are absent, the least integer.
  int key[NQ * VEC];
  auto own = [&](int q) { return ((wave * NQ + q) * 64 + lane) * VEC; };
  auto first = [&](int q) { return min(own(q), NP - VEC); };
  auto absent = [&](int q, int i) { return first(q) + i < own(q); };
  static_for<0, NQ>([&](auto q) {
    const float* p = sc + first(q);
    if constexpr (VEC == 1) {
      key[q] = __float_as_int(*p);
    } else {
      const keyvec v = *(const keyvec*)p;
      static_for<0, VEC>([&](auto i) { key[q * VEC + i] = v[(int)i]; });
    }
  });
  if (tid < 3 * kTopkBins / 4) ((int4*)S.hist)[tid] = int4{0, 0, 0, 0};
  if (tid == 0) S.ncand = 0;
  if ((wave + 1) * 64 * IPT > NP)
    static_for<0, NQ>([&](auto q) {
      static_for<0, VEC>([&](auto i) {
        if (absent(q, i)) key[q * VEC + i] = INT32_MIN;
      });
    });

  // What is counted first.  `exact`: all positive keys.
  int above = 0, cnt = 0;  // keys in front of the wanted bin and in it
  const bool exact = ALL || k > (NP / VEC) / 8 * 7;
  int npos = 0;
  uint32_t vmax = 0u, vmin = 0xffffffffu;
  auto counted = [&](auto f) {
    if constexpr (ALL) {
      static_for<0, NE>([&](auto e) { f(key[e], e); });
    } else if (topk_rare(exact)) {
      static_for<0, NE>([&](auto e) { f(key[e], e); });
    } else {
      static_for<0, NQ>([&](auto q) {
        f(max(max(key[4 * q], key[4 * q + 1]), max(key[4 * q + 2], key[4 * q + 3])), q);
      });
    }
  };
  counted([&](int v, auto) {
    npos += __popcll(__ballot(v > 0));
    vmax = max(vmax, (uint32_t)max(v, 0));
    vmin = min(vmin, (uint32_t)v - 1u);  // of those that are not positive: above all others
  });
  vmax = wave_reduce(vmax, OpMax{}, 0u);
  vmin = wave_reduce(vmin, OpMin{}, 0xffffffffu);
  if (lane == 0) S.wmax[wave] = vmax, S.wmin[wave] = vmin, S.npos[wave] = npos;
  __syncthreads();
  npos = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    vmax = max(vmax, S.wmax[w]), vmin = min(vmin, S.wmin[w]), npos += S.npos[w];
  vmax = uniform(vmax), vmin = uniform(vmin), npos = (int)uniform((uint32_t)npos);
  int top = (int)vmax;    // the largest key
  TopkBin b(0, 0, 0, 0);  // the wanted one
  bool listed = !exact;   // the counts of keys are still to come
  const int lowest = (int)vmin + 1;
  if (!topk_rare(npos < k || lowest == top)) {
    const int shift = topk_shift(top, lowest);
    counted([&](int v, auto) {
      if (v > 0) atomicAdd(&S.hist[0][(vmax - (uint32_t)v) >> shift], 1);
    });
    __syncthreads();
    const int bin = rank_bin(*(const int4*)&S.hist[0][4 * lane], k, above, cnt);
    b = TopkBin(top, lowest, shift, bin);
  } else if (npos >= k) {  // all equal
    b.lo = b.hi = top, cnt = npos;
  } else {
    uint32_t kmin = 0xffffffffu, kmax = 0u;  // of the keys that are not positive
    npos = 0;
    static_for<0, NQ>([&](auto q) {
      static_for<0, VEC>([&](auto i) {
        int& v = key[q * VEC + i];
        npos += __popcll(__ballot(v > 0));
        v ^= (int)((uint32_t)(v >> 31) >> 1);
        if (absent(q, i)) {
          v = INT32_MIN;
        } else if (v <= 0) {
          kmin = min(kmin, ordered(v)), kmax = max(kmax, ordered(v));
        }
      });
    });
    kmin = wave_reduce(kmin, OpMin{}, 0xffffffffu);
    kmax = wave_reduce(kmax, OpMax{}, 0u);
    if (lane == 0) S.rmin[wave] = kmin, S.rmax[wave] = kmax, S.np[wave] = npos;
    __syncthreads();
    npos = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w)
      kmin = min(kmin, S.rmin[w]), kmax = max(kmax, S.rmax[w]), npos += S.np[w];
    npos = (int)uniform((uint32_t)npos);
    const bool positive = npos >= k;
    const int low = positive ? 1 : (int)ordered((int)uniform(kmin));
    const int high = positive ? top : (int)ordered((int)uniform(kmax));
    above = positive ? 0 : npos;
    listed = false;
    if (low == high) {
      b.lo = b.hi = low, cnt = positive ? npos : NP - npos;
    } else {
      const int shift = topk_shift(high, low);
      static_for<0, IPT>([&](auto j) {
        if (low <= key[j] && key[j] <= high)
          atomicAdd(&S.hist[0][((uint32_t)high - (uint32_t)key[j]) >> shift], 1);
      });
      __syncthreads();
      const int bin = rank_bin(*(const int4*)&S.hist[0][4 * lane], k, above, cnt);
      b = TopkBin(high, low, shift, bin);
    }
  }

  // The keys at or above the bin's lower edge, `least`, which are few: every wavefront lists its own, n of
  // them, in page order, number 64*e + lane in left[e] as far as that goes.  (ALL: left is its own keys.)
  constexpr int NL = ALL ? IPT : IPT > 8 ? 4 : 2;
  const int least = b.lo;
  int left[NL];
  int n = 0;
  auto each = [&](auto f) {  // f(key, number of lane 0's / 64, whether it is one of them)
    if constexpr (ALL) {
      static_for<0, NL>([&](auto e) { f(left[e], e, true); });
    } else {
      f(left[0], 0, lane < n);
      if (topk_rare(n > 64)) {
        static_for<1, NL>([&](auto e) {
          if (64 * e < n) f(left[e], e, 64 * e + lane < n);
        });
        auto load = [&](int e) { return S.key[wave][min(64 * e + lane, n - 1)]; };
        int v = load(NL);
#pragma unroll 1
        for (int e = NL; 64 * e < n; ++e) {
          const bool there = 64 * e + lane < n;
          const int next = load(e + 1);
          f(there ? v : INT32_MIN, e, there);
          v = next;
        }
      }
    }
  };
  // start[q]: bits of the wavefront in front of this lane's of part q, four a part; returns their number.
  auto starts = [&](uint32_t bits, int (&start)[NQ]) {
    int sum = 0;
    static_for<0, (NQ + 1) / 2>([&](auto h) {  // counts of two parts in the halves of a word
      const uint32_t c = (uint32_t)__popc(bits >> (8 * h) & 0xfu) |
                         (uint32_t)__popc(bits >> (8 * h) & 0xf0u) << 16;
      const uint32_t incl = wave_scan(c, OpAdd{}, 0u);
      const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      start[2 * h] = sum + (int)((incl - c) & 0xffffu);
      sum += (int)(all & 0xffffu);
      if constexpr (2 * h + 1 < NQ) {
        start[2 * h + 1] = sum + (int)((incl - c) >> 16);
        sum += (int)(all >> 16);
      }
    });
    return sum;
  };
  auto below = [](uint32_t bits, int j) {  // bits of the part in front of bit j
    return __popc(bits & (0xfu << (j & ~3)) & ((1u << j) - 1u));
  };
  if constexpr (ALL) {
    static_for<0, NL>([&](auto e) { left[e] = key[e]; });
  } else {
    uint32_t has = 0u;
    static_for<0, IPT>([&](auto j) { has |= key[j] >= least ? 1u << j : 0u; });
    int start[NQ];
    n = starts(has, start);
    auto put = [&](int j, int at, int v) {
      S.key[wave][at] = v;
      S.page[wave][at] = (uint16_t)(first(j >> 2) + (j & 3));
    };
    if (!topk_rare(n > 128)) {
      for (uint32_t m = has; m; m &= m - 1u) {
        const int j = __ffs((int)m) - 1;
        put(j, pick_of(start, j >> 2) + below(has, j), pick_of(key, j));
      }
    } else {  // no search for the next one
      static_for<0, IPT>([&](auto j) {
        if (has >> j & 1u) put(j, start[j / 4] + below(has, j), key[j]);
      });
    }
    wave_lds_sync();
    left[0] = lane < n ? S.key[wave][lane] : INT32_MIN;
    if (topk_rare(n > 64))
      static_for<1, NL>([&](auto e) {
        left[e] = 64 * e + lane < n ? S.key[wave][64 * e + lane] : INT32_MIN;
      });
    if (!topk_rare(!listed)) {
      above = 0, cnt = INT32_MAX;
      if (!topk_rare(least == top)) {  // or they are all equal, and more than needed
        const int shift = topk_shift(top, least);
        each([&](int v, int, bool there) {
          if (there) atomicAdd(&S.hist[1][((uint32_t)top - (uint32_t)v) >> shift], 1);
        });
        __syncthreads();
        const int bin = rank_bin(*(const int4*)&S.hist[1][4 * lane], k, above, cnt);
        b = TopkBin(top, least, shift, bin);
      }
    }
  }

  // Of the keys in the wanted bin, the `rank` largest are taken, those of lowest page among equal ones.
  int rank = k - above;
  bool totals = false;  // S.tot holds every wavefront's keys above the bin and, shifted, in it
  for (int round = 0; topk_rare(rank < cnt && cnt > kTopkRanked && b.lo < b.hi); ++round) {
    uint32_t kmin = 0xffffffffu, kmax = 0u, sum = 0u;
    each([&](int v, auto, bool) {
      const bool in = b.holds(v);
      if (in) kmin = min(kmin, ordered(v)), kmax = max(kmax, ordered(v));
      sum += (uint32_t)__popcll(__ballot(v > b.hi)) + ((uint32_t)__popcll(__ballot(in)) << 16);
    });
    kmin = wave_reduce(kmin, OpMin{}, 0xffffffffu);
    kmax = wave_reduce(kmax, OpMax{}, 0u);
    if (lane == 0) S.rmin[wave] = kmin, S.rmax[wave] = kmax, S.tot[wave] = sum;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) kmin = min(kmin, S.rmin[w]), kmax = max(kmax, S.rmax[w]);
    kmin = uniform(kmin), kmax = uniform(kmax);
    const int low = (int)ordered((int)kmin), high = (int)ordered((int)kmax);
    if (low == high) {
      b.lo = b.hi = low;
      totals = true;
      break;
    }
    int* const h = S.hist[(round + 2) % 3];
    if (tid < kTopkBins / 4) ((int4*)S.hist[round % 3])[tid] = int4{0, 0, 0, 0};  // for the next round
    const int shift = topk_shift(high, low);
    each([&](int v, int, bool) {
      if (b.holds(v)) atomicAdd(&h[((uint32_t)high - (uint32_t)v) >> shift], 1);
    });
    __syncthreads();
    int front = 0;
    const int bin = rank_bin(*(const int4*)&h[4 * lane], rank, front, cnt);
    rank -= front;
    b = TopkBin(high, low, shift, bin);
  }
  if (rank < cnt && b.lo < b.hi) {
    each([&](int v, auto, bool) {
      if (b.holds(v)) S.cand[atomicAdd(&S.ncand, 1)] = v;
    });
    __syncthreads();
    const int mine = lane < cnt ? S.cand[min(lane, kTopkRanked - 1)] : INT32_MIN;
    int gt = 0;
    for (int i = 0; i < cnt; i += 4)  // (those behind the last one are the least integer)
#pragma unroll
      for (int j = 0; j < 4; ++j) gt += __builtin_amdgcn_readlane(mine, i + j) > mine;
    int larger = rank - 1;  // keys of the bin above the wanted one
    uint64_t eq;            // the candidates with its value
    while ((eq = __ballot(lane < cnt && gt == larger)) == 0) --larger;
    b.lo = b.hi = __builtin_amdgcn_readlane(
        mine, __builtin_amdgcn_readfirstlane(__ffsll((long long)eq) - 1));
    rank -= larger;
    cnt = __popcll(eq);
  }

  // Positions: the counts per wavefront, and the wavefronts in front of it.  `cut`: only the first `rank` of
  // the keys in the bin, which are equal, are taken.
  const bool cut = rank < cnt;
  if (!totals) {
    uint32_t sum = 0u;
    each([&](int v, auto, bool) {
      sum += (uint32_t)__popcll(__ballot(cut ? v > b.hi : v >= b.lo));
      if (topk_rare(cut)) sum += (uint32_t)__popcll(__ballot(v == b.lo)) << 16;
    });
    if (lane == 0) S.tot[wave] = sum;
    __syncthreads();
  }
  const uint32_t t = lane < NW ? S.tot[lane] : 0u;
  const uint32_t before =
      (uint32_t)__builtin_amdgcn_readlane((int)(wave_scan(t, OpAdd{}, 0u) - t), wave);
  int pos = (int)(before & 0xffffu);
  int at = 0;  // number of the next key in the bin (cut)
  if (topk_rare(cut)) {
    at = (int)(before >> 16);
    pos += min(at, rank);
  }
  if constexpr (ALL) {
    if (topk_rare(cut)) {
      static_for<0, NE>([&](auto e) { at += lanes_below(__ballot(left[e] == b.lo)); });
      static_for<0, NE>([&](auto e) {
        if (left[e] == b.lo && at++ >= rank) left[e] = INT32_MIN;
      });
    }
    static_for<0, NE>([&](auto e) { pos += lanes_below(__ballot(left[e] >= b.lo)); });
    static_for<0, NE>([&](auto e) {
      if (left[e] >= b.lo) emit(pos++, first(0) + e);
    });
  } else {
    each([&](int v, auto e, bool) {
      bool take = v >= b.lo;
      if (topk_rare(cut)) {
        const uint64_t same = __ballot(v == b.lo);
        take = v > b.hi || (v == b.lo && at + lanes_below(same) < rank);
        at += __popcll(same);
      }
      const uint64_t taken = __ballot(take);
      if (take) emit(pos + lanes_below(taken), (int)S.page[wave][64 * e + lane]);
      pos += __popcll(taken);
    });
  }
}

// The same for any scores of at most 128 pages (64 with fewer than 8 wavefronts): a page's place is the
// number of pages in front of it, which every wavefront counts over its share of the pages.  One
// barrier, where the forms above cross four: 8 streams of 64 pages, 16 kept, 5.9 us per step for 6.3.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_few(const float* __restrict__ sc, int NP, int k,
                                         TopkLds<IPT, THREADS>& S, Emit emit) {
  constexpr int NW = THREADS / 64, E = NW < 8 ? 1 : 2;  // pages per lane
  static_assert(NW * E * 64 <= 4 * kTopkBins, "counts of all wavefronts");
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
  int* const counts = S.hist[0];
  static_for<0, E>([&](auto e) { counts[(wave * E + e) * 64 + lane] = ahead[e]; });
  __syncthreads();
  int pos = 0;
  static_for<0, E>([&](auto e) {
    int place = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) place += counts[(w * E + e) * 64 + lane];
    const bool t = e * 64 + lane < NP && place < k;
    const uint64_t m = __ballot(t);
    if (wave == e && t) emit(pos + lanes_below(m), e * 64 + lane);
    pos += __popcll(m);
  });
}

// Top-k pages of a stream by one workgroup of THREADS threads, NP <= THREADS * IPT <= 8192: ties to
// the lowest page, emit(position in the ascending list, page) for every selected one.  `sc` must not
// lie in `S`.
template <int IPT, int THREADS, class Emit>
__device__ __forceinline__ void topk_block(const float* __restrict__ sc, int NP, int k,
                                           TopkLds<IPT, THREADS>& S, Emit emit) {
  if (IPT > 2 ? topk_rare(NP <= 3) : NP <= (THREADS < 512 ? 64 : 128))
    topk_few<IPT, THREADS>(sc, NP, k, S, emit);
  else
    topk_keys<IPT, THREADS>(sc, NP, k, S, emit);
}

}  // namespace stc
