// Sub-token value-group routing at cache-build time (paper Sec. 3.3): top-k
// routing mask per token (or, for the LLM setting of Sec. 3.4 / App. B.1, the N*K
// best token-group pairs of the whole stream), per-token offsets into the
// group-packed store, and the packed copy of the kept value groups.
#include "build_helpers.hpp"
#include "stc_common.hpp"
#include "stc_kernels.hpp"

namespace stc {

typedef __attribute__((ext_vector_type(4))) uint32_t pack_u32x4;

constexpr int kChunk = 256;  // tokens per workgroup in the route / pack kernels

__device__ __forceinline__ int block_sum_256(int v, int* lds4) {
  // sum over a 256-thread block; every thread gets the total
  v = (int)wave_reduce((uint32_t)v, OpAdd{}, 0u);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds4[wave] = v;
  __syncthreads();
  const int tot = lds4[0] + lds4[1] + lds4[2] + lds4[3];
  __syncthreads();
  return tot;
}

// Exclusive prefix sum over a 256-thread block (in thread order).
__device__ __forceinline__ int block_exscan_256(int v, int* lds4, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = (int)wave_scan((uint32_t)v, OpAdd{}, 0u);
  if (lane == 63) lds4[wave] = inc;
  __syncthreads();
  const int a = lds4[0], b = lds4[1], c = lds4[2];
  const int base = (wave > 0 ? a : 0) + (wave > 1 ? b : 0) + (wave > 2 ? c : 0);
  if (total) *total = a + b + c + lds4[3];
  __syncthreads();
  return base + inc - v;
}

// Where the routing masks come from: given, or the best groups of each token's logits.
struct RouteInputs {
  int mode;
  const float* logits;
  const uint8_t* kcount;
  int fixed_k;
  const uint16_t* mask_in;  // may be the array that the masks are written to
  int share;                // streams that read one set of these
};

// Routing mask of token t (< N) of a stream.
template <bool STREAM>
__device__ __forceinline__ uint32_t route_token(const RouteInputs& in, int stream, int t, int N,
                                                int G) {
  const size_t tok = (size_t)(stream / in.share) * N + t;  // the inputs are dense
  if (in.mode == STC_ROUTE_MASK) return in.mask_in[tok] & ((1u << G) - 1u);
  const int c = in.kcount ? (int)in.kcount[tok] : in.fixed_k;
  return rank_mask<STREAM>(in.logits + tok * G, min(c, G), G);
}

// Step 1: routing mask of every token and the number of kept groups per chunk.  STREAM: logits
// that are read once and do not fit the caches go past them (64 streams of 32768 tokens, 67 MB of
// logits: 9 us less, this launch and the packed copy behind it together).
template <bool STREAM>
__global__ __launch_bounds__(kChunk) void route_mask_kernel(
    const float* logits, const uint8_t* kcount, uint16_t* mask, uint32_t* __restrict__ chunk_sum,
    int N, int G, int nchunks, int Ncap, int share, int mode, int fixed_k,
    const uint16_t* mask_in) {
  const RouteInputs in{mode, logits, kcount, fixed_k, mask_in, share};
  __shared__ int red[4];
  const int stream = blockIdx.y;
  const int t = blockIdx.x * kChunk + threadIdx.x;
  uint32_t m = 0;
  if (t < N) {
    m = route_token<STREAM>(in, stream, t, N, G);
    mask[(size_t)stream * Ncap + t] = (uint16_t)m;
  }
  const int tot = block_sum_256(__popc(m), red);
  if (threadIdx.x == 0) chunk_sum[(size_t)stream * nchunks + blockIdx.x] = (uint32_t)tot;
}

// ---------------------------------------------------------------------------
// Global token-group budget (Sec. 3.4; App. B.1: M = N*K of the N x S pairs): the key of the
// M-th largest of a stream's N*G logits by a radix select (12 + 10 + 10 bits; the wide first
// digit spreads logits that share sign and exponent over many bins), then every pair above
// that key is kept plus the first `remaining` pairs equal to it in (token, group) order.
// Every pass over the logits is spread over the whole chip: many workgroups per stream build
// the digit histogram (shared memory first, then one atomic per non-empty bin), one workgroup
// per stream picks the digit.  Per-stream state lives in the workspace.  ("Stream" below is one
// set of logits: with shared routing inputs the streams of a batch element have one selection.)
// Sets of few logits are selected by one workgroup in one launch (global_small_kernel).
// ---------------------------------------------------------------------------
constexpr int kGlobalThreads = 1024;
constexpr int kGlobalBins = 4096;
constexpr int kHistThreads = 256;
constexpr int kHistSlice = 16384;  // logits per histogram workgroup

struct GlobalState {
  uint32_t prefix;     // key bits fixed so far
  uint32_t decided;    // mask of those bits
  uint32_t remaining;  // rank of the wanted key among the keys that share the prefix
  uint32_t take_all;   // after the last pass: every pair equal to the key is kept
};

// Order-preserving key of a finite float with -0 and +0 mapped to one key.
__device__ __forceinline__ uint32_t logit_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix sum over a 1024-thread block (thread order); *total = block sum.
__device__ __forceinline__ uint32_t block_exscan_1024(uint32_t v, uint32_t* lds16,
                                                      uint32_t* total) {
  constexpr int NW = kGlobalThreads / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t inc = wave_scan(v, OpAdd{}, 0u);
  if (lane == 63) lds16[wave] = inc;
  __syncthreads();
  const uint32_t w = lane < NW ? lds16[lane] : 0u;  // every wavefront scans the wavefronts' sums
  const uint32_t winc = wave_scan(w, OpAdd{}, 0u);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)winc, NW - 1);
  const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)(winc - w), wave);
  __syncthreads();
  return base + inc - v;
}

__device__ __forceinline__ int global_shift(int pass) { return pass == 0 ? 20 : (pass == 1 ? 10 : 0); }
__device__ __forceinline__ uint32_t global_bins(int pass) { return pass == 0 ? 4096u : 1024u; }

// Start of a selection: empty histograms, nothing decided, rank = budget.
__global__ __launch_bounds__(256) void global_init_kernel(uint32_t* __restrict__ hist,
                                                          GlobalState* __restrict__ state,
                                                          int streams, uint32_t budget) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < streams * kGlobalBins) hist[i] = 0u;
  if (i < streams) state[i] = GlobalState{0u, 0u, budget, 0u};
}

// Histogram of digit `pass` over the keys that share the stream's prefix; workgroup
// blockIdx.x covers logits [blockIdx.x * slice, +slice) of stream blockIdx.y.
__global__ __launch_bounds__(kHistThreads) void global_hist_kernel(
    const float* __restrict__ logits, uint32_t* __restrict__ hist,
    const GlobalState* __restrict__ state, uint32_t n, uint32_t slice, int pass) {
  __shared__ uint32_t lh[kGlobalBins];
  const int stream = blockIdx.y;
  const int tid = threadIdx.x;
  const int shift = global_shift(pass);
  const uint32_t bins = global_bins(pass);
  const uint32_t prefix = state[stream].prefix, decided = state[stream].decided;
  for (uint32_t i = tid; i < bins; i += kHistThreads) lh[i] = 0u;
  __syncthreads();
  const float* a = logits + (size_t)stream * n;
  const uint32_t lo = blockIdx.x * slice, hi = n - lo < slice ? n : lo + slice;
  auto count = [&](float f) {
    const uint32_t key = logit_key(f);
    if ((key & decided) == prefix) atomicAdd(&lh[(key >> shift) & (bins - 1)], 1u);
  };
  if ((n & 3u) == 0) {  // every stream and slice starts on a 16-byte boundary
    for (uint32_t i = lo + 4 * tid; i < hi; i += 4 * kHistThreads) {
      const float4 v = *(const float4*)(a + i);
      count(v.x), count(v.y), count(v.z), count(v.w);
    }
  } else {
    for (uint32_t i = lo + tid; i < hi; i += kHistThreads) count(a[i]);
  }
  __syncthreads();
  uint32_t* gh = hist + (size_t)stream * kGlobalBins;
  for (uint32_t i = tid; i < bins; i += kHistThreads) {
    const uint32_t c = lh[i];
    if (c) atomicAdd(&gh[i], c);
  }
}

// The digit that holds the wanted key: block scan over the stream's histogram in descending
// digit order.  Leaves the histogram empty for the next pass.
__global__ __launch_bounds__(kGlobalThreads) void global_pick_kernel(
    uint32_t* __restrict__ hist, GlobalState* __restrict__ state, int pass) {
  __shared__ uint32_t waves[kGlobalThreads / 64];
  const int stream = blockIdx.x;
  const int tid = threadIdx.x;
  const int shift = global_shift(pass);
  const uint32_t bins = global_bins(pass);
  uint32_t* gh = hist + (size_t)stream * kGlobalBins;
  const GlobalState st = state[stream];
  // thread t owns the 4 adjacent digits 4095-4t .. 4092-4t (descending order)
  uint32_t c[4], own = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t d = kGlobalBins - 1 - (4 * tid + j);
    c[j] = d < bins ? gh[d] : 0u;
    if (d < bins) gh[d] = 0u;
    own += c[j];
  }
  uint32_t tot;
  uint32_t above = block_exscan_1024(own, waves, &tot);  // pairs with a larger digit
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (above < st.remaining && st.remaining <= above + c[j]) {
      GlobalState nx;
      nx.prefix = st.prefix | ((uint32_t)(kGlobalBins - 1 - (4 * tid + j)) << shift);
      nx.decided = st.decided | ((bins - 1) << shift);
      nx.remaining = st.remaining - above;
      nx.take_all = nx.remaining == c[j] ? 1u : 0u;
      state[stream] = nx;
    }
    above += c[j];
  }
}

// Pairs equal to the stream's key per chunk of 256 tokens (the chunks of the mask kernel).
__global__ __launch_bounds__(kChunk) void global_eq_kernel(const float* __restrict__ logits,
                                                           const GlobalState* __restrict__ state,
                                                           uint32_t* __restrict__ chunk_eq, int N,
                                                           int G, int nchunks) {
  __shared__ int red[4];
  const int stream = blockIdx.y;
  if (state[stream].take_all) return;  // no ranks among equal pairs needed
  const uint32_t key = state[stream].prefix;
  const uint32_t n = (uint32_t)N * (uint32_t)G;
  const float* a = logits + (size_t)stream * n;
  const uint32_t lo = (uint32_t)blockIdx.x * kChunk * G;
  const uint32_t hi = n - lo < (uint32_t)kChunk * G ? n : lo + (uint32_t)kChunk * G;
  int eq = 0;
  for (uint32_t i = lo + threadIdx.x; i < hi; i += kChunk) eq += logit_key(a[i]) == key;
  const int tot = block_sum_256(eq, red);
  if (threadIdx.x == 0) chunk_eq[(size_t)stream * nchunks + blockIdx.x] = (uint32_t)tot;
}

// Exclusive scan of a stream's per-chunk counts, in place.
__global__ __launch_bounds__(256) void global_eq_scan_kernel(uint32_t* chunk_eq,
                                                             const GlobalState* __restrict__ state,
                                                             int nchunks) {
  __shared__ int red[4];
  if (state[blockIdx.x].take_all) return;
  uint32_t* cs = chunk_eq + (size_t)blockIdx.x * nchunks;
  int carry = 0;
  for (int base = 0; base < nchunks; base += 256) {
    const int i = base + threadIdx.x;
    const int v = i < nchunks ? (int)cs[i] : 0;
    int tot;
    const int ex = block_exscan_256(v, red, &tot);
    if (i < nchunks) cs[i] = (uint32_t)(carry + ex);
    carry += tot;
  }
}

// Masks of a chunk of 256 tokens from the stream's key: pairs above it, and the first
// `remaining` pairs equal to it in (token, group) order.  Also the chunk's number of kept
// groups, as route_mask_kernel writes it.  budget == 0 keeps nothing.
template <int G>
__global__ __launch_bounds__(kChunk) void global_mask_kernel(
    const float* __restrict__ logits, const GlobalState* __restrict__ state,
    const uint32_t* __restrict__ chunk_eq, uint16_t* __restrict__ mask,
    uint32_t* __restrict__ chunk_sum, int N, int nchunks, int Ncap, uint32_t budget, int share) {
  __shared__ int red[4];
  const int stream = blockIdx.y;
  const int t = blockIdx.x * kChunk + threadIdx.x;
  const int set = stream / share;  // streams that share a set of logits share its selection
  const GlobalState gs = state[set];
  const uint32_t prefix = gs.prefix, remaining = gs.remaining;
  const bool ranked = budget > 0 && !gs.take_all;  // equal pairs are taken in order
  float lg[G];
  load_token_logits<G>(logits + ((size_t)set * N + min(t, N - 1)) * G, lg);
  uint32_t key[G];
  int eq = 0;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    key[g] = t < N ? logit_key(lg[g]) : 0u;
    eq += (t < N && ranked) && key[g] == prefix;
  }
  uint32_t e = (ranked ? chunk_eq[(size_t)set * nchunks + blockIdx.x] : 0u) +
               (uint32_t)block_exscan_256(eq, red, nullptr);
  uint32_t m = 0;
  if (budget > 0 && t < N) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (key[g] > prefix) m |= 1u << g;
      else if (key[g] == prefix && (!ranked || e++ < remaining)) m |= 1u << g;
    }
  }
  if (t < N) mask[(size_t)stream * Ncap + t] = (uint16_t)m;
  const int tot = block_sum_256(__popc(m), red);
  if (threadIdx.x == 0) chunk_sum[(size_t)stream * nchunks + blockIdx.x] = (uint32_t)tot;
}

// The whole selection of one set of logits, masks and chunk sums of every gridDim.y-th stream of
// the set included, by one workgroup with the keys in registers: thread i owns the tokens i,
// i + 1024, ...  Same order among equal keys as the kernels above.
//
// Bins of equal width between the smallest and the largest logit, and the keys of the wanted one's bin
// ranked one by one.  Logits that crowd a few bins cost more, because their atomics wait for each
// other and the bin holds too many keys: a wavefront that sees a crowd counts it by ballots, and the
// bin's own smallest and largest key end the search (one value) or give a second set of bins.  What
// crowds those too differs in scale and goes digit by digit, as do ranges that float cannot divide.
// Bound by latency (histograms in LDS, block scans) and by instruction issue of the one CU.
// Routing and packing, us, as one selection per stream in nine launches over the chip / in this form
// with digits wherever the first bins fail and every key an atomic / with bins in the bin and crowds
// counted / now, with scans and reductions on the DPP path and the wanted bin's keys found by a range
// of keys instead of every key's bin once more:
//                        normal       halves         all equal      1 in 10 at -1e9  outliers x 1e4
//   8 sets of 32768,
//   32 streams each   87/56/56/53  98/91/73/66   151/131/46/41   85/85/66/62      87/89/65/61
//   4 sets of 65536   45/27/27/23  48/97/62/53    75/196/27/19   45/85/47/42      45/90/50/45
//   8 sets of 1200    32/11/11/10  33/19/19/16    34/20/12/9     32/18/16/13      32/43/16/13
// So sets of 65536 logits rounded to few values are the one case that the launches over the chip do
// faster; logits of a linear map are not like that.
constexpr int kSmallTokens = 16384;
// Of the first keys of a wavefront, this many in one bin are a crowd (normal logits: 0.05 expected).
constexpr int kGlobalCrowd = 6;
// Keys of a bin that are ranked one by one: more are slower that way than in further bins (1199 of
// 1200 logits: 43 us, 16 with further bins) or by digits (900 of 65536: 74 us, 57 by digits).
constexpr uint32_t kGlobalRanked = 256;

template <int G, int KPT>
__global__ __launch_bounds__(kGlobalThreads) void global_small_kernel(
    const float* __restrict__ logits, uint16_t* __restrict__ mask,
    uint32_t* __restrict__ chunk_sum, int N, int nchunks, int Ncap, uint32_t budget, int share) {
  constexpr int TPT = KPT / G;  // tokens per thread: tid, tid + 1024, ...
  static_assert(TPT * kGlobalThreads <= kSmallTokens, "masks and chunk counters in LDS");
  __shared__ uint32_t hist[kGlobalBins];
  __shared__ uint32_t waves[kGlobalThreads / 64];
  __shared__ uint32_t s_pick[3];  // digit, rank inside it, keys that have it
  __shared__ uint32_t s_count, s_crowd;
  __shared__ __align__(4) uint16_t s_mask[kSmallTokens];
  __shared__ uint32_t s_chunk[kSmallTokens / kChunk];
  const int tid = threadIdx.x;
  auto token = [&](int i) { return i * kGlobalThreads + tid; };
  const float* a = logits + (size_t)blockIdx.x * N * G;
  uint32_t key[TPT][G];
#pragma unroll
  for (int i = 0; i < TPT; ++i) {
    float lg[G];
    load_token_logits<G>(a + (size_t)min(token(i), N - 1) * G, lg);
#pragma unroll
    for (int g = 0; g < G; ++g) key[i][g] = logit_key(lg[g]);
  }
  for (int i = tid; i < kSmallTokens / kChunk; i += kGlobalThreads) s_chunk[i] = 0u;
  uint32_t prefix = 0u, decided = 0u, remaining = budget;
  bool take_all = false, found = false;
  // Bins of equal width spread the keys over the histogram (a digit of the key's bits puts logits
  // that share sign and exponent into a few bins).  The bin is monotone in the logit.
  float lo = 0.f, scale = 0.f;
  uint32_t bin_of_kth = 0u;
  auto bin = [&](uint32_t k) -> uint32_t {
    const float f = __uint_as_float(~(k ^ ((uint32_t)((int)k >> 31) >> 1)));  // value of the key
    return min((uint32_t)((f - lo) * scale), (uint32_t)(kGlobalBins - 1));
  };
  // The bin that holds the key of rank `remaining` among those in the histogram, that rank in the
  // bin, and its number of keys -> s_pick.  Thread t owns the 4 adjacent bins 4095-4t .. 4092-4t
  // (descending order).
  auto pick = [&]() __attribute__((always_inline)) {
    uint32_t c[4], own = 0, tot;
#pragma unroll
    for (int j = 0; j < 4; ++j) own += c[j] = hist[kGlobalBins - 1 - (4 * tid + j)];
    uint32_t above = block_exscan_1024(own, waves, &tot);  // keys in larger bins
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (above < remaining && remaining <= above + c[j]) {
        s_pick[0] = (uint32_t)(kGlobalBins - 1 - (4 * tid + j));
        s_pick[1] = remaining - above;
        s_pick[2] = c[j];
      }
      above += c[j];
    }
    __syncthreads();
  };
  // The wanted key among the `cnt` keys listed in hist, one per thread.
  auto rank = [&](uint32_t cnt) __attribute__((always_inline)) {
    __syncthreads();
    found = true;
    if (cnt <= 64 && tid < 64) {  // one wavefront, a key per lane
      const uint32_t mine = hist[tid];
      uint32_t gt = 0, ge = 0;
      for (int j = 0; j < (int)cnt; ++j) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)mine, j);
        gt += o > mine, ge += o >= mine;
      }
      if (tid < (int)cnt && gt < remaining && remaining <= ge)  // equal keys agree
        s_pick[0] = mine, s_pick[1] = remaining - gt, s_pick[2] = ge - gt;
    }
    if (cnt > 64 && tid < (int)cnt) {
      const uint32_t mine = hist[tid];
      uint32_t gt = 0, ge = 0;
      for (uint32_t j = 0; j < cnt; ++j) gt += hist[j] > mine, ge += hist[j] >= mine;
      if (gt < remaining && remaining <= ge)  // equal keys agree
        s_pick[0] = mine, s_pick[1] = remaining - gt, s_pick[2] = ge - gt;
    }
    __syncthreads();
    prefix = s_pick[0];
    remaining = s_pick[1];
    take_all = s_pick[1] == s_pick[2];
  };
  // Smallest of the threads' kmin and largest of their kmax, through hist.
  auto block_range = [&](uint32_t& kmin, uint32_t& kmax) __attribute__((always_inline)) {
    constexpr int NW = kGlobalThreads / 64;
    const int lane = tid & 63;
    kmin = wave_reduce(kmin, OpMin{}, 0xffffffffu);
    kmax = wave_reduce(kmax, OpMax{}, 0u);
    if (lane == 0) hist[tid >> 6] = kmin, hist[64 + (tid >> 6)] = kmax;
    __syncthreads();
    kmin = wave_reduce(hist[lane & (NW - 1)], OpMin{}, 0xffffffffu);
    kmax = wave_reduce(hist[64 + (lane & (NW - 1))], OpMax{}, 0u);
    __syncthreads();
  };
  auto value = [](uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k); };
  if (budget > 0) {
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int i = 0; i < TPT; ++i)
#pragma unroll
      for (int g = 0; g < G; ++g) kmin = min(kmin, key[i][g]), kmax = max(kmax, key[i][g]);
    block_range(kmin, kmax);
    lo = value(kmin);
    const float hi = value(kmax);
    scale = (float)(kGlobalBins - 1) / (hi - lo);
    if (kmin == kmax) {  // one value everywhere
      prefix = kmin;
      take_all = remaining == (uint32_t)N * G;
      found = true;
    }
    // a range that float cannot divide: every key is in bin 0
    if (!(hi > lo) || !(hi - lo < 3.0e38f) || !(scale < 3.0e38f)) lo = 0.f, scale = 0.f;
  }
  if (budget > 0 && scale > 0.f) {
#pragma unroll
    for (int j = 0; j < kGlobalBins / kGlobalThreads; ++j) hist[j * kGlobalThreads + tid] = 0u;
    if (tid == 0) s_count = 0u, s_crowd = 0u;
    __syncthreads();
    // A wavefront in which many of the first keys share a bin counts its keys in it without atomics.
    const int first = token(0) < N ? (int)bin(key[0][0]) : -1;
    const int crowd = __builtin_amdgcn_readfirstlane(first);
    if (__builtin_expect(crowd >= 0 && __popcll(__ballot(first == crowd)) >= kGlobalCrowd, 0)) {
      uint32_t crowded = 0;
#pragma unroll
      for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int b = token(i) < N ? (int)bin(key[i][g]) : -1;
          crowded += __popcll(__ballot(b == crowd));
          if (b >= 0 && b != crowd) atomicAdd(&hist[b], 1u);
        }
      if ((tid & 63) == 0) atomicAdd(&hist[crowd], crowded);
    } else {
#pragma unroll
      for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (token(i) < N) atomicAdd(&hist[bin(key[i][g])], 1u);
    }
    __syncthreads();
    pick();
    bin_of_kth = s_pick[0];
    remaining = s_pick[1];
    const uint32_t cnt = s_pick[2];
    if (cnt <= kGlobalRanked) {
      // Keys from a little below the wanted bin to a little above it: a superset of the bin's, as
      // 1/64 is more than the rounding of a bin's number (below 2^-10), and rounding is monotone.
      const float at = (float)bin_of_kth;
      const uint32_t k0 = logit_key(lo + (at - 0.015625f) / scale);
      const uint32_t near = logit_key(lo + (at + 1.015625f) / scale) - k0;
#pragma unroll
      for (int i = 0; i < TPT; ++i) {
        uint32_t any = 0u;
        static_for<0, G>([&](auto g) { any |= key[i][g] - k0 <= near ? 1u << g : 0u; });
        if (token(i) >= N) any = 0u;
        for (; any; any &= any - 1u) {
          const uint32_t k = pick_of(key[i], __ffs((int)any) - 1);
          if (bin(k) == bin_of_kth) hist[atomicAdd(&s_count, 1u)] = k;
        }
      }
      rank(cnt);
    }
  }
  if (__builtin_expect(budget > 0 && !found, 0)) {
    uint32_t klo = 0u, khi = 0xffffffffu;  // the wanted key is in [klo, khi]
    if (scale > 0.f) {
      // The smallest and the largest key of the bin: it may be one value, and if not, bins between
      // these two spread its keys.
      klo = 0xffffffffu, khi = 0u;
#pragma unroll
      for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (token(i) < N && bin(key[i][g]) == bin_of_kth)
            klo = min(klo, key[i][g]), khi = max(khi, key[i][g]);
      block_range(klo, khi);
      if (klo == khi) {
        prefix = klo;
        take_all = remaining == s_pick[2];
        found = true;
      }
      const float lo2 = value(klo), scale2 = (float)(kGlobalBins - 1) / (value(khi) - lo2);
      auto in_bin = [&](int i, int g) {
        return token(i) < N && key[i][g] >= klo && key[i][g] <= khi;
      };
      auto bin2 = [&](uint32_t k) -> uint32_t {  // of such a key
        return min((uint32_t)((value(k) - lo2) * scale2), (uint32_t)(kGlobalBins - 1));
      };
      bool spread = !found && scale2 < 3.0e38f;
      if (spread) {
#pragma unroll
        for (int j = 0; j < kGlobalBins / kGlobalThreads; ++j) hist[j * kGlobalThreads + tid] = 0u;
        // where a wavefront's keys crowd a bin again, the logits differ in scale: digits spread them
        const int first = in_bin(0, 0) ? (int)bin2(key[0][0]) : -1;
        const uint64_t any = __ballot(first >= 0);
        const int crowd = __builtin_amdgcn_readlane(first, any ? __ffsll((long long)any) - 1 : 0);
        if (any && __popcll(__ballot(first == crowd)) >= kGlobalCrowd) s_crowd = 1u;
        __syncthreads();
        spread = s_crowd == 0u;
      }
      if (spread) {
        const uint32_t rank_in_bin = remaining;
#pragma unroll
        for (int i = 0; i < TPT; ++i)
#pragma unroll
          for (int g = 0; g < G; ++g)
            if (in_bin(i, g)) atomicAdd(&hist[bin2(key[i][g])], 1u);
        __syncthreads();
        pick();
        const uint32_t b = s_pick[0], cnt = s_pick[2];
        remaining = s_pick[1];
        if (cnt <= kGlobalRanked) {
#pragma unroll
          for (int i = 0; i < TPT; ++i)
#pragma unroll
            for (int g = 0; g < G; ++g)
              if (in_bin(i, g) && bin2(key[i][g]) == b)
                hist[atomicAdd(&s_count, 1u)] = key[i][g];
          rank(cnt);
        } else {
          remaining = rank_in_bin;
        }
      }
    }
    for (int pass = 0; pass < 3 && !found; ++pass) {
      const int shift = global_shift(pass);
      const uint32_t bins = global_bins(pass);
#pragma unroll
      for (int j = 0; j < kGlobalBins / kGlobalThreads; ++j) hist[j * kGlobalThreads + tid] = 0u;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (token(i) < N && (key[i][g] & decided) == prefix && key[i][g] >= klo &&
              key[i][g] <= khi)
            atomicAdd(&hist[(key[i][g] >> shift) & (bins - 1)], 1u);
      __syncthreads();
      pick();  // (bins past `bins` are empty)
      prefix |= s_pick[0] << shift;
      decided |= (bins - 1) << shift;
      remaining = s_pick[1];
      take_all = s_pick[1] == s_pick[2];
    }
  }
  if (budget == 0 || take_all) __syncthreads();  // (no scan below: the chunk counters are cleared)
  uint32_t before = 0;  // equal keys of tokens in front of the current 1024
#pragma unroll
  for (int i = 0; i < TPT; ++i) {
    const int t = token(i);
    uint32_t m = 0, e = 0;
    if (budget > 0) {
      if (!take_all) {  // equal keys are taken in token order
        uint32_t eq = 0, tot;
#pragma unroll
        for (int g = 0; g < G; ++g) eq += t < N && key[i][g] == prefix;
        e = before + block_exscan_1024(eq, waves, &tot);
        before += tot;
      }
      if (take_all) {
#pragma unroll
        for (int g = 0; g < G; ++g) m |= key[i][g] >= prefix ? 1u << g : 0u;
        if (t >= N) m = 0;
      } else if (t < N) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (key[i][g] > prefix) m |= 1u << g;
          else if (key[i][g] == prefix && e++ < remaining) m |= 1u << g;
        }
      }
    }
    if (t < N) s_mask[t] = (uint16_t)m;
    // the 64 tokens of a wavefront lie in one chunk
    const uint32_t kept = wave_reduce((uint32_t)__popc(m), OpAdd{}, 0u);
    if ((tid & 63) == 0 && kept) atomicAdd(&s_chunk[t / kChunk], kept);
  }
  __syncthreads();
  for (int r = blockIdx.y; r < share; r += gridDim.y) {
    const size_t stream = (size_t)blockIdx.x * share + r;
    uint16_t* dst = mask + stream * Ncap;
    if ((Ncap & 1) == 0) {  // two masks at a time
      for (int i = tid; i < N / 2; i += kGlobalThreads) ((uint32_t*)dst)[i] = ((uint32_t*)s_mask)[i];
      if ((N & 1) && tid == 0) dst[N - 1] = s_mask[N - 1];
    } else {
      for (int i = tid; i < N; i += kGlobalThreads) dst[i] = s_mask[i];
    }
    for (int i = tid; i < nchunks; i += kGlobalThreads)
      chunk_sum[stream * nchunks + i] = s_chunk[i];
  }
}

// Step 2: per stream, exclusive scan of the chunk sums (in place); writes the
// stream total to tok_off[N] and flags a packed store that is too small.
__global__ __launch_bounds__(256) void scan_chunks_kernel(uint32_t* chunk_sum, uint32_t* tok_off,
                                                          int32_t* dev_status, int N, int nchunks,
                                                          long long cap, int Ncap) {
  __shared__ int red[4];
  const int stream = blockIdx.x;
  uint32_t* cs = chunk_sum + (size_t)stream * nchunks;
  int carry = 0;
  for (int base = 0; base < nchunks; base += 256) {
    const int i = base + threadIdx.x;
    const int v = i < nchunks ? (int)cs[i] : 0;
    int tot;
    const int ex = block_exscan_256(v, red, &tot);
    if (i < nchunks) cs[i] = (uint32_t)(carry + ex);
    carry += tot;
  }
  if (threadIdx.x == 0) {
    tok_off[(size_t)stream * (Ncap + 1) + N] = (uint32_t)carry;
    if (dev_status && (long long)carry > cap) *dev_status = 1;
  }
}

// Step 3: per-token offsets, then the packed copy, kPackTokens tokens per workgroup.  The kept
// pieces of V are read as they lie (streaming loads, 16 bytes per lane), put next to each other
// in LDS and written from there as one contiguous run that starts on whole 128-byte lines
// (streaming stores: nothing here is read again, and lines written completely need no
// merging in the caches).
// Bound by memory.  Measured on 64 streams of 32768 tokens, 8 groups, half of them kept
// (805 MB): 116 us (6.9 TB/s); 122 while the scan of a workgroup's counts went through shuffles and
// its arguments were loaded when it started, 158 for the form before that, in which every lane
// stored its piece where it belongs, 256 tokens per workgroup, through the caches.  (Against 122:
// 128 tokens per workgroup 128 us, 32: 132, with the values requested before the masks are known
// 129, with streaming loads or streaming stores alone 143 and 141.)
// What is in front of a workgroup's tokens, by FORM:
//   kPackSums     chunk_sum holds the chunks' own sums, and every workgroup adds up those in front
//                 of its chunk itself
//   kPackScanned  they have been scanned by a launch of its own, which also wrote the totals
//   kPackRoute    streams of a single chunk (256 tokens): the workgroup routes its tokens and those
//                 in front of them itself, so that no launch for the masks is needed (64 x 32
//                 streams of 208 tokens, compaction and bounds included: 129.5 us for 134.5)
enum { kPackSums, kPackScanned, kPackRoute };
constexpr int kPackTokens = 64;

template <int D, int FORM>
__global__ __launch_bounds__(kChunk) void pack_kernel(
    const float* logits, const uint8_t* kcount, uint16_t* mask,
    const pack_u32x4* __restrict__ V, const uint32_t* __restrict__ chunk_sum, int N, int G,
    int nchunks, int Ncap, int share, int mode, int fixed_k, const uint16_t* mask_in,
    uint32_t* __restrict__ tok_off, pack_u32x4* __restrict__ vpacked, int32_t* dev_status,
    long long cap) {
  const RouteInputs in{mode, logits, kcount, fixed_k, mask_in, share};
  constexpr int PPT = D / 8;                         // 16-byte pieces per token row
  constexpr int PER = kPackTokens * PPT / kChunk;    // pieces per thread
  __shared__ int red[4], red2[4];
  __shared__ uint32_t s_off[kPackTokens + 1];
  __shared__ uint32_t s_mask[kPackTokens];
  __shared__ __align__(16) pack_u32x4 s_run[kPackTokens * PPT];
  const int stream = blockIdx.y;
  const int t0 = blockIdx.x * kPackTokens;
  const int chunk = t0 / kChunk;
  uint32_t* off_s = tok_off + (size_t)stream * (Ncap + 1);
  // thread i looks at token i of the chunk, up to the end of this workgroup's tokens
  const int t = chunk * kChunk + threadIdx.x;
  uint16_t* mask_t = mask + (size_t)stream * Ncap + t;
  uint32_t m = 0, before = 0;  // the token's mask; kept groups in front of the chunk
  if (t < N && t < t0 + kPackTokens) {
    if constexpr (FORM == kPackRoute) {
      m = route_token<false>(in, stream, t, N, G);
      if (t >= t0) *mask_t = (uint16_t)m;
    } else {
      m = *mask_t;
    }
  }
  if constexpr (FORM != kPackRoute) {
    const uint32_t* cs = chunk_sum + (size_t)stream * nchunks;
    if constexpr (FORM == kPackSums) {
      uint32_t part = 0;
      for (int i = threadIdx.x; i < chunk; i += kChunk) part += cs[i];
      before = (uint32_t)block_sum_256((int)part, red2);
    } else {
      before = cs[chunk];
    }
  }
  int upto;
  const int ex = block_exscan_256(__popc(m), red, &upto);
  const uint32_t off = before + (uint32_t)ex;
  const uint32_t end = before + (uint32_t)upto;
  const int rel = t - t0;
  if (rel >= 0 && rel < kPackTokens) {
    if (t < N) off_s[t] = off;
    s_off[rel] = off;
    s_mask[rel] = m;  // 0 behind the last token
  }
  if (threadIdx.x == 0 && FORM != kPackScanned && t0 + kPackTokens >= N) {
    off_s[N] = end;
    if (dev_status && (long long)end > cap) *dev_status = 1;
  }
  __syncthreads();
  const int lg_ppg = 31 - __clz(PPT / G);  // log2(pieces per group)
  const pack_u32x4* src = V + ((size_t)stream * N + t0) * PPT;
  const uint32_t base = s_off[0];
  pack_u32x4 v[PER];
  int at[PER];  // place in the run, -1: dropped
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = i * kChunk + threadIdx.x;
    const int tok = e / PPT, pc = e % PPT;
    const int g = pc >> lg_ppg, within = pc - (g << lg_ppg);
    const uint32_t mk = s_mask[tok];
    const bool kept = (mk >> g) & 1u;
    const uint32_t slot = s_off[tok] - base + __popc(mk & ((1u << g) - 1u));
    at[i] = kept ? (int)((slot << lg_ppg) + within) : -1;
    // a dropped piece reads the workgroup's first one instead, so that the loads stay together
    v[i] = __builtin_nontemporal_load(src + (kept ? e : 0));
  }
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (at[i] >= 0) s_run[at[i]] = v[i];
  __syncthreads();
  const long long lim = (min((long long)end, cap) - (long long)base) * (1 << lg_ppg);
  pack_u32x4* dst = vpacked + (((size_t)stream * (size_t)cap + base) << lg_ppg);
  const int skew = (int)((reinterpret_cast<uintptr_t>(dst) >> 4) & 7);  // pieces into a line
  for (int o = (int)threadIdx.x - skew; o < lim; o += kChunk)
    if (o >= 0) __builtin_nontemporal_store(s_run[o], dst + o);
}

// Row gather used to compact a cache to the tokens a token-level method kept.
template <int D>
__global__ __launch_bounds__(256) void compact_kernel(const uint4* __restrict__ src,
                                                      const int32_t* __restrict__ token_idx,
                                                      uint4* __restrict__ dst, int Hkv, int N_src,
                                                      int n_keep, int32_t* dev_status) {
  constexpr int PPT = D / 8;
  const int stream = blockIdx.y, b = stream / Hkv;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= n_keep * PPT) return;
  const int i = e / PPT, pc = e % PPT;
  const int t = token_idx[(size_t)b * n_keep + i];
  uint4 v = make_uint4(0, 0, 0, 0);
  if (t >= 0 && t < N_src) {
    v = src[((size_t)stream * N_src + t) * PPT + pc];
  } else if (dev_status && pc == 0) {
    *dev_status = 1;
  }
  dst[((size_t)stream * n_keep + i) * PPT + pc] = v;
}

namespace {

// Workspace: kept groups per chunk, then (global budget only) equal-key counts per chunk,
// the per-stream digit histograms and the per-stream selection state.
struct RouteWs {
  size_t chunk_sum, chunk_eq, hist, state, total;
};

RouteWs route_ws_layout(const stc_shape_t& s) {
  const size_t streams = (size_t)s.B * s.Hkv;
  const size_t nchunks = (s.N + kChunk - 1) / kChunk;
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  RouteWs w;
  w.chunk_sum = 0;
  w.chunk_eq = up(streams * nchunks * sizeof(uint32_t));
  w.hist = w.chunk_eq + up(streams * nchunks * sizeof(uint32_t));
  w.state = w.hist + up(streams * kGlobalBins * sizeof(uint32_t));
  w.total = w.state + up(streams * sizeof(GlobalState));
  return w;
}

}  // namespace

size_t route_ws_bytes(const stc_shape_t& s) { return route_ws_layout(s).total; }

int launch_route_pack(const stc_shape_t& s, int mode, const void* V, const float* logits,
                      const uint8_t* kcount, int fixed_k, const uint16_t* mask_in, uint16_t* mask,
                      uint32_t* tok_off, void* vpacked, int32_t* dev_status, void* ws,
                      hipStream_t st) {
  // STC_ROUTE_SHARED: one set of routing inputs per batch element, read by all its KV heads
  const int share = (mode & STC_ROUTE_SHARED) ? s.Hkv : 1;
  mode &= ~STC_ROUTE_SHARED;
  const int streams = s.B * s.Hkv;
  const int nchunks = (s.N + kChunk - 1) / kChunk;
  const int Ncap = token_cap(s);  // stride of mask and tok_off; V, logits, kcount are dense
  const RouteWs lay = route_ws_layout(s);
  uint32_t* chunk = (uint32_t*)((char*)ws + lay.chunk_sum);
  dim3 grid(nchunks, streams);
  bool in_pack = false;  // the packed copy routes the tokens itself
  if (mode == STC_ROUTE_GLOBAL) {
    uint32_t* chunk_eq = (uint32_t*)((char*)ws + lay.chunk_eq);
    uint32_t* hist = (uint32_t*)((char*)ws + lay.hist);
    GlobalState* state = (GlobalState*)((char*)ws + lay.state);
    const uint32_t budget = (uint32_t)((long long)s.N * fixed_k);
    const uint32_t n = (uint32_t)s.N * (uint32_t)s.G;
    const int sets = streams / share;
    // one workgroup holds the keys of a set (16, 32 or 64 per thread) and its masks
    if (n <= 64u * kGlobalThreads && s.N <= kSmallTokens) {
      // the streams of a set are shared out among workgroups that each repeat the selection, as
      // long as there are CUs for them: one CU takes long to write many streams' masks
      const int parts = max(1, min(share, 256 / sets));
#define STC_GLOBAL_SMALL(GG, KPT)                                                             \
  if constexpr (KPT / GG * kGlobalThreads <= kSmallTokens)                                    \
  global_small_kernel<GG, KPT><<<dim3(sets, parts), kGlobalThreads, 0, st>>>(                 \
      logits, mask, chunk, s.N, nchunks, Ncap, budget, share)
#define STC_GLOBAL_SMALL_CASE(GG)                                                             \
  case GG:                                                                                    \
    if (n <= 16u * kGlobalThreads) { STC_GLOBAL_SMALL(GG, 16); }                              \
    else if (n <= 32u * kGlobalThreads) { STC_GLOBAL_SMALL(GG, 32); }                         \
    else { STC_GLOBAL_SMALL(GG, 64); }                                                        \
    break;
      switch (s.G) {
        STC_GLOBAL_SMALL_CASE(1)
        STC_GLOBAL_SMALL_CASE(2)
        STC_GLOBAL_SMALL_CASE(4)
        STC_GLOBAL_SMALL_CASE(8)
        STC_GLOBAL_SMALL_CASE(16)
        default:
          return -1;
      }
#undef STC_GLOBAL_SMALL_CASE
#undef STC_GLOBAL_SMALL
    } else {
      global_init_kernel<<<(sets * kGlobalBins + 255) / 256, 256, 0, st>>>(hist, state, sets,
                                                                           budget);
      if (budget > 0) {
        dim3 hgrid((unsigned)(((unsigned long long)n + kHistSlice - 1) / kHistSlice), sets);
        for (int pass = 0; pass < 3; ++pass) {
          global_hist_kernel<<<hgrid, kHistThreads, 0, st>>>(logits, hist, state, n, kHistSlice,
                                                             pass);
          global_pick_kernel<<<sets, kGlobalThreads, 0, st>>>(hist, state, pass);
        }
        global_eq_kernel<<<dim3(nchunks, sets), kChunk, 0, st>>>(logits, state, chunk_eq, s.N, s.G,
                                                                 nchunks);
        global_eq_scan_kernel<<<sets, 256, 0, st>>>(chunk_eq, state, nchunks);
      }
#define STC_GLOBAL_MASK(GG)                                                                   \
  case GG:                                                                                    \
    global_mask_kernel<GG><<<grid, kChunk, 0, st>>>(logits, state, chunk_eq, mask, chunk, s.N, \
                                                    nchunks, Ncap, budget, share);            \
    break;
      switch (s.G) {
        STC_GLOBAL_MASK(1)
        STC_GLOBAL_MASK(2)
        STC_GLOBAL_MASK(4)
        STC_GLOBAL_MASK(8)
        STC_GLOBAL_MASK(16)
        default:
          return -1;
      }
#undef STC_GLOBAL_MASK
    }
  } else {
    in_pack = nchunks == 1;
    if (!in_pack) {
      // logits that several streams read come from the caches after the first
      const bool stream_loads = mode == STC_ROUTE_TOPK && share == 1 &&
                                (long long)streams * s.N * s.G * 4 >= (32ll << 20);
      if (stream_loads)
        route_mask_kernel<true><<<grid, kChunk, 0, st>>>(logits, kcount, mask, chunk, s.N, s.G, nchunks,
                                                    Ncap, share, mode, fixed_k, mask_in);
      else
        route_mask_kernel<false><<<grid, kChunk, 0, st>>>(logits, kcount, mask, chunk, s.N, s.G, nchunks,
                                                      Ncap, share, mode, fixed_k, mask_in);
    }
  }
  if (hipGetLastError() != hipSuccess) return -1;
  // Up to this many chunks per stream (524288 tokens) a workgroup of the packed copy adds up
  // the sums in front of its chunk itself, which costs less than a launch in between: us, added up
  // / scanned, 256 streams of 2 chunks 9.0 / 11.0, 64 of 16 23.4 / 24.7, 8 of 512 77.3 / 78.7, 2 of
  // 2048 78.0 / 82.0, one of 2048 42.3 / 46.8.  At 4096 the reads of the sums begin to count: 151 / 154,
  // at D = 64 103 / 99.
  constexpr int kScanInPackChunks = 2048;
  const bool fold = nchunks <= kScanInPackChunks;
  if (!fold) {
    scan_chunks_kernel<<<streams, 256, 0, st>>>(chunk, tok_off, dev_status, s.N, nchunks,
                                                (long long)s.v_cap_groups, Ncap);
    if (hipGetLastError() != hipSuccess) return -1;
  }
  dim3 pgrid((s.N + kPackTokens - 1) / kPackTokens, streams);
#define STC_PACK(DD, FORM)                                                                    \
  pack_kernel<DD, FORM><<<pgrid, kChunk, 0, st>>>(                                            \
      logits, kcount, mask, (const pack_u32x4*)V, chunk, s.N, s.G, nchunks, Ncap, share, mode, \
      fixed_k, mask_in, tok_off, (pack_u32x4*)vpacked, dev_status, (long long)s.v_cap_groups)
#define STC_PACK_FORMS(DD)                                                                    \
  if (in_pack) STC_PACK(DD, kPackRoute);                                                      \
  else if (fold) STC_PACK(DD, kPackSums);                                                     \
  else STC_PACK(DD, kPackScanned);
  if (s.D == 128) {
    STC_PACK_FORMS(128)
  } else {
    STC_PACK_FORMS(64)
  }
#undef STC_PACK_FORMS
#undef STC_PACK
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_compact(const void* src, const int32_t* token_idx, void* dst, int B, int Hkv, int N_src,
                   int n_keep, int D, int32_t* dev_status, hipStream_t st) {
  const int per_stream = n_keep * (D / 8);
  dim3 grid((per_stream + 255) / 256, B * Hkv);
  if (D == 128)
    compact_kernel<128><<<grid, 256, 0, st>>>((const uint4*)src, token_idx, (uint4*)dst, Hkv, N_src,
                                              n_keep, dev_status);
  else
    compact_kernel<64><<<grid, 256, 0, st>>>((const uint4*)src, token_idx, (uint4*)dst, Hkv, N_src,
                                             n_keep, dev_status);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
