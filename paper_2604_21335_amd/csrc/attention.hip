// Routed decode attention over the selected pages: kernels, launch plan and dispatch around the
// work of one workgroup (attention_block.hpp).
#include "attention_block.hpp"

namespace stc {

// No bound on the registers is needed: the forms of several pairs take 120 to 125 of them at D = 64, two
// workgroups per CU, and 188 at most at D = 128; those of one pair or page 64 at D = 64.
template <int D, int WAVES, bool TAIL, int SELECT_IPT, bool STREAM, bool MULTI, int NX>
__global__ __launch_bounds__(64 * WAVES) void attn_mfma_kernel(
    const void* list_or_score, const uint16_t* q, const uint16_t* K, const uint16_t* mask,
    const uint32_t* tok_off, int NP, int k_pages, int Ncap, int R_by_xcd, const AttnParams rest) {
  AttnParams P = AttnFirst{q, K, mask, tok_off, NP, k_pages, Ncap, R_by_xcd & 0xff}.with(rest);
  P.page_idx = SELECT_IPT > 0 ? nullptr : (const int32_t*)list_or_score;
  extern __shared__ __align__(16) unsigned char lds[];  // WAVES * AttnCfg<D>::WAVE_LDS bytes
  int stream = blockIdx.y, split = blockIdx.x;
  if (R_by_xcd >> 8) {
    // Workgroup i of a launch runs on XCD i % 8: all workgroups of a stream get the same i % 8,
    // so that what they share (the stream's page scores, its query) passes through one L2
    stream = blockIdx.z * kXcds + blockIdx.x;
    split = blockIdx.y;
  }
  attn_block<D, WAVES, TAIL, SELECT_IPT, STREAM, MULTI, NX>(
      P, stream, split, lds, (const float*)list_or_score + (size_t)stream * NP,
      (TopkLds<SELECT_IPT, 64 * WAVES>*)lds);
}

constexpr int kCombineThreads = 256;

// Merge the split partials of a query head by WAVES wavefronts.  Bound by latency: a launch and a round
// trip to memory per BATCH splits, then a chain of dependent instructions.  So the splits are shared out
// among D/4 threads each (4 adjacent channels a thread), whose sums meet at the end, and lane i of every
// wavefront has maximum, sum and weight of split i, which all channels share.  The order of the
// additions is fixed.  With 4 wavefronts 1.1 us for 32 splits from the launch's first instruction to its
// last; with a thread per channel that went through the splits one after the other, an exponential
// each, 2.6, and 1.35 for 16 (4 heads of 471 splits of one long stream: a step of 24.9 us instead of
// 44.8).  Up to 16 splits a wavefront of its own is enough for a head, and many heads then take a
// quarter of the wavefronts.  Attention with the merge, us, thread per channel / 4 wavefronts / one:
//   heads x splits   8 x  9              7.7 /  6.6 /  6.5     D = 64      6.6 /  5.9 /  5.6
//                    8 x 17              7.8 /  6.7 /  7.2                 6.9 /  5.9 /  6.3
//                  448 x  9             17.1 / 15.4 / 15.3                10.7 /  9.6 /  9.5
//                  448 x 17             25.5 / 22.6 / 22.9                16.4 / 14.5 / 14.8
//                 4224 x  4             27.3 / 24.6 / 23.1                16.3 / 15.4 / 15.3
//                 4224 x 17            101.9 / 92.8 / 92.6                54.7 / 49.5 / 48.2
//                32768 x  2             85.8 / 86.4 / 73.6                47.4 / 54.0 / 42.7
template <int D, int WAVES>
__global__ __launch_bounds__(kCombineThreads) void attn_combine_kernel(
    const float* __restrict__ partial, float* __restrict__ out, int splits, int heads) {
  constexpr int ST = partial_stride(D);
  constexpr int ROW = D / 4, GROUPS = 64 * WAVES / ROW;  // splits at a time
  constexpr int BATCH = WAVES == 1 ? 16 : 64;            // splits requested at once
  typedef __attribute__((ext_vector_type(4), aligned(8))) float f32x4_row;
  const int tid = threadIdx.x % (64 * WAVES), lane = tid & 63;
  const int head = blockIdx.x * (kCombineThreads / 64 / WAVES) +
                   __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * WAVES));
  if (head >= heads) return;
  const int group = tid / ROW, c = tid % ROW * 4;
  const float* pr = partial + (size_t)head * splits * ST;
  auto all_lanes = [](float x, auto op) {
    x = op(x, dpp_f32<0x128>(x));  // row_ror:8, 4, 2, 1: over the 16 lanes of a row
    x = op(x, dpp_f32<0x124>(x));
    x = op(x, dpp_f32<0x122>(x));
    x = op(x, dpp_f32<0x121>(x));
    return BATCH > 16 ? across_k_groups(x, op) : x;
  };
  float m = kNegBig, l = 0.f;
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < splits; s0 += BATCH) {
    const int mine = s0 + lane % BATCH;
    const f32x2 ml = *(const f32x2*)(pr + min(mine, splits - 1) * ST);
    f32x4 v[BATCH / GROUPS];
    static_for<0, BATCH / GROUPS>([&](auto j) {
      v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (s0 + j * GROUPS < splits)
        v[j] = *(const f32x4_row*)(pr + min(s0 + j * GROUPS + group, splits - 1) * ST + 2 + c);
    });
    const bool there = mine < splits;
    const float m_new = fmaxf(
        m, all_lanes(there ? ml.x : kNegBig, [](float x, float y) { return fmaxf(x, y); }));
    const float r = __builtin_amdgcn_exp2f(m - m_new);
    const float w = there ? __builtin_amdgcn_exp2f(ml.x - m_new) : 0.f;
    l = fmaf(l, r, all_lanes(w * ml.y, [](float x, float y) { return x + y; }));
    a *= r;
    m = m_new;
    static_for<0, BATCH / GROUPS>([&](auto j) {
      if (s0 + j * GROUPS < splits) {
        const float wj = __shfl(w, j * GROUPS + group);  // 0 past the last split
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = fmaf(wj, v[j][e], a[e]);
      }
    });
  }
  if constexpr (WAVES == 1) {
    // the groups' sums meet in registers; every group then divides and writes a part of the channels
    f32x4 sum;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (GROUPS == 4) {
        sum[e] = across_k_groups(a[e], [](float x, float y) { return x + y; });
      } else {
        const uint32_t u = __float_as_uint(a[e]);
        const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        sum[e] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      }
    }
    float* o = out + (size_t)head * D + c;
    if constexpr (GROUPS == 4) {
      const float own = group & 2 ? (group & 1 ? sum[3] : sum[2]) : (group & 1 ? sum[1] : sum[0]);
      o[group] = l > 0.f ? own / l : 0.f;
    } else {
      const f32x2 own = group ? f32x2{sum[2], sum[3]} : f32x2{sum[0], sum[1]};
      *(f32x2*)(o + 2 * group) = l > 0.f ? f32x2{own.x / l, own.y / l} : f32x2{0.f, 0.f};
    }
  } else {
    __shared__ float s_sum[GROUPS][D];
    *(f32x4*)&s_sum[group][c] = a;
    __syncthreads();
    if (tid < D) {
      float sum = 0.f;
#pragma unroll
      for (int g = 0; g < GROUPS; ++g) sum += s_sum[g][tid];
      out[(size_t)head * D + tid] = l > 0.f ? sum / l : 0.f;
    }
  }
}

// Shape of the launch: wavefronts per workgroup, pairs of pages per wavefront, workgroups per
// stream.
//   Up to 16 pages one workgroup takes them all, one pair per wavefront, and nothing is left to
//   merge by a launch of its own (32 streams of 16 pages: 11.1 us per step; 14.0 with two
//   workgroups of 4 wavefronts and the merge).
//   Where about one workgroup per CU takes a whole stream, its wavefronts take several pairs one
//   after the other, up to 8, and there is nothing to merge either (256 streams, step in us,
//   against one pair per wavefront: 24 pages 21.4 / 23.1, 40: 25.6 / 28.3, 64: 30.9 / 32.9, 128:
//   50.4 / 53.4; with 7 heads per KV head 96 pages 56.2 / 74.0; 192 streams, 64 pages 29.6 / 31.3;
//   D = 64, 512 streams, 64 pages 30.4 / 34.6).  The several-pairs kernel fills the registers
//   of a CU with one workgroup at D = 128, two at D = 64, so more streams than that run in
//   rounds (320 streams of 48 pages: 41.3 / 34.4), and with fewer the chip is not full (128
//   streams of 48 pages: 23.4 / 23.1).
//   Lists of the query heads of one KV head share pages, which come from the caches after the first
//   head: such launches are bound by latency more than by bandwidth and gain from several pairs
//   only up to 3 (224 streams of 7 heads, us, against one pair per wavefront: 40 pages 14.3 / 15.8,
//   64: 18.7 / 19.0, 128: 32.3 / 28.1; 256 streams of 4 heads, 24 pages 9.8 / 11.5, 64: 21.8 / 20.6,
//   128: 35.3 / 31.7; of 16 heads, 32 pages 12.2 / 12.8, 64: 20.3 / 18.4).
//   Otherwise 8 wavefronts with a pair each, which beats 4 with a pair each also where that
//   leaves CUs idle (8 streams of 90 pages: 13.5 / 14.7), or with a page each.  A page is half the
//   chain of dependent instructions of a pair and half the traffic through a CU, for twice as many
//   partial results and selections: faster while every CU has at most one of these workgroups, or
//   where some CUs would have two with pairs and still no more than two with single pages (those
//   that select; the others come when there is room).  Step in us, pages / pairs:
//     workgroups with pages, pairs                               D = 128          D = 64
//     192, 112   16 streams of 90 of 1000 pages                12.6 / 13.6      10.9 / 11.4
//     256, 128   32 streams of 64 of 500                       12.9 / 13.9
//     128,  64   28 layers of 4 streams of 256 of 8192          466 / 486
//     320, 160   20 streams of 128 of 2048                     17.2 / 16.7
//     384, 192   32 streams of 90 of 1000                      15.8 / 15.4      13.2 / 13.1
//     512, 256   64 streams of 64 of 500                       16.7 / 16.4
//     390, 260   130 streams of 24 of 500                      18.3 / 20.2      13.9 / 14.9
//     484, 264   44 streams of 88 of 1000                      17.6 / 18.9
//     520, 280   40 streams of 90 of 751 and 7 of a tail       16.7 / 17.9      13.0 / 14.4
//     516, 258   43 streams of 90 of 1000                      19.9 / 18.3
//     533, 287   41 streams of 104 of 1000                     21.0 / 19.3      16.2 / 15.2
struct AttnPlan {
  int waves, nx, pairs, splits;  // nx: pages that a wavefront takes at a time
  int slots() const { return waves * nx * pairs; }  // page slots per workgroup
};

// Keys per thread of the selection inside the launch of a plan, for streams of NP pages; 0 if no form of
// it holds that many (64 * waves * keys).  Several pairs go with 4 only: 192 to 255 streams of more than
// 2048 pages with 17 to 32 page slots leave the selection to a launch of its own.
static int select_keys(const AttnPlan& p, int NP) {
  if (p.waves != 8) return NP <= 64 * 4 * 8 ? 8 : 0;
  if (NP <= 64 * 8 * 4) return 4;
  return p.pairs == 1 && NP <= 64 * 8 * 16 ? 16 : 0;
}

// Streams of 2049..8192 pages can select inside the attention kernel, 16 keys per thread, while its
// workgroups are fewer than two per compute unit.  Step in us, inside / as a launch of its own: 12
// streams of 256 of 8192 pages 22.4 / 23.4, 24 of them 34.9 / 37.9; 16 of 300 of 4096 22.1 / 22.6; 48 of
// 100 of 3000 28.6 / 29.9.
// The line is not where the two meet: at 512 workgroups, which stay three launches as they always were
// (the tests of the step ask for that form there), inside would be faster still: 64 streams of 128 of 2049
// pages 30.2 / 30.5 (D = 64: 19.8 / 20.4), of 4096 38.6 / 40.0; 32 of 256 of 8192 41.4 / 42.1 (D = 64:
// 25.9 / 27.9).
static bool long_select_shape(const stc_shape_t& s, int k_pages) {
  const int NP = (s.N + kPage - 1) / kPage;
  return NP > 2048 && NP <= 8192 && k_pages > 8 &&
         (long long)s.B * s.Hkv * ((k_pages + 15) / 16) < 512;
}

// Workgroups that take a whole stream each and are resident at once: the registers of a CU hold one at
// D = 128, two at D = 64, with and without a tail.  Step in us at D = 64, a workgroup per stream / splits
// and a merge (tail: its pages):
//   512 streams of  64 of  250 pages  27.3 / 30.5   and a tail of 2  30.2 / 31.4
//   512         of  64 of  512        33.4 / 36.0
//   512         of  64 of 1100                      and a tail of 2  48.8 / 51.8
//   512         of 100 of  512                      and a tail of 4  46.4 / 46.1
//   384         of  40 of  500                      and a tail of 2  21.6 / 24.5
//   300         of  48 of  400                      and a tail of 2  24.0 / 24.4
//   260         of  64 of  300        24.0 / 24.2   and a tail of 2  26.5 / 24.6
// (Just above 256 streams few CUs have a second one.)
static int resident_streams(const stc_shape_t& s) { return s.D == 128 ? 256 : 512; }

// K rows and value runs are read once per step.  What a launch cannot know is whether they still lie
// in the last-level cache (256 MB): behind the other layers of a decoder they do not, where one
// cache is stepped by itself they do.  us per step with ordinary / streaming loads of them:
//   keys + bounds, MiB             out of the cache     in it
//    8 + 15   40 streams of  751    18.5 / 18.5        14.8 / 15.0
//   20 + 16  128 of  250            22.5 / 22.0        19.8 / 19.0
//   16 + 32   32 of 2048            22.9 / 22.5        20.8 / 21.0
//   38 + 31  160 of  400            30.8 / 30.2        25.9 / 26.8
//   64 + 32  256 of  256            32.4 / 29.4        26.8 / 28.6
//   32 + 64   64 of 2048            32.8 / 31.9        30.7 / 30.1
//   75 + 47  320 of  300            44.4 / 42.7        37.2 / 39.8
//   64 + 64  256 of  512            37.8 / 34.2        32.0 / 32.7
// Below 80 MiB the two differ by 2 % out of the cache and by 4 % either way in it; above, streaming
// loads gain 3 to 10 % out of the cache, for which a step of one cache by itself pays up to 7 %.
// Pages that several query heads of a KV head select (kv_div > 1) count once: they come from the
// caches after the first.
static bool streaming_loads(const stc_shape_t& s, int k_pages, int tail_pages, int kv_div) {
  const int NP = (s.N + kPage - 1) / kPage;
  const long long streams = (long long)s.B * s.Hkv / kv_div;
  const long long keys = streams * (k_pages + tail_pages) * kPage * s.D * 2;
  const long long bounds = k_pages < NP ? streams * NP * s.D * 4 : 0;
  return keys + bounds >= (80ll << 20);
}

// kv_div query heads per KV head with page lists of their own (each of them a stream here).
static AttnPlan attention_plan(const stc_shape_t& s, int k_pages, int tail_pages, int kv_div = 1) {
  const int streams = s.B * s.Hkv, slots = k_pages + tail_pages;
  AttnPlan p{slots <= 8 ? 4 : 8, 2, 1, 0};
  const int max_pairs = kv_div > 1 ? kMaxPairsShared : kMaxPairs;
  auto workgroups = [&](int pages, int each) { return (long long)streams * ((pages + each - 1) / each); };
  if (slots > 16 && slots <= 16 * max_pairs && streams >= 192 && streams <= resident_streams(s))
    p.pairs = (slots + 15) / 16;
  else if (slots > 16 && !streaming_loads(s, k_pages, tail_pages, kv_div) &&
           (workgroups(slots, 8) <= 256 ||
            (workgroups(slots, 16) > 256 && workgroups(k_pages, 8) <= 512 &&
             workgroups(slots, 8) <= 768)))
    p.nx = 1;
  p.splits = (slots + p.slots() - 1) / p.slots();
  return p;
}

int attention_splits(const stc_shape_t& s, int k_pages, int tail_pages, int kv_div) {
  return attention_plan(s, k_pages, tail_pages, kv_div).splits;
}
int attention_wave_pages(const stc_shape_t& s, int k_pages, int tail_pages, int kv_div) {
  const AttnPlan p = attention_plan(s, k_pages, tail_pages, kv_div);
  return p.nx * p.pairs;
}

// The per-query-head form is the ordinary launch on a shape with one KV head per query head
// (the kernel then maps kv_div of those onto one cache).
static stc_shape_t launch_shape(const stc_shape_t& s, bool per_head) {
  stc_shape_t t = s;
  if (per_head) t.Hkv = s.Hq;
  return t;
}

// Room for the split partials of any launch over at most k_pages page slots: the plan with
// the most workgroups per stream (4 wavefronts of 2 pages each), so that the size never
// shrinks when k_pages grows and a buffer sized for the largest count serves every smaller one.
size_t attention_ws_bytes(const stc_shape_t& s0, int k_pages, bool per_head) {
  const stc_shape_t s = launch_shape(s0, per_head);
  const int splits = (k_pages + 7) / 8;
  if (splits <= 1) return 0;
  return (size_t)s.B * s.Hq * splits * partial_stride(s.D) * sizeof(float);
}

namespace {

struct AttnLaunch {
  AttnParams p;
  dim3 grid;
  hipStream_t st;
};

template <int D, int WAVES, bool TAIL, int SELECT_IPT, bool STREAM, bool MULTI, int NX>
int attn_go(const AttnLaunch& a) {
  // workgroups of 8 wavefronts at D = 128 need more than the default 64 KiB of LDS
  // (the selection uses the same memory)
  constexpr int attn_lds = WAVES * AttnCfg<D>::WAVE_LDS;
  constexpr int topk_lds = SELECT_IPT > 0 ? (int)sizeof(TopkLds<SELECT_IPT, 64 * WAVES>) : 0;
  constexpr int lds_bytes = attn_lds > topk_lds ? attn_lds : topk_lds;
  static std::atomic<uint64_t> allowed{0};
  if (!allow_dynamic_lds((const void*)attn_mfma_kernel<D, WAVES, TAIL, SELECT_IPT, STREAM, MULTI, NX>,
                         lds_bytes, allowed))
    return -1;
  attn_mfma_kernel<D, WAVES, TAIL, SELECT_IPT, STREAM, MULTI, NX>
      <<<a.grid, 64 * WAVES, lds_bytes, a.st>>>(
          SELECT_IPT > 0 ? (const void*)a.p.sel_score : (const void*)a.p.page_idx, a.p.q, a.p.K,
          a.p.mask, a.p.tok_off, a.p.NP, a.p.k_pages, a.p.Ncap, a.p.R | (int)a.p.by_xcd << 8, a.p);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int D, int WAVES, int SELECT_IPT, bool STREAM, bool MULTI = false, int NX = 2>
int attn_tail(const AttnLaunch& a, bool tail) {
  return tail ? attn_go<D, WAVES, true, SELECT_IPT, STREAM, MULTI, NX>(a)
              : attn_go<D, WAVES, false, SELECT_IPT, STREAM, MULTI, NX>(a);
}

template <int D>
int attn_dispatch(const AttnLaunch& a, const AttnPlan& plan, bool tail, int keys,
                  bool stream_loads) {
  if (plan.waves != 8)  // few pages: nothing to keep out of the caches
    return keys ? attn_tail<D, 4, 8, false>(a, tail) : attn_tail<D, 4, 0, false>(a, tail);
  if (plan.nx == 1) {  // few workgroups, ordinary loads
    if (keys == 16) return attn_tail<D, 8, 16, false, false, 1>(a, tail);
    return keys ? attn_tail<D, 8, 4, false, false, 1>(a, tail)
                : attn_tail<D, 8, 0, false, false, 1>(a, tail);
  }
  if (plan.pairs > 1) {
    if (keys)
      return stream_loads ? attn_tail<D, 8, 4, true, true>(a, tail)
                          : attn_tail<D, 8, 4, false, true>(a, tail);
    return stream_loads ? attn_tail<D, 8, 0, true, true>(a, tail)
                        : attn_tail<D, 8, 0, false, true>(a, tail);
  }
  // (streaming loads lose with 16 keys: 24 streams of 256 of 8192 pages 36.6 us per step, 34.9)
  if (keys == 16) return attn_tail<D, 8, 16, false>(a, tail);
  if (keys) return stream_loads ? attn_tail<D, 8, 4, true>(a, tail) : attn_tail<D, 8, 4, false>(a, tail);
  return stream_loads ? attn_tail<D, 8, 0, true>(a, tail) : attn_tail<D, 8, 0, false>(a, tail);
}

}  // namespace

// Selection inside the attention kernel repeats a stream's top-k in each of its workgroups.
// Measured against the separate selection launch it is faster while all workgroups are
// resident at once (two per compute unit) and a stream's keys fit four per thread, and
// slower beyond (the repeated prologue then delays a second round of workgroups).
bool attention_can_select(const stc_shape_t& s, int k_pages, int tail_pages) {
  const int NP = (s.N + kPage - 1) / kPage;
  const AttnPlan p = attention_plan(s, k_pages, tail_pages);
  if (k_pages >= NP || select_keys(p, NP) == 0) return false;
  if (NP > 2048) return long_select_shape(s, k_pages + tail_pages);
  // the workgroups that select must all be resident at once; those that hold only pages of
  // the tail skip the selection and may come in a second round
  const long long streams = (long long)s.B * s.Hkv;
  return streams * ((k_pages + p.slots() - 1) / p.slots()) <= 512 && streams * p.splits <= 768;
}

int attention_select_pages(const stc_shape_t& s, int k_pages, int tail_pages) {
  const AttnPlan p = attention_plan(s, k_pages, tail_pages);
  return 64 * p.waves * select_keys(p, (s.N + kPage - 1) / kPage);
}

// Parameters of an attention launch without a page list's consumers filled in.
static AttnParams attn_params(const stc_shape_t& s, const stc_shape_t& s0, const AttnPlan& plan,
                              const void* q, const void* K, const void* vpacked,
                              const uint16_t* mask, const uint32_t* tok_off,
                              const int32_t* page_idx, int k_pages, const void* K_tail,
                              const void* V_tail, int n_tail, int tail_cap,
                              const uint16_t* page_heads, const float* sel_score,
                              int32_t* sel_list, float* out, void* ws) {
  if (n_tail == 0) K_tail = V_tail = K;  // any valid address: never read
  return AttnParams{(const uint16_t*)q, (const uint16_t*)K, (const unsigned char*)vpacked, mask,
                    tok_off, page_idx, (float*)ws, out, s.Hq / s.Hkv, s.N,
                    (s.N + kPage - 1) / kPage, s.G, (uint32_t)s.v_cap_groups, k_pages, plan.splits,
                    (const uint16_t*)K_tail, (const uint16_t*)V_tail, n_tail, tail_cap,
                    s.Hkv / s0.Hkv, page_heads, token_cap(s), sel_score, sel_list, plan.pairs, false};
}

int launch_attention(const stc_shape_t& s0, const void* q, const void* K, const void* vpacked,
                     const uint16_t* mask, const uint32_t* tok_off, const int32_t* page_idx,
                     int k_pages, const void* K_tail, const void* V_tail, int n_tail, int tail_cap,
                     bool per_head, const uint16_t* page_heads, const float* sel_score,
                     int32_t* sel_list, float* out, void* ws, hipStream_t st) {
  const stc_shape_t s = launch_shape(s0, per_head);
  const int NP = (s.N + kPage - 1) / kPage;
  const int streams = s.B * s.Hkv;
  const int tail_pages = (n_tail + kPage - 1) / kPage;
  const int kv_div = s.Hkv / s0.Hkv;
  const AttnPlan plan = attention_plan(s, k_pages, tail_pages, kv_div);
  AttnLaunch a{attn_params(s, s0, plan, q, K, vpacked, mask, tok_off, page_idx, k_pages, K_tail,
                           V_tail, n_tail, tail_cap, page_heads, sel_score, sel_list, out, ws),
               dim3(plan.splits, streams), st};
  const int keys = sel_score ? select_keys(plan, NP) : 0;
  if (sel_score && (keys == 0 || per_head || page_heads)) return -1;
  // with the selection inside, the workgroups of a stream all read the stream's scores: keep
  // them on one XCD (measured on the headline shape: 34.2 against 34.6 us per step)
  if (sel_score && plan.splits > 1 && streams % kXcds == 0) {
    a.p.by_xcd = true;
    a.grid = dim3(kXcds, plan.splits, streams / kXcds);
  }
  const bool stream_loads = streaming_loads(s, k_pages, tail_pages, kv_div);
  const bool tail = tail_pages > 0;
  const int rc = s.D == 128 ? attn_dispatch<128>(a, plan, tail, keys, stream_loads)
                            : attn_dispatch<64>(a, plan, tail, keys, stream_loads);
  if (rc) return -1;
  if (plan.splits > 1) {
    const int heads = s.B * s.Hq;
    const bool few = plan.splits <= 16;  // one round of requests of a wavefront (table at the kernel)
#define STC_COMBINE(DD, WAVES)                                                                  \
  attn_combine_kernel<DD, WAVES><<<(heads * WAVES + 3) / 4, kCombineThreads, 0, st>>>(          \
      a.p.partial, out, plan.splits, heads)
    if (s.D == 128) {
      if (few) STC_COMBINE(128, 1);
      else STC_COMBINE(128, 4);
    } else {
      if (few) STC_COMBINE(64, 1);
      else STC_COMBINE(64, 4);
    }
#undef STC_COMBINE
    if (hipGetLastError() != hipSuccess) return -1;
  }
  return 0;
}

// One workgroup per stream does the whole step where the attention has no splits anyway, all
// workgroups are resident at once, and scoring a stream in one workgroup costs no more than the
// launches it saves: streams of few pages (more than 4 heads per KV head take twice as long per
// page), or enough streams that the chip is full either way.  Step in us, one launch / several:
// 8 streams of 64 pages 8.0 / 9.5; 32 of 125 pages, 16 kept 10.1 / 11.1; 256 of 256 pages, 64 kept
// 29.4 / 30.9; D = 64, 256 of 256 pages, 32 kept 13.6 / 16.2; 256 of 1024 pages with 7 heads, 96
// kept 54.2 / 54 is where the two meet.  Not: 8 streams of 500 pages 12.6 / 11.0; 64 of 250 pages with 7 heads 13.7 /
// 13.3; 512 of 250 pages at D = 128 (two rounds) 31.8 / 27.3.
bool step_is_one_kernel(const stc_shape_t& s, int k_pages, int tail_pages) {
  const int NP = (s.N + kPage - 1) / kPage, streams = s.B * s.Hkv, R = s.Hq / s.Hkv;
  if (k_pages >= NP || R > 8 || streams > resident_streams(s)) return false;
  if (!(NP <= (R <= 4 ? 256 : 192) || (streams >= 192 && NP <= kStepKeys))) return false;
  return attention_plan(s, k_pages, tail_pages).splits == 1;
}

int launch_step(const stc_shape_t& s, const void* q, const void* bounds, const void* K,
                const void* vpacked, const uint16_t* mask, const uint32_t* tok_off, int k_pages,
                const void* K_tail, const void* V_tail, int n_tail, int tail_cap, float* score,
                int32_t* list, float* out, hipStream_t st) {
  const int tail_pages = (n_tail + kPage - 1) / kPage;
  const AttnPlan plan = attention_plan(s, k_pages, tail_pages);
  const AttnParams p =
      attn_params(s, s, plan, q, K, vpacked, mask, tok_off, nullptr, k_pages, K_tail, V_tail, n_tail,
                  tail_cap, nullptr, nullptr, list, out, nullptr);
  return launch_step_kernel(p, s.D, s.B * s.Hkv, bounds, score, tail_pages > 0,
                            streaming_loads(s, k_pages, tail_pages, 1), st);
}

// New token of every stream -> row n_tail of the stream's uncompressed tail (K and V).
template <int D>
__global__ __launch_bounds__(256) void append_tail_kernel(const uint4* __restrict__ k_new,
                                                          const uint4* __restrict__ v_new,
                                                          uint4* __restrict__ K_tail,
                                                          uint4* __restrict__ V_tail, int streams,
                                                          int n_tail, int tail_cap) {
  constexpr int LPR = D / 8;  // 16-byte pieces per row
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= streams * LPR) return;
  const int stream = i / LPR, piece = i % LPR;
  const size_t dst = ((size_t)stream * tail_cap + n_tail) * LPR + piece;
  K_tail[dst] = k_new[i];
  V_tail[dst] = v_new[i];
}

int launch_append_tail(const stc_shape_t& s, const void* k_new, const void* v_new, void* K_tail,
                       void* V_tail, int n_tail, int tail_cap, hipStream_t st) {
  const int streams = s.B * s.Hkv;
  const int n = streams * (s.D / 8);
  if (s.D == 128)
    append_tail_kernel<128><<<(n + 255) / 256, 256, 0, st>>>(
        (const uint4*)k_new, (const uint4*)v_new, (uint4*)K_tail, (uint4*)V_tail, streams, n_tail,
        tail_cap);
  else
    append_tail_kernel<64><<<(n + 255) / 256, 256, 0, st>>>(
        (const uint4*)k_new, (const uint4*)v_new, (uint4*)K_tail, (uint4*)V_tail, streams, n_tail,
        tail_cap);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
