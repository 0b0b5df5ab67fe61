// The work of one workgroup of routed decode attention: shared by the attention kernel
// (attention.hip) and by the kernel that runs a whole decode step per workgroup (step.hip).
//
// Routed decode attention over the selected pages (paper Sec. 3.3: softmax over
// full-width keys, values read from the group-packed store, dropped groups
// contribute nothing, no renormalisation).  Split over pages with online-softmax
// partials, merged inside the workgroup and then by a fixed-order combine.
//
// The R <= 16 query heads of a KV head share every K page and every packed V
// run, so both contractions are 16-wide dense tiles and run on the matrix cores
// (v_mfma_f32_16x16x32_bf16, float accumulation):
//   S^T[token][head] = K_page[token][:] . q[head][:]        (contract channels)
//   O^T[chan][head] += V~^T[chan][token] . P^T[token][head] (contract tokens)
// S^T leaves the first MFMA with tokens along the registers of a lane, which is
// the operand layout the second MFMA wants for P^T, so the weights never leave
// registers.  Each weight is split into two bf16 parts (p = hi + lo) so the
// product with V carries ~2^-17 relative error instead of bf16's 2^-9.
// Both K and the routed (zero-filled) V of a page pass through a dense LDS tile.
#pragma once
#include "stc_common.hpp"
#include "stc_kernels.hpp"
#include "topk_block.hpp"

namespace stc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
// 16-byte register values are native vectors: copies of the HIP uint4 struct go through
// memcpy, which can leave a register array in scratch memory
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;  // "no token seen yet" running maximum
constexpr int kMaxPairs = 8;         // pairs of pages per wavefront at most
constexpr int kMaxPairsShared = 3;   // the same where heads of a KV head have lists of their own
constexpr int kXcds = 8;
constexpr int kTailPage = 1 << 30;   // flag of a page slot that lies in the uncompressed tail

// Partial result of one (query head, split): [0] running max (base-2 logits),
// [1] sum of weights, [2 .. 2+D) weighted value sum.
__host__ __device__ constexpr int partial_stride(int D) { return D + 2; }

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // round to nearest even
}

template <int D>
struct AttnCfg {
  static constexpr int KC = D / 32;         // QK MFMAs per page (32 channels each)
  static constexpr int CB = D / 16;         // output channels per lane and token (see PV below)
  static constexpr int LPR = D / 8;         // 16-byte pieces (lanes of a flat load) per token row
  static constexpr int NLD = kPage * D * 2 / 1024;  // flat 1 KiB loads per page of K (or of a full V run)
  static constexpr int ROW = D * 2 + 16;    // LDS bytes per token row of the K tile (padded)
  static constexpr int TILE = kPage * ROW;  // K tile of a page; reused for the page's packed V run
  static constexpr int META = 2 * TILE;     // per pair: 2 x 16 words (mask | relative offset << 16)
  static constexpr int ZERO = META + 128;   // 16 zero bytes: what dropped units read
  static constexpr int WAVE_LDS = ZERO + 16;
  // merge buffer of a wavefront: 16 head rows of D floats, each row padded by 4 floats so that
  // the 16 heads' 16-byte writes of one channel group fall into different banks
  static constexpr int MROW = D + 4;
  static constexpr int MML = 16 * MROW * 4;  // byte offset of the 16 (m, l) pairs behind it
  static_assert(MML + 16 * 2 * 4 <= 2 * TILE, "merge buffer fits the tiles");
};

// Lanes that differ in lane bit 4 or 5 hold parts of the same sum or maximum: every lane gets op over
// the four of them.  (Swaps of register halves; a shuffle would go through shared memory.)
template <class Op>
__device__ __forceinline__ float across_k_groups(float x, Op op) {
  const uint32_t a = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const uint32_t b = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto s = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

// One wavefront takes one pair of page slots of one stream (NX = 2), one page slot (NX = 1), or, with
// MULTI, P.pairs adjacent pairs one after the other (up to kMaxPairs), each a partial result of its
// own; the WAVES wavefronts of a workgroup then merge their partial results in LDS.
// Page slots are the selected pages of the compressed cache followed, with TAIL, by the pages
// of the uncompressed tail; kv_div query-head streams may share one KV head's cache.
//
// Per pair of pages:
//   1. K pages and packed V runs are read flat (every request is 1 KiB of adjacent
//      addresses, 16 bytes per lane) and staged in LDS.  Loading straight into the
//      MFMA operand layout, or unit by unit for V, turns each request into scattered
//      32..64-byte pieces and costs about 30 % of the achievable bandwidth.
//   2. QK: lane (token r16, k-group kg) reads 16 bytes per 32-channel step from the
//      K tile; S^T = K.q^T; online softmax per head; weights split into hi+lo bf16.
//   3. PV: lane (r16, kg) owns the CB adjacent channels r16*CB.. (one 16-byte value
//      unit for D = 128).  For each of its 8 tokens it computes where that unit sits
//      in the staged run (slot = offset of the token + rank of the group among the
//      kept ones) or takes zeros if the group was dropped, reads it, transposes the
//      8x8 block in registers with byte permutes and feeds MFMA row m of block cb
//      <-> channel m*CB + cb.  The accumulators of a lane cover channels 32*kg...
// Request order: page indices; masks/offsets and the K rows of the pair; then, as soon as
// the offsets are there, the pair's V runs.  All loads are unconditional (addresses of absent pages or
// tokens collapse to one valid location and the result is discarded) so that they
// stay in flight across the arithmetic.
// SELECT_IPT > 0: no page list is given; every workgroup first selects the stream's k pages
// from the page scores itself (the same selection as the stand-alone kernel, SELECT_IPT keys
// per thread), keeps the ones of its own split and writes them to the list.  Tail pages keep
// their slots behind the k selected ones.
// Arguments of the attention kernels (one struct, passed by value).
struct AttnParams {
  const uint16_t *q, *K;
  const unsigned char* vpacked;
  const uint16_t* mask;
  const uint32_t* tok_off;
  const int32_t* page_idx;
  float *partial, *out;
  int R, N, NP, G;  // R: query heads per stream (KV head)
  uint32_t cap;
  int k_pages, splits;
  const uint16_t *K_tail, *V_tail;
  int n_tail, tail_cap, kv_div;
  const uint16_t* page_heads;
  int Ncap;
  const float* sel_score;
  int32_t* sel_list;
  int pairs;    // pairs of pages per wavefront (MULTI kernels)
  bool by_xcd;  // grid (kXcds, splits, streams / kXcds): a stream's workgroups on one XCD
};

// The arguments that a workgroup needs first come in front of the struct, one by one: the first 14
// words of a kernel's scalar arguments are in registers when it starts (a struct is not), the
// others are a load from memory away.
struct AttnFirst {
  const uint16_t *q, *K, *mask;
  const uint32_t* tok_off;
  int NP, k_pages, Ncap, R;

  __device__ __forceinline__ AttnParams with(AttnParams p) const {
    p.q = q, p.K = K, p.mask = mask, p.tok_off = tok_off;
    p.NP = NP, p.k_pages = k_pages, p.Ncap = Ncap, p.R = R;
    return p;
  }
};

// Keys that the selection inside a step kernel holds (pages per stream at most), and the bounds
// tiles that a wavefront of it has in flight.
constexpr int kStepKeys = 1024;
constexpr int kStepTilesAhead = 2;

// One launch for a whole step (step.hip): one workgroup of 8 wavefronts per stream, no splits.
int launch_step_kernel(const AttnParams& p, int D, int streams, const void* bounds, float* score,
                       bool tail, bool stream_loads, hipStream_t st);

// The work of one workgroup: split `split` of stream `stream`.  `lds` = WAVES * WAVE_LDS bytes
// of shared memory.  sel_score (SELECT_IPT > 0) = the stream's page scores; they and the memory
// of the selection, sel_lds, may lie in `lds`, which is written only after the selection.
template <int D, int WAVES, bool TAIL, int SELECT_IPT, bool STREAM, bool MULTI, int NX>
__device__ __forceinline__ void attn_block(const AttnParams& P, const int stream, const int split,
                                           unsigned char* lds, const float* sel_score,
                                           TopkLds<SELECT_IPT, 64 * WAVES>* sel_lds) {
  using C = AttnCfg<D>;
  static_assert(NX == 2 || !MULTI, "several pairs, or one page, per wavefront");
  const int ppw = MULTI ? 2 * P.pairs : NX;  // pages per wavefront
  const uint16_t* __restrict__ q = P.q;
  const uint16_t* __restrict__ K = P.K;
  const unsigned char* __restrict__ vpacked = P.vpacked;
  const uint16_t* __restrict__ mask = P.mask;
  const uint32_t* __restrict__ tok_off = P.tok_off;
  const int32_t* __restrict__ page_idx = P.page_idx;
  float* __restrict__ partial = P.partial;
  float* __restrict__ out = P.out;
  const int R = P.R, N = P.N, NP = P.NP, G = P.G;
  const uint32_t cap = P.cap;
  const int k_pages = P.k_pages, splits = P.splits;
  const uint16_t* __restrict__ K_tail = P.K_tail;
  const uint16_t* __restrict__ V_tail = P.V_tail;
  const int n_tail = P.n_tail, tail_cap = P.tail_cap, kv_div = P.kv_div;
  const uint16_t* __restrict__ page_heads = P.page_heads;
  const int Ncap = P.Ncap;
  int32_t* __restrict__ sel_list = P.sel_list;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kg = lane >> 4;  // MFMA row/column and k-group of this lane
  const int lg_g = 31 - __clz(G);                 // G is a power of two
  const uint32_t gbytes = (D * 2) >> lg_g;
  const int lg_upg = 31 - __clz(D / 8) - lg_g;  // log2(16-byte units per group)
  const float scale = kLog2e / sqrtf((float)D);

  unsigned char* wl = lds + wave * C::WAVE_LDS;

  // per-stream bases (wave-uniform); everything below is addressed with 32-bit byte offsets.
  // kv_div > 1: the launch has one "stream" (page list, query, output) per query head and
  // kv_div of them share the cache of one KV head.
  const int kvs = kv_div == 1 ? stream : stream / kv_div;
  const unsigned char* Ks = (const unsigned char*)K + (size_t)kvs * Ncap * D * 2;
  const unsigned char* mask_s = (const unsigned char*)mask + (size_t)kvs * Ncap * 2;
  const unsigned char* off_s = (const unsigned char*)tok_off + (size_t)kvs * (Ncap + 1) * 4;
  const unsigned char* vs = vpacked + (size_t)kvs * (size_t)cap * gbytes;
  // the uncompressed tail: dense K and V rows, i.e. a packed store in which every token kept
  // every group; its pages follow the selected ones in the list of page slots
  const unsigned char* Kts = (const unsigned char*)K_tail + (size_t)kvs * tail_cap * D * 2;
  const unsigned char* vts = (const unsigned char*)V_tail + (size_t)kvs * tail_cap * D * 2;
  const int tail_pages = TAIL ? (n_tail + kPage - 1) / kPage : 0;
  const uint32_t full_mask = (1u << G) - 1u;

  // this wavefront's pages: lane i holds page slot pi0 + i (-1: none; kTailPage | p: tail page)
  const int pi0 = (split * WAVES + wave) * ppw;
  const int npages = max(0, min(ppw, k_pages + tail_pages - pi0));
  int my_pg = -1;
  int my_heads = 0xffff;  // heads of the group that attend the page (all, unless a list is given)
  if (lane < npages) {
    const int slot = pi0 + lane;
    if (slot < k_pages) {
      my_pg = page_idx ? page_idx[(size_t)stream * k_pages + slot] : slot;  // no list: pages 0..
      // every page attended and the caller wants the list: each wavefront writes its own part
      if (SELECT_IPT == 0 && !page_idx && sel_list)
        sel_list[(size_t)stream * k_pages + slot] = slot;
      if (page_heads) my_heads = page_heads[(size_t)stream * k_pages + slot];
      if (my_pg < 0 || my_pg >= NP) my_pg = -1;
    } else {
      my_pg = kTailPage | (slot - k_pages);
    }
  }
  // (a workgroup whose page slots all lie in the uncompressed tail needs no list)
  const int lo = split * WAVES * ppw;  // first list position of this workgroup
  __shared__ int32_t s_pages[SELECT_IPT > 0 ? WAVES * 2 * (MULTI ? kMaxPairs : 1) : 1];
  if constexpr (SELECT_IPT > 0) if (lo < k_pages) {
    if ((int)threadIdx.x < WAVES * ppw) s_pages[threadIdx.x] = -1;
    __syncthreads();
    topk_block<SELECT_IPT, 64 * WAVES>(sel_score, NP, k_pages, *sel_lds, [&](int pos, int page) {
      const unsigned r = (unsigned)(pos - lo);
      if (r < (unsigned)(WAVES * ppw)) {
        s_pages[r] = page;
        if (MULTI) sel_list[(size_t)stream * k_pages + pos] = page;
      }
    });
    __syncthreads();
    if (lane < npages && pi0 + lane < k_pages) my_pg = s_pages[wave * ppw + lane];
  }
  if (lane < 4) *(uint32_t*)(wl + C::ZERO + lane * 4) = 0;
  const int npairs = (npages + NX - 1) / NX;

  // PV role: the value unit this lane reads for each of its tokens
  const uint32_t unit = (D == 128) ? r16 : (r16 >> 1);
  const uint32_t u_g = unit >> lg_upg;                    // its group
  const uint32_t u_below = (1u << u_g) - 1u;              // groups stored before it
  const uint32_t u_within = (unit - (u_g << lg_upg)) * 16 + ((D == 128) ? 0 : (r16 & 1) * 8);

  // Masks and offsets of a pair: lanes 0..15 carry the tokens of its first page, 16..31 of its
  // second page.
  struct PairMeta {
    uint32_t mk, off, run0[NX], run1[NX];
    uint32_t moi;  // token index behind off (tail pages derive their offsets from it)
    bool mvalid;
    bool mtail;    // this lane's meta words belong to a tail page
    int pgs[NX];
  };
  u32x4 kreg[NX][C::NLD];

  // Lanes 0..15 fetch mask and offset of the tokens of the pair's first page, lanes
  // 16..31 of its second page; lanes 32 and 33 fetch the offset just past each page
  // (the end of its packed run).  Vector loads on purpose: scalar loads of these
  // scattered words queue up in the scalar cache for several microseconds.
  // Page slot -> page number, token limit of its store, and whether it is a tail page.
  auto is_tail = [&](int pg) { return TAIL && pg >= kTailPage; };  // never, if no tail is given
  auto page_no = [&](int pg) { return pg & (kTailPage - 1); };
  auto tok_lim = [&](int pg) { return (uint32_t)(is_tail(pg) ? n_tail : N); };
  auto issue_meta = [&](PairMeta& M, int pair) {
#pragma unroll
    for (int x = 0; x < NX; ++x) M.pgs[x] = __builtin_amdgcn_readlane(my_pg, NX * pair + x);
    const int pg = (lane & 1) ? M.pgs[NX - 1] : M.pgs[0];     // lanes 32, 33
    const int pgt = (lane & 16) ? M.pgs[NX - 1] : M.pgs[0];   // token lanes
    const uint32_t t = (pgt < 0 ? 0 : page_no(pgt) * kPage) + r16;
    const bool tv = lane < 16 * NX && pgt >= 0 && t < tok_lim(pgt);
    const uint32_t tend =
        pg < 0 ? 0u : min((uint32_t)page_no(pg) * kPage + kPage, tok_lim(pg));
    const uint32_t oi = tv ? t : ((lane == 32 || lane == 33) ? tend : 0u);
    const bool tl = lane < 32 ? (pgt >= 0 && is_tail(pgt)) : (pg >= 0 && is_tail(pg));
    M.mvalid = tv;
    M.moi = oi;
    M.mtail = tl;
    // tail lanes read word 0 of the stream's arrays and replace the result later
    M.mk = *(const uint16_t*)(mask_s + ((tv && !tl) ? t : 0u) * 2);  // discarded if !tv
    M.off = *(const uint32_t*)(off_s + (tl ? 0u : oi) * 4);
  };
  // start and end of the packed runs of a pair (wave-uniform), once the offsets are there.
  // A tail token keeps every group and its G groups sit at token index * G.
  auto finish_meta = [&](PairMeta& M) {
    if (M.mtail) {
      M.mk = full_mask;
      M.off = M.moi * G;
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      M.run0[x] = __builtin_amdgcn_readlane(M.off, 16 * x);  // token 0 of a page is valid
      M.run1[x] = __builtin_amdgcn_readlane(M.off, 32 + x);
    }
  };
  auto issue_k = [&](const PairMeta& M) {
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const int pg = M.pgs[x];
      const uint32_t t0 = pg < 0 ? 0 : page_no(pg) * kPage;
      // absent tokens read the end of the store's last row, those of an absent page the store's first
      // bytes: their logits are discarded
      const uint32_t last = pg < 0 ? 0u : tok_lim(pg) * (D * 2) - 16;
      const unsigned char* kb = (pg >= 0 && is_tail(pg)) ? Kts : Ks;  // wave-uniform
#pragma unroll
      for (int j = 0; j < C::NLD; ++j) {
        const uint32_t ko = min(t0 * (D * 2) + (j * 64 + lane) * 16, last);
        const u32x4* a = (const u32x4*)(kb + ko);
        kreg[x][j] = STREAM ? __builtin_nontemporal_load(a) : *a;
      }
    }
  };
  // Groups of a page present in the store (wave-uniform).
  auto run_groups = [&](const PairMeta& M, int x) -> uint32_t {
    const uint32_t r0 = M.run0[x];
    const uint32_t store = is_tail(M.pgs[x]) ? (uint32_t)tail_cap * G : cap;
    const uint32_t r1 = M.pgs[x] < 0 ? 0u : min(M.run1[x], store);
    const uint32_t rg = r1 > r0 ? r1 - r0 : 0u;
    return min(rg, (uint32_t)(kPage * G));
  };
  // Packed V runs of a pair, flat; lanes past the end of a run read its last unit (of an empty run
  // the store's first), which no token refers to.
#define STC_ISSUE_V(vreg, M)                                                                   \
  static_for<0, NX>([&](auto x) {                                                               \
    const uint32_t rbytes = run_groups(M, x) * gbytes;                                         \
    const unsigned char* vrun = ((M.pgs[x] >= 0 && is_tail(M.pgs[x])) ? vts : vs) +            \
                                (rbytes ? (size_t)M.run0[x] * gbytes : (size_t)0);             \
    const uint32_t last = rbytes ? rbytes - 16u : 0u;                                          \
    static_for<0, C::NLD>([&](auto j) {                                                        \
      const u32x4* a = (const u32x4*)(vrun + min((uint32_t)((j * 64 + lane) * 16), last));     \
      vreg[x][j] = STREAM ? __builtin_nontemporal_load(a) : *a;                                \
    });                                                                                        \
  })

  // acc: a pair's weighted values relative to the pair's own maximum; sum: of all pairs so far.
  // Every pair is a partial result of its own, merged like those of different wavefronts: weights
  // relative to a running maximum would lose the exact 1 that each pair's largest weight is (256
  // streams of 64 pages: 1.1e-6 against 64 bits instead of 8.3e-7).
  f32x4 acc[C::CB], sum[MULTI ? C::CB : 1];
#pragma unroll
  for (int cb = 0; cb < C::CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (MULTI) {
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) sum[cb] = acc[cb];
  }
  float m_run = kNegBig, l_part = 0.f;
  float r_sum = 0.f, r_pair = 1.f;  // factors of sum and acc in the merge (MULTI)

  // The scheduling fences keep the request order stated above.
  PairMeta meta;
  issue_meta(meta, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue_k(meta);
  __builtin_amdgcn_sched_barrier(0);

  // B operand of the QK product: this lane's 8 channels of head r16 for every 32-channel step
  u32x4 qreg[C::KC];
  {
    const unsigned char* qs = (const unsigned char*)q + (size_t)stream * R * D * 2;
    const uint32_t qo = ((r16 < R ? r16 : 0) * D + 8 * kg) * 2;
#pragma unroll
    for (int j = 0; j < C::KC; ++j)
      qreg[j] = *(const u32x4*)(qs + (qo + 64 * j));  // columns >= R repeat head 0, never used
  }
  __builtin_amdgcn_sched_barrier(0);

  // logits of a pair, online softmax; leaves the weights of the pair in phi/plo
  u32x4 phi, plo;
  auto qk_softmax = [&](const PairMeta& M, int pair) {
    // K rows of the pair -> LDS tiles (row stride ROW), then back in MFMA operand layout
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
      for (int j = 0; j < C::NLD; ++j)
        *(u32x4*)(wl + (x * C::TILE + ((j * 64 + lane) / C::LPR) * C::ROW +
                        (lane % C::LPR) * 16)) = kreg[x][j];
    wave_lds_sync();
    float s[NX][4];
    float mx = kNegBig;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      f32x4 sv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < C::KC; ++j) {
        // A operand: token r16, channels 32*j + 8*kg .. +8 from the K tile
        const u32x4 a = *(const u32x4*)(wl + (x * C::TILE + r16 * C::ROW + (4 * j + kg) * 16));
        sv = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(qreg[j]), sv, 0, 0, 0);
      }
      // this lane holds tokens 4*kg + i of page x for head r16
      const int pg = M.pgs[x];
      const uint32_t t0 = pg < 0 ? 0 : page_no(pg) * kPage;
      const uint32_t lim = tok_lim(pg);
      // a head that did not select this page gives its tokens no weight
      const bool mine = (__builtin_amdgcn_readlane(my_heads, NX * pair + x) >> r16) & 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool tv = pg >= 0 && mine && (t0 + 4 * kg + i < lim);
        s[x][i] = tv ? sv[i] * scale : -INFINITY;  // weight of an absent token is exactly 0
        mx = fmaxf(mx, s[x][i]);
      }
    }
    mx = across_k_groups(mx, [](float a, float b) { return fmaxf(a, b); });
    const float m_pair = fmaxf(kNegBig, mx);
    float p[4 * NX];
    float psum = 0.f;
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[x * 4 + i] = __builtin_amdgcn_exp2f(s[x][i] - m_pair);  // m_pair is finite
        psum += p[x * 4 + i];
      }
    if constexpr (MULTI) {
      const float m_new = fmaxf(m_run, m_pair);
      r_sum = __builtin_amdgcn_exp2f(m_run - m_new);
      r_pair = __builtin_amdgcn_exp2f(m_pair - m_new);
      m_run = m_new;
      l_part = l_part * r_sum + psum * r_pair;
    } else {
      m_run = m_pair;
      l_part = psum;
    }
    // weights as two bf16 parts; contraction index: (kg, e) e<4 page 0, e>=4 page 1
    uint32_t h[4] = {0u, 0u, 0u, 0u}, l[4] = {0u, 0u, 0u, 0u};  // one page: no weight for another
#pragma unroll
    for (int r = 0; r < 2 * NX; ++r) {
      h[r] = pack_bf16(p[2 * r], p[2 * r + 1]);
      l[r] = pack_bf16(p[2 * r] - bf16_lo(h[r]), p[2 * r + 1] - bf16_hi(h[r]));
    }
    phi = u32x4{h[0], h[1], h[2], h[3]};
    plo = u32x4{l[0], l[1], l[2], l[3]};
  };

  // packed runs of a pair -> LDS, then O^T += V~^T . P^T
#define STC_PV(vreg, M)                                                                        \
  {                                                                                            \
    wave_lds_sync(); /* the K tiles have been read */                                          \
    static_for<0, NX>([&](auto x) {                                                             \
      static_for<0, C::NLD>([&](auto j) {                                                      \
        *(u32x4*)(wl + (x * C::TILE + (j * 64 + lane) * 16)) = vreg[x][j];                     \
      });                                                                                      \
    });                                                                                        \
    if (lane < 32) { /* token lane: kept-group mask and offset relative to the run */         \
      const uint32_t r0 = (lane & 16) ? M.run0[NX - 1] : M.run0[0];                            \
      const uint32_t rel = min(M.off - r0, 0xffffu);                                           \
      *(uint32_t*)(wl + C::META + lane * 4) = (M.mvalid ? M.mk : 0u) | (rel << 16);            \
    }                                                                                          \
    wave_lds_sync();                                                                           \
    /* t[e]: channels r16*CB .. +CB of token e of this lane's k-group (e < 4: page 0) */       \
    uint32_t t[4 * NX][C::CB / 2];                                                             \
    _Pragma("unroll") for (int x = 0; x < NX; ++x) {                                            \
      const uint32_t rg = run_groups(M, x);                                                    \
      const u32x4 mt = *(const u32x4*)(wl + C::META + x * 64 + kg * 16);                       \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                          \
        const uint32_t m = mt[i] & 0xffffu;                                                    \
        const uint32_t slot = (mt[i] >> 16) + __popc(m & u_below);                             \
        const bool kept = ((m >> u_g) & 1u) && slot < rg;                                      \
        const uint32_t a = kept ? x * C::TILE + slot * gbytes + u_within : (uint32_t)C::ZERO;  \
        if constexpr (D == 128) {                                                              \
          const u32x4 v = *(const u32x4*)(wl + a);                                             \
          t[x * 4 + i][0] = v.x, t[x * 4 + i][1] = v.y, t[x * 4 + i][2] = v.z,                 \
                       t[x * 4 + i][3] = v.w;                                                  \
        } else {                                                                               \
          const u32x2 v = *(const u32x2*)(wl + a);                                             \
          t[x * 4 + i][0] = v.x, t[x * 4 + i][1] = v.y;                                        \
        }                                                                                      \
      }                                                                                        \
    }                                                                                          \
    _Pragma("unroll") for (int cb = 0; cb < C::CB; ++cb) {                                     \
      const uint32_t sel = (cb & 1) ? 0x07060302u : 0x05040100u;                               \
      uint32_t a[4] = {0u, 0u, 0u, 0u};                                                        \
      _Pragma("unroll") for (int r = 0; r < 2 * NX; ++r) a[r] =                                \
          __builtin_amdgcn_perm(t[2 * r + 1][cb >> 1], t[2 * r][cb >> 1], sel);                \
      const bf16x8 av = as_bf16x8(u32x4{a[0], a[1], a[2], a[3]});                              \
      acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, as_bf16x8(phi), acc[cb], 0, 0, 0); \
      acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, as_bf16x8(plo), acc[cb], 0, 0, 0); \
    }                                                                                          \
    wave_lds_sync(); /* the next pair overwrites the tiles */                                  \
  }

  if (npairs > 0) {
    // The value requests of a pair are held back until its masks/offsets have arrived:
    // a wavefront then has one pair of K pages or one pair of V runs plus the next K
    // pages outstanding, which keeps the chip-wide volume of outstanding requests near
    // what the memory system sustains.  (Requesting everything at once is slower.)
    // With several pairs per wavefront the masks, offsets and K pages of the next pair are
    // requested as soon as the current pair's K pages have left their registers.
    for (int pair = 0;; ++pair) {
      finish_meta(meta);
      u32x4 vreg[2][C::NLD];
      STC_ISSUE_V(vreg, meta);
      __builtin_amdgcn_sched_barrier(0);
      PairMeta next;
      if constexpr (MULTI) {
        issue_meta(next, pair + 1);  // past the last pair: no pages
        __builtin_amdgcn_sched_barrier(0);
      }
      qk_softmax(meta, pair);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (MULTI) {
        issue_k(next);
        __builtin_amdgcn_sched_barrier(0);
      }
      STC_PV(vreg, meta);
      if constexpr (MULTI) {
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[cb][i] = fmaf(sum[cb][i], r_sum, acc[cb][i] * r_pair);
          acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      if (!MULTI || pair + 1 >= npairs) break;
      meta = next;
    }
  }

  if constexpr (MULTI) {
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) acc[cb] = sum[cb];
  }
  // sum of weights of head r16 over this wavefront's tokens
  const float l = across_k_groups(l_part, [](float a, float b) { return a + b; });

  // ---- merge the workgroup's wavefronts: each leaves (m, l, acc[16][D]) in its own LDS region.
  // acc[cb][i] of lane (head r16, kg) is channel (4*kg + i)*CB + cb.
  float* macc = (float*)wl;             // [16][MROW]
  float* mml = (float*)(wl + C::MML);    // [16][2]
  if (r16 < R) {  // the other columns are copies of head 0
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float* dst = macc + r16 * C::MROW + (4 * kg + i) * C::CB;
#pragma unroll
      for (int c4 = 0; c4 < C::CB / 4; ++c4)
        *(f32x4*)(dst + 4 * c4) = f32x4{acc[4 * c4][i], acc[4 * c4 + 1][i], acc[4 * c4 + 2][i],
                                        acc[4 * c4 + 3][i]};
    }
    if (kg == 0) *(f32x2*)(mml + r16 * 2) = f32x2{m_run, l};
  }
  __syncthreads();
  // A thread takes 4 adjacent channels of a head, or one where that still is one round and the
  // channels are divided by the sum (divisions of a thread follow each other; one head of 64
  // channels: 6.5 us per step with 4, 6.3 with one).
  auto merge = [&](auto vec) {
    constexpr int V = vec;
    typedef __attribute__((ext_vector_type(V), aligned(4 * V))) float fvec;
    typedef __attribute__((ext_vector_type(V), aligned(V > 1 ? 8 : 4))) float fvec_partial;
    for (int i = threadIdx.x; i < R * (D / V); i += 64 * WAVES) {
      const int head = i / (D / V), c = i % (D / V) * V;
      f32x2 ml[WAVES];
      fvec part[WAVES];
      float m = kNegBig;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        ml[w] = *(const f32x2*)(lds + w * C::WAVE_LDS + C::MML + head * 8);
        part[w] = *(const fvec*)(lds + w * C::WAVE_LDS + (head * C::MROW + c) * 4);
        m = fmaxf(m, ml[w].x);
      }
      float lsum = 0.f;
      fvec a = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const float wgt = __builtin_amdgcn_exp2f(ml[w].x - m);
        lsum = fmaf(wgt, ml[w].y, lsum);
#pragma unroll
        for (int e = 0; e < V; ++e) a[e] = fmaf(wgt, part[w][e], a[e]);
      }
      const size_t hf = (size_t)stream * R + head;
      if (splits == 1) {
        fvec o;
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = lsum > 0.f ? a[e] / lsum : 0.f;
        *(fvec*)(out + hf * D + c) = o;
      } else {
        float* pr = partial + (hf * splits + split) * partial_stride(D);
        *(fvec_partial*)(pr + 2 + c) = a;
        if (c == 0) *(f32x2*)pr = f32x2{m, lsum};
      }
    }
  };
  if (splits == 1 && R * D <= 64 * WAVES)
    merge(IC<1>{});
  else
    merge(IC<4>{});
  // One pair per wavefront: the list is written behind all loads, with which a store in front of
  // them would be waited for.
  if constexpr (SELECT_IPT > 0 && !MULTI) {
    if ((int)threadIdx.x < WAVES * ppw && lo + (int)threadIdx.x < k_pages)
      sel_list[(size_t)stream * k_pages + lo + threadIdx.x] = s_pages[threadIdx.x];
  }
}

#undef STC_ISSUE_V
#undef STC_PV

}  // namespace stc
