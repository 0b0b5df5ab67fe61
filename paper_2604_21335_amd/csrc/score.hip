// Quest page scores (query-aware token-level stage, Sec. 3.2):
//   U_h[p] = sum_c max(q_h[c]*mn[p,c], q_h[c]*mx[p,c]),  score[p] = max_h U_h[p]
// in float, the D terms summed as a balanced tree over adjacent channels.
//
// Because mn <= mx, the larger product is q*mx for q >= 0 and q*mn for q < 0, so with
// q- = min(q, 0) and q+ = max(q, 0) a term is q-*mn + q+*mx, where one of the two products
// is an exact zero.  That is a 2-slot dot product, and the matrix cores compute it:
// v_mfma_f32_4x4x4_16b_bf16 multiplies, per block, a 4x4 A (rows = query heads, 4 k-slots)
// with a 4x4 B (k-slots, columns = pages).  A k-slot pair holds (mn, mx) of one channel
// and the A row holds (q-, q+) in that pair and zeros in the other pair.  A product of two
// bf16 values is exact in float and the other three addends are zeros, so the result is
// the exact term whatever rounding the unit applies to longer sums (it does not round
// sums of two non-zero products to nearest, which is why the pair sums stay on the VALU).
// All additions of the tree are then ordinary float additions, in the fixed order.
//
// The bounds are stored in tiles of 8 pages laid out for this kernel (see
// bounds_tile_unit): a wavefront fetches a tile with D/32 fully contiguous 1 KiB
// requests and every 64-bit register pair it receives is a B operand as it stands.
// Lane l of a wavefront holds, for page 4*(l/32) + l%4 of the tile, the D/8 channels
// of chunk (l/4)%8; the 16 blocks of the MFMA are the 16 (page group, chunk) pairs.
#include "score_tiles.hpp"
#include "stc_common.hpp"
#include "stc_kernels.hpp"
#include "topk_block.hpp"

namespace stc {

typedef score_u32x4 u32x4;

// The scores of a range of a stream's tiles with the query operands in shared memory
// (score_tiles.hpp): at most 128 registers, so four wavefronts per SIMD for any number of heads
// per KV head.  R up to 8 is exact; R = 16 serves 9 .. 16 heads.  Measured against the forms that
// were used for up to 4 heads (operands in registers, two tiles ahead), D = 64 and more
// than 8 heads (one head at a time on the vector ALUs): 256 streams of 1024 pages 21.8 us for
// 26.9, 32 streams of 4096 pages at 3 heads 12.0 for 14.6, 40 of 1001 pages at 16 heads and
// D = 64 5.8 for 14.7, 64 of 2048 pages at 16 heads 18.6 for 67.7.
template <int D, int R, bool PER_HEAD, int WAVES, bool STREAM>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(4, 8)))
void score_lds_kernel(const u32x4* __restrict__ tiles, const uint16_t* __restrict__ q,
                      float* __restrict__ score, int NP, int group, int tiles_per_block,
                      int tiles_cap) {
  constexpr int T16 = (D / 32) * 64;
  __shared__ __align__(16) unsigned char s_q[score_q_lds_bytes<D, R>()];
  const int stream = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntiles = (NP + kBoundsTilePages - 1) / kBoundsTilePages;
  const int t0 = blockIdx.x * tiles_per_block;
  const int t1 = min(t0 + tiles_per_block, ntiles);
  const int heads = R > 8 ? group : R;  // groups of more than 8 heads share one instance
  ScoreQuery<D, R, 64 * WAVES> sq;
  sq.load(q + (size_t)stream * heads * D, heads);  // [B, Hkv, heads, D]
  score_tile_range<D, R, PER_HEAD, WAVES, 1, STREAM>(
      (const score_u32x4*)tiles + (size_t)stream * tiles_cap * T16 + lane,
      score + (size_t)stream * (PER_HEAD ? heads : 1) * NP, NP, t0, t1, s_q, wave, lane,
      [&] {
        sq.store(s_q, heads);
        __syncthreads();
      },
      heads);
}

template <int D>
static void launch_score_d(const stc_shape_t& s, const void* q, const void* bounds, float* score,
                           int NP, bool per_head, hipStream_t st) {
  const int streams = s.B * s.Hkv;
  const int R = s.Hq / s.Hkv;
  const int ntiles = (NP + kBoundsTilePages - 1) / kBoundsTilePages;
  const int tcap = bounds_tiles(token_cap(s));  // tiles per stream in memory
  constexpr int T16 = (D / 32) * 64;            // 16-byte units per tile
  const u32x4* t4 = (const u32x4*)bounds;
  const uint16_t* q16 = (const uint16_t*)q;
  // Query operands in shared memory, one tile requested at a time per wavefront (measured: two
  // requested ahead is slower at every grid), about 4096 wavefronts (512 workgroups of 8 or 1024 of
  // 4).  Streaming loads from 64 MiB of bounds on.  us, bounds in the caches / out of them:
  //                                    ordinary loads, wavefronts           streaming loads
  //    MiB  streams x pages, heads    2048         4096         8192              4096
  //     16   128 x  250, 4          4.0 /  5.9   3.6 /  5.5   3.6 /  5.6       4.2 /  5.8
  //     32   256 x  256, 4          5.3 /  8.7   4.8 /  7.6   5.1 /  8.1       6.8 /  7.5
  //     32    32 x 2048, 7          6.6 /  9.1   6.2 /  7.8   6.2 /  8.5       7.7 /  8.2
  //     64    64 x 2048, 7         12.5 / 15.8  12.2 / 13.4  12.3 / 13.3      12.3 / 12.8
  //     64   256 x 1024, 1, D = 64 11.5 / 16.9  11.5 / 14.9  11.2 / 14.0      12.5 / 13.1
  //    128   256 x 1024, 4         20.7 / 25.6  20.3 / 25.1  20.4 / 25.5      20.9 / 21.9
  // So up to 32 MiB ordinary loads are no slower even where nothing is cached, and much faster
  // where it is; from 64 MiB on streaming ones gain 5 to 13 % where a decoder's other layers have
  // pushed the bounds out, and lose 1 to 8 % where a single cache is stepped by itself.
  const bool stream_loads = (long long)streams * ntiles * T16 * 16 >= (64ll << 20);
  // Up to 4 heads per KV head, whose tiles take half as long, half as many workgroups of twice the
  // size start sooner (128 streams of 250 pages: 19.9 against 20.4 us per step; the figures of 4
  // heads above are of this form).
  const int waves = R <= 4 ? 8 : 4;
  const int want = max(1, 4096 / waves / streams);
  int tp = (ntiles + want - 1) / want;
  tp = (tp + waves - 1) / waves * waves;
  const dim3 grid((ntiles + tp - 1) / tp, streams);
#define STC_SCORE_GO(RR, PH, STREAM)                                                              \
  score_lds_kernel<D, RR, PH, (RR <= 4 ? 8 : 4), STREAM><<<grid, 64 * waves, 0, st>>>(            \
      t4, q16, score, NP, R, tp, tcap)
#define STC_SCORE_CASE(RR)                                                                        \
  case RR:                                                                                        \
    if (per_head) {                                                                               \
      if (stream_loads) STC_SCORE_GO(RR, true, true);                                             \
      else STC_SCORE_GO(RR, true, false);                                                         \
    } else {                                                                                      \
      if (stream_loads) STC_SCORE_GO(RR, false, true);                                            \
      else STC_SCORE_GO(RR, false, false);                                                        \
    }                                                                                             \
    break;
  switch (R <= 8 ? R : 16) {
    STC_SCORE_CASE(1)
    STC_SCORE_CASE(2)
    STC_SCORE_CASE(3)
    STC_SCORE_CASE(4)
    STC_SCORE_CASE(5)
    STC_SCORE_CASE(6)
    STC_SCORE_CASE(7)
    STC_SCORE_CASE(8)
    STC_SCORE_CASE(16)
  }
#undef STC_SCORE_CASE
#undef STC_SCORE_GO
}

// One workgroup of 8 wavefronts scores a whole stream (NP <= PAGES) into LDS and then selects the
// stream's k pages itself (`score` is an optional copy of the scores): the form for many streams
// of few pages each, where a stream per workgroup still fills the chip and the selection needs
// no launch of its own.  RM: at most this many query heads per KV head.
template <int D, int RM, int PAGES>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8)))
void score_select_kernel(const u32x4* __restrict__ tiles, const uint16_t* __restrict__ q,
                         float* __restrict__ score, int NP, int heads, int tiles_cap,
                         int32_t* __restrict__ page_idx, int k_pages) {
  constexpr int WAVES = 8, T16 = (D / 32) * 64;
  __shared__ __align__(16) unsigned char s_q[score_q_lds_bytes<D, RM>()];
  __shared__ __align__(16) float s_score[PAGES];
  __shared__ TopkLds<PAGES / 512, 512> s_topk;
  const int stream = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntiles = (NP + kBoundsTilePages - 1) / kBoundsTilePages;
  ScoreQuery<D, RM, 64 * WAVES> sq;
  sq.load(q + (size_t)stream * heads * D, heads);
  score_tile_range<D, RM, false, WAVES, 2>(
      tiles + (size_t)stream * tiles_cap * T16 + lane, s_score, NP, 0, ntiles, s_q, wave, lane,
      [&] {
        sq.store(s_q, heads);
        __syncthreads();
      },
      heads);
  __syncthreads();
  if (score)
    for (int i = threadIdx.x; i < NP; i += 64 * WAVES) score[(size_t)stream * NP + i] = s_score[i];
  int32_t* list = page_idx + (size_t)stream * k_pages;
  topk_block<PAGES / (64 * WAVES), 64 * WAVES>(
      s_score, NP, k_pages, s_topk, [list](int pos, int page) { list[pos] = page; });
}

template <int D>
static int launch_score_select_d(const stc_shape_t& s, const void* q, const void* bounds,
                                 float* score, int32_t* page_idx, int k_pages, int NP,
                                 hipStream_t st) {
  const int streams = s.B * s.Hkv, R = s.Hq / s.Hkv;
  const int tcap = bounds_tiles(token_cap(s));
#define STC_SCORE_SELECT(RM, PAGES)                                                            \
  score_select_kernel<D, RM, PAGES><<<streams, 512, 0, st>>>(                                  \
      (const u32x4*)bounds, (const uint16_t*)q, score, NP, R, tcap, page_idx, k_pages)
#define STC_SCORE_SELECT_PAGES(RM)                                                             \
  if (NP <= 512) STC_SCORE_SELECT(RM, 512);                                                    \
  else STC_SCORE_SELECT(RM, 1024);
  if (R == 1) { STC_SCORE_SELECT_PAGES(1) }
  else if (R == 2) { STC_SCORE_SELECT_PAGES(2) }
  else if (R <= 4) { STC_SCORE_SELECT_PAGES(4) }
  else if (R <= 8) STC_SCORE_SELECT(8, 512);  // (score_can_select: at most 256 pages)
  else return -1;
#undef STC_SCORE_SELECT_PAGES
#undef STC_SCORE_SELECT
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Where the single workgroup per stream wins: on short streams, where both forms are bound by their
// launches, and on longer ones with few heads per KV head while the streams fill the chip without
// many rounds (two of the workgroups fit a CU at D = 128, four at D = 64).  Its time over that of
// scoring and selection as two launches, bounds in the caches / out of them, 4 heads:
//   D   pages    128 streams    192         256         320         512         1024
//   128   257    0.81 / 0.88  0.73 / 0.81 0.74 / 0.83 0.90 / 0.89 0.97 / 0.95 0.93 / 1.02
//         512    1.01 / 1.06  1.01 / 0.92 0.91 / 0.98 0.94 / 1.01 0.99 / 1.02 0.94 / 1.06
//        1024    0.97 / 1.13  0.87 / 1.04 0.94 / 1.02 0.92 / 1.09 0.97 / 1.10 1.10 / 1.09
//    64   512    0.98 / 0.97  0.87 / 0.89 0.87 / 0.94 0.88 / 0.86 0.94 / 0.95 0.91 / 0.96
//        1024    1.07 / 1.18  1.00 / 0.96 0.83 / 0.96 0.87 / 0.99 0.94 / 1.02 0.91 / 1.01
// 64 streams of 512 pages 1.09 / 1.15; with 7 heads 128 streams of 512 pages 1.11 / 1.18, 320 of 384
// 1.04 / 1.07.  (256 streams of 257 pages: 8.1 us for 11.2.)  Whole steps of 512 streams: 300 pages
// 57.6 / 60.5 us for 58.4 / 59.0, 500 pages 88.1 / 94.1 for 90.6 / 90.1.
bool score_can_select(const stc_shape_t& s, int k_pages) {
  const int NP = (s.N + kPage - 1) / kPage;
  const int R = s.Hq / s.Hkv, streams = s.B * s.Hkv;
  if (k_pages >= NP || R > 8) return false;
  if (NP <= 256) return true;
  if (R > 4 || streams < 128) return false;
  return NP <= 640 && streams <= (s.D == 128 ? 384 : 1024);
}

int launch_score_select(const stc_shape_t& s, const void* q, const void* bounds, float* score,
                        int32_t* page_idx, int k_pages, hipStream_t st) {
  const int NP = (s.N + kPage - 1) / kPage;
  return s.D == 128 ? launch_score_select_d<128>(s, q, bounds, score, page_idx, k_pages, NP, st)
                    : launch_score_select_d<64>(s, q, bounds, score, page_idx, k_pages, NP, st);
}

int launch_score(const stc_shape_t& s, const void* q, const void* bounds, float* score,
                 bool per_head, hipStream_t st) {
  const int NP = (s.N + kPage - 1) / kPage;
  if (s.D == 128)
    launch_score_d<128>(s, q, bounds, score, NP, per_head, st);
  else
    launch_score_d<64>(s, q, bounds, score, NP, per_head, st);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
