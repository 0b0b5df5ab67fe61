// Device helpers shared by the cache-construction kernels and the kernel that appends tokens
// to a built cache.
#pragma once
#include "stc_common.hpp"

namespace stc {

typedef __attribute__((ext_vector_type(4))) float logit4;

// The G logits of one token (16-byte loads when G is a multiple of 4: the row is then
// 16-byte aligned).  STREAM: with loads that leave the caches alone.
template <int G, bool STREAM = false>
__device__ __forceinline__ void load_token_logits(const float* __restrict__ lp, float (&a)[G]) {
  if constexpr ((G & 3) == 0) {
#pragma unroll
    for (int q = 0; q < G / 4; ++q) {
      const logit4* p = (const logit4*)(lp + 4 * q);
      const logit4 v = STREAM ? __builtin_nontemporal_load(p) : *p;
      a[4 * q] = v.x, a[4 * q + 1] = v.y, a[4 * q + 2] = v.z, a[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g) a[g] = lp[g];
  }
}

// Routing mask of one token: bit g set iff group g is among the c largest of its G logits
// (equal logits: the lower group first).
template <int G, bool STREAM>
__device__ __forceinline__ uint32_t rank_mask_g(const float* __restrict__ lp, int c) {
  float a[G];
  load_token_logits<G, STREAM>(lp, a);
  uint32_t m = 0;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    int ahead = 0;  // groups ranked before g: larger logit, or equal with lower index
#pragma unroll
    for (int g2 = 0; g2 < G; ++g2)
      if (g2 != g) ahead += (a[g2] > a[g]) || (g2 < g && a[g2] == a[g]);
    if (ahead < c) m |= 1u << g;
  }
  return m;
}

// The same for a group count known at run time (a power of two up to 16, uniform over the
// launch: the switch is a scalar branch).
template <bool STREAM = false>
__device__ __forceinline__ uint32_t rank_mask(const float* __restrict__ lp, int c, int G) {
  switch (G) {
    case 1: return rank_mask_g<1, STREAM>(lp, c);
    case 2: return rank_mask_g<2, STREAM>(lp, c);
    case 4: return rank_mask_g<4, STREAM>(lp, c);
    case 8: return rank_mask_g<8, STREAM>(lp, c);
    case 16: return rank_mask_g<16, STREAM>(lp, c);
    default: return 0u;
  }
}

typedef __attribute__((ext_vector_type(2))) short i16x2;
typedef __attribute__((ext_vector_type(4))) uint32_t bounds_u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t bounds_u32x2;

// Two bf16 patterns per dword <-> two signed 16-bit integers in the same order (-0 below +0);
// the map is its own inverse.
__device__ __forceinline__ i16x2 bf16_order2(i16x2 x) {
  return x ^ ((x >> 15) & (i16x2){0x7fff, 0x7fff});
}

// Lanes that differ in lane bit 5 (SWAP 32) or bit 4 (SWAP 16) hold the same two quantities a
// and b for different rows: the swap gives one half of the lanes both values of a, the other
// half both values of b, so one min/max reduces both.
template <int SWAP, class Op>
__device__ __forceinline__ i16x2 fold_pair(i16x2 a, i16x2 b, Op op) {
  const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
  const auto r = SWAP == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                            : __builtin_amdgcn_permlane16_swap(x, y, false, false);
  return op(__builtin_bit_cast(i16x2, (uint32_t)r[0]), __builtin_bit_cast(i16x2, (uint32_t)r[1]));
}

// A wavefront's part of a page's bounds in the tiled layout: the two channels 8*piece + 2*(lane/16), +1
// of the lane's piece (lane % (D/8)), as (minimum | maximum << 16) each.
template <int D>
__device__ __forceinline__ void put_page_bounds(uint32_t* __restrict__ stream_tiles, int page,
                                                bounds_u32x2 w, int lane) {
  const int c = 8 * (lane % (D / 8)) + 2 * (lane >> 4);
  if (D == 128 || (lane & 8) == 0)
    *(bounds_u32x2*)(stream_tiles + (size_t)(page / kBoundsTilePages) * bounds_tile_dwords(D) +
                     bounds_tile_unit(D, page % kBoundsTilePages, c) * 4 + c % 4) = w;
}

// The bounds of a page by one wavefront.  v[j]: the lane's 16-byte piece of row j*RPL + lane/LPR, with
// LPR = D/8 lanes per token row and RPL = 64/LPR rows per request, so that lanes l + LPR*i hold
// the same channels of different rows.  Minima and maxima are taken on packed 16-bit integers, first
// over a lane's own rows, then across lanes by swapping halves of register pairs, which leaves
// every lane with the minimum and maximum of two channels.  !present: a padding page, zeros.
template <int D>
__device__ __forceinline__ void store_page_bounds(uint32_t* __restrict__ stream_tiles, int page,
                                                  bool present, const bounds_u32x4 (&v)[D / 32],
                                                  int lane) {
  auto lo = [](i16x2 a, i16x2 b) { return __builtin_elementwise_min(a, b); };
  auto hi = [](i16x2 a, i16x2 b) { return __builtin_elementwise_max(a, b); };
  i16x2 mn[4], mx[4];  // channels 8*piece + 2*d, +1
#pragma unroll
  for (int d = 0; d < 4; ++d) {
#pragma unroll
    for (int j = 0; j < D / 32; ++j) {
      const i16x2 k = bf16_order2(__builtin_bit_cast(i16x2, (uint32_t)v[j][d]));
      mn[d] = j ? lo(mn[d], k) : k;
      mx[d] = j ? hi(mx[d], k) : k;
    }
  }
  // lane bit 5 chooses between dwords d and d + 2, lane bit 4 between d and d + 1
  i16x2 a = fold_pair<16>(fold_pair<32>(mn[0], mn[2], lo), fold_pair<32>(mn[1], mn[3], lo), lo);
  i16x2 b = fold_pair<16>(fold_pair<32>(mx[0], mx[2], hi), fold_pair<32>(mx[1], mx[3], hi), hi);
  if constexpr (D == 64) {  // rows also differ in lane bit 3
    a = lo(a, __builtin_bit_cast(i16x2, dpp_f32<0x128>(__builtin_bit_cast(float, a))));
    b = hi(b, __builtin_bit_cast(i16x2, dpp_f32<0x128>(__builtin_bit_cast(float, b))));
  }
  uint32_t mnw = __builtin_bit_cast(uint32_t, bf16_order2(a));
  uint32_t mxw = __builtin_bit_cast(uint32_t, bf16_order2(b));
  if (!present) mnw = mxw = 0u;
  // minimum in the low half, maximum in the high half of each channel's dword
  put_page_bounds<D>(
      stream_tiles, page,
      bounds_u32x2{(mnw & 0xffffu) | (mxw << 16), (mnw >> 16) | (mxw & 0xffff0000u)}, lane);
}

}  // namespace stc
