// Shared device helpers for the libstc kernels (gfx950 only, 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stc_kernels.hpp"

namespace stc {

// Compile-time loop: f(integral_constant<int, I>) for I in [B, E).  Register arrays
// indexed through it have constant indices from the start, so they never land in
// scratch memory.
template <int I>
struct IC {
  static constexpr int value = I;
  constexpr operator int() const { return I; }
};
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(IC<B>{});
    static_for<B + 1, E>(f);
  }
}

constexpr int kWave = 64;
constexpr int kPage = 16;

// Page bounds are stored in tiles of 8 pages.  A tile is D/32 rows of 64 units of 16 bytes;
// a unit holds 4 adjacent channels of one page, each as a dword (bf16 minimum in the low
// half, bf16 maximum in the high half).  With CH = D/8 channels per chunk, channel c of page
// pt of the tile sits in row (c % CH) / 4, unit (pt % 4) + 4 * (c / CH) + 32 * (pt / 4),
// dword c % 4.  (The unit number is the lane of the wavefront that scores it.)
__host__ __device__ constexpr int bounds_tile_dwords(int D) { return kBoundsTilePages * D; }
__host__ __device__ constexpr int bounds_tile_unit(int D, int pt, int c) {
  return ((c % (D / 8)) / 4) * 64 + (pt % 4) + 4 * (c / (D / 8)) + 32 * (pt / 4);
}

// bf16 pair in one dword: element 2i in the low half, 2i+1 in the high half.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// DPP lane move inside a row of 16 lanes (control codes of the gfx9 DPP encoding; lanes
// without a source read 0).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Rows 0,1 and rows 2,3 (of 16 lanes) exchange values: every lane gets the sum of its own
// and the partner row's value.
__device__ __forceinline__ float row_pair_sum(float u) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u), __float_as_uint(u), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the 8 lanes that share lane bits 0, 1 and 5 (lane bits 2, 3, 4 count the chunks of
// a page, or the pieces of a token's channel chunk), continuing the balanced tree: chunks
// (0,1)(2,3).. first.  row_ror:n makes lane i read lane i-n of its row, so after the
// two rotations the lanes with bit 2 set hold ((c0+c1)+(c2+c3)) of their row; the row
// exchange adds chunks 4..7.  Valid in lanes with (lane & 0x1c) == 4.
__device__ __forceinline__ float chunk_tree_sum(float u) {
  u += dpp_f32<0x124>(u);  // row_ror:4
  u += dpp_f32<0x128>(u);  // row_ror:8
  return row_pair_sum(u);
}
constexpr int kChunkSumLanes = 4;  // (lane & 0x1c) of the lanes that hold the sum

// Order-preserving map of float bits to unsigned keys (finite inputs).
__device__ __forceinline__ uint32_t float_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Orders a wavefront's own accesses to shared memory across its lanes.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One step of a wavefront scan on the data-parallel-primitive path (no LDS traffic): lanes
// whose source lies outside the row, or whose row is masked off, combine with `ident`.
#define STC_DPP_STEP(v, op, ident, ctrl, row_mask) \
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)(ident), (int)(v), ctrl, row_mask, 0xf, false))

struct OpAdd {
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; }
};
struct OpMin {
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return min(a, b); }
};
struct OpMax {
  __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); }
};

// Inclusive scan over the 64 lanes: shifts by 1, 2, 4, 8 inside each row of 16 lanes, then
// lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v, Op op, uint32_t ident) {
  STC_DPP_STEP(v, op, ident, 0x111, 0xf);  // row_shr:1
  STC_DPP_STEP(v, op, ident, 0x112, 0xf);  // row_shr:2
  STC_DPP_STEP(v, op, ident, 0x114, 0xf);  // row_shr:4
  STC_DPP_STEP(v, op, ident, 0x118, 0xf);  // row_shr:8
  STC_DPP_STEP(v, op, ident, 0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  STC_DPP_STEP(v, op, ident, 0x143, 0xc);  // row_bcast:31 into rows 2 and 3
  return v;
}
#undef STC_DPP_STEP

// Reduction over the 64 lanes, in a scalar register.
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op, uint32_t ident) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(v, op, ident), 63);
}

// a[j] by selects.  An array that is indexed at run time would be put into memory, which is also what
// the compiler makes of selects between two elements unless it cannot see that they are.
template <class T, int N>
__device__ __forceinline__ T pick_of(const T (&a)[N], int j) {
  if constexpr (N == 1) {
    return a[0];
  } else {
    T half[N / 2];
    static_for<0, N / 2>([&](auto i) {
      T even = a[2 * i], odd = a[2 * i + 1];
      asm("" : "+v"(even), "+v"(odd));
      half[i] = (j & 1) ? odd : even;
    });
    return pick_of(half, j >> 1);
  }
}

}  // namespace stc
