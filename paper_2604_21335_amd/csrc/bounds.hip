// Quest page summary: per-page, per-channel min and max of the cached keys
// (token-level stage of the paper, Sec. 3.2; chunk size 16 from App. C.1).
#include "build_helpers.hpp"
#include "stc_common.hpp"
#include "stc_kernels.hpp"

namespace stc {

constexpr int kBoundsWavePages = 2;  // adjacent pages per wavefront, all requested at once
constexpr int kBoundsStreamWaves = 7;  // streams of at most this many wavefronts are one workgroup

// One wavefront takes 2 adjacent pages.  Every request is 1 KiB of adjacent addresses (4 token
// rows at D = 128, 8 at D = 64): lane l receives channels 8*(l % LPR) .. +8 of row l / LPR, so
// the lanes l + LPR*i hold the same channels of different rows.  Minima and maxima are taken
// on packed 16-bit integers, first over a lane's own rows, then across lanes by swapping halves
// of register pairs, which leaves every lane with the minimum and maximum of two channels.
// Bound by memory (K is read once, 1/8 of it written).  K is read with streaming loads, which
// leave the caches alone.  Where K was written just before, ordinary loads would be faster for this
// launch (2048 streams of 208 tokens, 109 MB, behind their copy 19.9 us, 21.5), but they push out
// values written beside the keys: compaction of both, bounds and packing of that shape 137.8 us,
// 129.5 with streaming loads.  Measured on 64
// streams of 32768 tokens (604 MB): 95.8 us (6.3 TB/s) against 106.5 with ordinary loads, 113
// with 4 pages per wavefront, 124-137 with wavefronts that walk a run of pages, and 131 for
// the form before, in which a thread walked the 16 rows of a page four loads at a time (a request
// was four pieces of 256 bytes in four pages).
// A workgroup is 4 wavefronts.  A stream of up to 7 is one workgroup that has no wavefronts for the
// padding pages of its last tile: the one with the last page writes their zeros (2048 streams of
// 130 tokens, 9 pages in two tiles: 16.2 us, 19.4 with wavefronts for the padding; 8 wavefronts are
// better as two workgroups, 24.4 us, than as one, 25.9).
template <int D>
__global__ __launch_bounds__(64 * kBoundsStreamWaves) void bounds_kernel(
    const bounds_u32x4* __restrict__ K, uint32_t* __restrict__ bounds, int N, int NP, int Ncap) {
  constexpr int LPR = D / 8;            // lanes per token row
  constexpr int RPL = 64 / LPR;         // rows per request
  constexpr int NLD = kPage / RPL;      // requests per page
  constexpr int PW = kBoundsWavePages;
  const int stream = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int p0 = (blockIdx.x * (blockDim.x >> 6) + wave) * PW;
  const int ptile = (NP + kBoundsTilePages - 1) / kBoundsTilePages * kBoundsTilePages;
  if (p0 >= ptile) return;
  const int piece = lane % LPR, row = lane / LPR;
  const bounds_u32x4* Ks = K + (size_t)stream * Ncap * LPR + piece;
  // rows past the last token repeat it, which changes neither minimum nor maximum
  bounds_u32x4 v[PW][NLD];
#pragma unroll
  for (int p = 0; p < PW; ++p)
#pragma unroll
    for (int j = 0; j < NLD; ++j)
      v[p][j] = __builtin_nontemporal_load(
          Ks + (size_t)min((p0 + p) * kPage + j * RPL + row, N - 1) * LPR);
  uint32_t* tiles = bounds + (size_t)stream * bounds_tiles(Ncap) * bounds_tile_dwords(D);
#pragma unroll
  for (int p = 0; p < PW; ++p) store_page_bounds<D>(tiles, p0 + p, p0 + p < NP, v[p], lane);
  if (gridDim.x == 1 && p0 + PW >= NP)  // the padding pages behind the last wavefront's own
    for (int page = p0 + PW; page < ptile; ++page)
      put_page_bounds<D>(tiles, page, bounds_u32x2{0u, 0u}, lane);
}

int launch_bounds(const stc_shape_t& s, const void* K, void* bounds, hipStream_t st) {
  const int NP = (s.N + kPage - 1) / kPage;
  const int streams = s.B * s.Hkv;
  const int need = (NP + kBoundsWavePages - 1) / kBoundsWavePages;  // wavefronts with a page
  const bool one = need <= kBoundsStreamWaves;
  const int waves = one ? need : 4;
  const int ptile = (NP + kBoundsTilePages - 1) / kBoundsTilePages * kBoundsTilePages;
  dim3 grid(one ? 1 : (ptile / kBoundsWavePages + waves - 1) / waves, streams);
  if (s.D == 128)
    bounds_kernel<128><<<grid, 64 * waves, 0, st>>>((const bounds_u32x4*)K, (uint32_t*)bounds, s.N,
                                                    NP, token_cap(s));
  else
    bounds_kernel<64><<<grid, 64 * waves, 0, st>>>((const bounds_u32x4*)K, (uint32_t*)bounds, s.N,
                                                   NP, token_cap(s));
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
