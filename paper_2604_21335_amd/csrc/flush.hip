// Appending tokens to a built cache: the oldest n tokens of the uncompressed tail become
// tokens N .. N+n-1 of the compressed cache.  Their keys are copied, their values are routed
// (given masks, or per-token top-K of given logits) and packed behind the stream's packed
// store, the offsets are continued from tok_off[N], and the bounds of every page that holds
// one of them are recomputed (the first such page may already hold older tokens).  The
// result is, bit for bit, the cache that construction from scratch over all N+n tokens gives.
// The rows that stay in the tail are then moved to its front.
#include "build_helpers.hpp"
#include "stc_common.hpp"
#include "stc_kernels.hpp"

namespace stc {

// TILE tokens are taken at a time; a thread each routes them, MOVERS other threads move their rows.
template <int TILE, int MOVERS>
constexpr int flush_threads() {
  return (TILE + 63) / 64 * 64 + MOVERS;
}

// One workgroup per stream (cache construction, not the decode path), bound by latency: one chain of
// dependent accesses per stream.  So the rows of a tile are requested while its tokens are routed, by
// other wavefronts, and the bounds are taken from the rows on their way through shared memory
// (64 tokens of 64 streams 4.4 us; 7.6 when the rows were requested after the routing, four times one
// after the other, and the bounds read them back from the cache).
// 128 tokens and 512 movers are one round trip for most flushes, but three such workgroups fill a CU.
// Where the streams are more than the CUs, few tokens go by workgroups of 192 threads and tiles of 32.
// us with the large / the small form (one form of 256 threads, as before the large one):
//   tokens, streams            256            384           1024            4096
//     1, D = 128      3.9 /  3.7 ( 5.8)  5.9 /  3.9   10.3 /  4.5 ( 6.5)  36.8 / 11.9 (19.9)
//    16               4.0 /  3.9 ( 6.7)  6.1 /  4.2   10.7 /  5.3 ( 8.2)  40.5 / 17.9 (26.7)
//    64               5.2 /  6.8 ( 7.7)  8.1 /  7.7   17.1 / 15.0 (16.9)  68.2 / 54.2 (67.2)
//    96               6.1 /  9.0 ( 9.2)  9.0 / 10.5   20.5 / 19.8 (23.6)  86.2 / 90.0 (94.7)
//     1, D = 64       3.8 /  3.6 ( 5.6)  5.6 /  3.8    9.5 /  4.1 ( 6.8)  33.0 /  9.2 (19.1)
//    64               4.5 /  5.8 ( 6.9)  6.5 /  6.3   12.4 /  8.0 (11.0)  43.7 / 26.3 (34.8)
//   128               5.0 /  9.1 ( 7.7)  7.7 / 10.0   16.2 / 14.7 (16.4)  65.1 / 55.0 (65.7)
template <int D, int TILE, int MOVERS>
__global__ __launch_bounds__((flush_threads<TILE, MOVERS>())) void flush_tail_kernel(
    bounds_u32x4* K_tail, bounds_u32x4* V_tail, bounds_u32x4* K, const float* __restrict__ logits,
    const uint8_t* __restrict__ kcount, int n, int N, int Ncap, int tail_cap, int n_tail, int mode,
    int G, int fixed_k, const uint16_t* __restrict__ mask_in, uint32_t* __restrict__ bounds,
    uint16_t* __restrict__ mask, uint32_t* tok_off, bounds_u32x4* __restrict__ vpacked,
    int32_t* dev_status, long long cap) {
  constexpr int PPT = D / 8;                      // 16-byte pieces per token row
  constexpr int NJ = TILE * PPT / MOVERS;         // pieces per thread and tile
  constexpr int THREADS = flush_threads<TILE, MOVERS>(), TW = THREADS / 64 - MOVERS / 64;
  constexpr int RPL = 64 / PPT, NLD = kPage / RPL;  // rows per wavefront access of a page
  __shared__ bounds_u32x4 rows[(TILE + kPage) * PPT];  // key rows from a page's first on
  __shared__ uint32_t s_rel[64 * TW], s_mask[64 * TW], s_tot[2];
  const int stream = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mover = tid - 64 * TW;  // >= 0: moves rows
  bounds_u32x4* Ks = K + (size_t)stream * Ncap * PPT;
  bounds_u32x4* Kt = K_tail + (size_t)stream * tail_cap * PPT;
  bounds_u32x4* Vt = V_tail + (size_t)stream * tail_cap * PPT;
  uint16_t* mk = mask + (size_t)stream * Ncap;
  uint32_t* off = tok_off + (size_t)stream * (Ncap + 1);
  const int lg_ppg = 31 - __clz(PPT) - (31 - __clz(G));  // log2(16-byte pieces per group)
  bounds_u32x4* dst = vpacked + ((size_t)stream * (size_t)cap << lg_ppg);
  uint32_t* tiles = bounds + (size_t)stream * bounds_tiles(Ncap) * bounds_tile_dwords(D);
  const int N1 = N + n;

  uint32_t carry = off[N];  // kept groups of the stream so far = offset of token N
  for (int i0 = 0; i0 < n; i0 += TILE) {
    const int ntok = min(TILE, n - i0);
    const int older = (N + i0) % kPage;  // tokens of the first page that are in the cache already
    bounds_u32x4 kv[NJ], vv[NJ];
    uint32_t m = 0, inc = 0;
    if (wave < TW) {
      const int i = i0 + tid;
      if (tid < ntok) {
        const size_t tok = (size_t)stream * n + i;  // dense per-token inputs of the new tokens
        if (mode == STC_ROUTE_MASK) {
          m = mask_in[tok] & ((1u << G) - 1u);
        } else {
          const int c = kcount ? (int)kcount[tok] : fixed_k;
          m = rank_mask(logits + tok * G, min(c, G), G);
        }
        mk[N + i] = (uint16_t)m;
      }
      const uint32_t kept = __popc(m);
      inc = wave_scan(kept, OpAdd{}, 0u);
      s_rel[tid] = inc - kept;  // of the wavefront's tokens, in front of this one
      s_mask[tid] = m;
      if (lane == 63) s_tot[wave] = inc;
    } else {
      const bounds_u32x4 *kt = Kt + (size_t)i0 * PPT, *vt = Vt + (size_t)i0 * PPT;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int e = min(mover + j * MOVERS, ntok * PPT - 1);
        kv[j] = kt[e], vv[j] = vt[e];
      }
      for (int e = mover; e < older * PPT; e += MOVERS)  // later tiles find them in the tail
        rows[e] = i0 == 0 ? Ks[(size_t)(N - older) * PPT + e] : kt[e - older * PPT];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int e = mover + j * MOVERS;
        if (e < ntok * PPT) rows[older * PPT + e] = kv[j];
      }
    }
    __syncthreads();
    if (wave < TW) {
      if (tid < ntok) off[N + i0 + tid + 1] = carry + (wave ? s_tot[0] : 0u) + inc;
    } else {
      bounds_u32x4* kd = Ks + (size_t)(N + i0) * PPT;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int e = mover + j * MOVERS;
        if (e < ntok * PPT) {
          kd[e] = kv[j];
          const int tk = e / PPT, pc = e % PPT, g = pc >> lg_ppg;
          const uint32_t mm = s_mask[tk];
          if ((mm >> g) & 1u) {
            const long long slot = (long long)(carry + (tk >= 64 ? s_tot[0] : 0u) + s_rel[tk]) +
                                   __popc(mm & ((1u << g) - 1u));
            if (slot < cap) dst[(slot << lg_ppg) + (pc & ((1 << lg_ppg) - 1))] = vv[j];
          }
        }
      }
    }
    // Bounds of the pages that hold a token of the tile, a page per wavefront at a time; one that the
    // next tile continues is left to it.
    const int p0 = (N + i0) / kPage, p1 = (N + i0 + ntok + kPage - 1) / kPage;
    for (int p = p0 + wave; p < p1; p += THREADS / 64) {
      if (i0 + ntok < n && (p + 1) * kPage > N + i0 + ntok) break;
      bounds_u32x4 v[NLD];
#pragma unroll
      for (int j = 0; j < NLD; ++j)  // rows past the last token repeat it
        v[j] = rows[min((p - p0) * kPage + j * RPL + lane / PPT, older + ntok - 1) * PPT + lane % PPT];
      store_page_bounds<D>(tiles, p, true, v, lane);
    }
    carry += s_tot[0] + (TW > 1 ? s_tot[1] : 0u);
    __syncthreads();
  }
  if (tid == 0 && dev_status && (long long)carry > cap) *dev_status = 1;
  // pages of the last tile past the last token hold zeros (they may never have been written)
  const int pad0 = (N1 - 1) / kPage + 1, pad1 = (pad0 - 1) / kBoundsTilePages * kBoundsTilePages + kBoundsTilePages;
  for (int p = pad0 + wave; p < pad1; p += THREADS / 64)
    put_page_bounds<D>(tiles, p, bounds_u32x2{0u, 0u}, lane);

  // The rows that stay in the tail (n .. n_tail-1) move to its front, 16 bytes per work item.
  // Source and destination overlap, so the rows go in ascending chunks, each read completely
  // before any of it is written: a chunk's destination holds sources of this and of earlier
  // chunks only (the rows moved into the cache above have been read: barrier above).
  constexpr int U = 4;
  const int total = (n_tail - n) * PPT, shift = n * PPT;
  for (int base = 0; base < total; base += THREADS * U) {
    bounds_u32x4 kv[U], vv[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int e = base + j * THREADS + tid;
      if (e < total) kv[j] = Kt[e + shift], vv[j] = Vt[e + shift];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int e = base + j * THREADS + tid;
      if (e < total) Kt[e] = kv[j], Vt[e] = vv[j];
    }
    __syncthreads();
  }
}

int launch_flush_tail(const stc_shape_t& s, void* K_tail, void* V_tail, int n, int n_tail,
                      int tail_cap, int mode, const float* logits, const uint8_t* kcount,
                      int fixed_k, const uint16_t* mask_in, void* K, void* bounds, uint16_t* mask,
                      uint32_t* tok_off, void* vpacked, int32_t* dev_status, hipStream_t st) {
  const int streams = s.B * s.Hkv;
#define STC_FLUSH(DD, TILE, MOVERS)                                                             \
  flush_tail_kernel<DD, TILE, MOVERS><<<streams, flush_threads<TILE, MOVERS>(), 0, st>>>(       \
      (bounds_u32x4*)K_tail, (bounds_u32x4*)V_tail, (bounds_u32x4*)K, logits, kcount, n, s.N,   \
      token_cap(s), tail_cap, n_tail, mode, s.G, fixed_k, mask_in, (uint32_t*)bounds, mask,     \
      tok_off, (bounds_u32x4*)vpacked, dev_status, (long long)s.v_cap_groups)
  // few tokens of many streams by small workgroups (the table at the kernel)
  const bool many = (streams > 256 && n <= 64) || (streams >= 768 && (long long)n * s.D <= 64 * 128);
  if (s.D == 128) {
    if (many) STC_FLUSH(128, 32, 128);
    else STC_FLUSH(128, 128, 512);
  } else {
    if (many) STC_FLUSH(64, 32, 128);
    else STC_FLUSH(64, 128, 512);
  }
#undef STC_FLUSH
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
