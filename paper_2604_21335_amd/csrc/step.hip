// A whole decode step of one stream by one workgroup: page scores, selection and routed attention
// in one launch, for streams whose bounds and selected pages one workgroup gets through in the
// time that further launches cost.
#include "attention_block.hpp"
#include "score_tiles.hpp"

namespace stc {

// Bytes of shared memory in front of the selection's: query operands and page scores.
template <int D, int RM>
constexpr int step_score_lds() {
  return score_q_lds_bytes<D, RM>() + kStepKeys * 4;
}

// The three parts are those of the separate kernels and give the same bits: the scoring of
// score_tiles.hpp into LDS (and to `score`, where the caller finds the scores afterwards), the
// selection of topk_block.hpp from there, the attention of attention_block.hpp without splits.
// RM: query heads per KV head are at most this; `heads` = their number.
// Bound by memory while many workgroups are in different parts, by the chain of dependent
// accesses of one stream where there are few.
// At D = 64 two workgroups share a CU: 120 registers, 122 with a tail, nothing spilled (the bound of 128
// holds them to that, and the compiler stays below it without one).
template <int D, int RM, bool TAIL, bool STREAM>
__global__ __launch_bounds__(512, D == 64 ? 4 : 2) void step_kernel(
    const score_u32x4* __restrict__ tiles, float* __restrict__ score, const uint16_t* q,
    const uint16_t* K, const uint32_t* tok_off, int NP, int k_pages, int Ncap, int R,
    const AttnParams rest) {
  const AttnParams P = AttnFirst{q, K, rest.mask, tok_off, NP, k_pages, Ncap, R}.with(rest);
  const int tiles_cap = bounds_tiles(Ncap);
  constexpr int WAVES = 8, T16 = (D / 32) * 64;
  extern __shared__ __align__(16) unsigned char lds[];
  const int stream = blockIdx.x;
  const int heads = P.R;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  ScoreQuery<D, RM, 64 * WAVES> sq;
  sq.load(P.q + (size_t)stream * heads * D, heads);
  float* s_score = (float*)(lds + score_q_lds_bytes<D, RM>());
  const int ntiles = (P.NP + kBoundsTilePages - 1) / kBoundsTilePages;
  score_tile_range<D, RM, false, WAVES, kStepTilesAhead, STREAM>(
      tiles + (size_t)stream * tiles_cap * T16 + lane, s_score, P.NP, 0, ntiles, lds, wave, lane,
      [&] {
        sq.store(lds, heads);
        __syncthreads();
      },
      heads);
  __syncthreads();
  for (int i = threadIdx.x; i < P.NP; i += 64 * WAVES) score[(size_t)stream * P.NP + i] = s_score[i];
  attn_block<D, WAVES, TAIL, kStepKeys / (64 * WAVES), STREAM, true, 2>(
      P, stream, 0, lds, s_score, (TopkLds<kStepKeys / 512, 512>*)(lds + step_score_lds<D, RM>()));
}

template <int D, int RM, bool TAIL, bool STREAM>
static int step_go(const AttnParams& p, int streams, const void* bounds, float* score,
                   hipStream_t st) {
  constexpr int attn_lds = 8 * AttnCfg<D>::WAVE_LDS;
  constexpr int score_lds = step_score_lds<D, RM>() + (int)sizeof(TopkLds<kStepKeys / 512, 512>);
  constexpr int lds_bytes = attn_lds > score_lds ? attn_lds : score_lds;
  static std::atomic<uint64_t> allowed{0};
  if (!allow_dynamic_lds((const void*)step_kernel<D, RM, TAIL, STREAM>, lds_bytes, allowed))
    return -1;
  step_kernel<D, RM, TAIL, STREAM>
      <<<streams, 512, lds_bytes, st>>>((const score_u32x4*)bounds, score, p.q, p.K, p.tok_off, p.NP,
                                        p.k_pages, p.Ncap, p.R, p);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int D, int RM>
static int step_dispatch(const AttnParams& p, int streams, const void* bounds, float* score,
                         bool tail, bool stream_loads, hipStream_t st) {
  if (stream_loads)
    return tail ? step_go<D, RM, true, true>(p, streams, bounds, score, st)
                : step_go<D, RM, false, true>(p, streams, bounds, score, st);
  return tail ? step_go<D, RM, true, false>(p, streams, bounds, score, st)
              : step_go<D, RM, false, false>(p, streams, bounds, score, st);
}

template <int D>
static int step_dispatch_heads(const AttnParams& p, int streams, const void* bounds,
                               float* score, bool tail, bool stream_loads,
                               hipStream_t st) {
  const int R = p.R;
  if (R == 1) return step_dispatch<D, 1>(p, streams, bounds, score, tail, stream_loads, st);
  if (R == 2) return step_dispatch<D, 2>(p, streams, bounds, score, tail, stream_loads, st);
  if (R <= 4) return step_dispatch<D, 4>(p, streams, bounds, score, tail, stream_loads, st);
  if (R <= 8) return step_dispatch<D, 8>(p, streams, bounds, score, tail, stream_loads, st);
  return -1;
}

int launch_step_kernel(const AttnParams& p, int D, int streams, const void* bounds, float* score,
                       bool tail, bool stream_loads, hipStream_t st) {
  return D == 128
             ? step_dispatch_heads<128>(p, streams, bounds, score, tail, stream_loads, st)
             : step_dispatch_heads<64>(p, streams, bounds, score, tail, stream_loads, st);
}

}  // namespace stc
