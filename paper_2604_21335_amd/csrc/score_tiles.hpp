// Quest page scores of a range of bounds tiles by one workgroup (the arithmetic and the tile
// layout are described at the top of score.hip).  The query operands of the matrix-core
// products live in shared memory, one 64-bit operand per (head group, channel, lane), so that
// the registers of a wavefront hold only tile data and partial sums: the form with at most 128
// registers, i.e. four wavefronts per SIMD, also for more than four heads per KV head.
#pragma once
#include "stc_common.hpp"

namespace stc {

typedef __attribute__((ext_vector_type(4))) short score_bf16x4;
typedef __attribute__((ext_vector_type(4))) float score_f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t score_u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t score_u32x2;

// Bytes of shared memory for the query operands of one KV head's R query heads.
template <int D, int R>
__host__ __device__ constexpr int score_q_lds_bytes() {
  return ((R + 3) / 4) * (D / 8) * 64 * 8;
}

// The operand table of the first `heads` of R heads at `qs` ([R][D] bf16).  Entry (g, c, lane) is the A
// operand of lane `lane` for channel c of its chunk and head 4g + lane%4: the query value in
// the k-slot of the channel's minimum when it is negative, of its maximum otherwise, zeros in
// the three other slots (the channel pair of a B operand occupies two slots each).  All
// threads of the workgroup load and store it; the caller synchronises before the table is read.
// The loads go out in front of the tiles', so that the table is written while the tiles travel: behind
// them they would return last, since loads return in order.
template <int D, int R, int THREADS>
struct ScoreQuery {
  // one work item = 8 adjacent channels of one (head group, lane): a single 16-byte load
  static constexpr int CH = D / 8, NG = (R + 3) / 4, PIECES = CH / 8;  // 16-byte pieces per chunk
  static constexpr int ITEMS = NG * PIECES * 64, PER = (ITEMS + THREADS - 1) / THREADS;
  score_u32x4 v[PER];

  __device__ __forceinline__ void load(const uint16_t* __restrict__ qs, int heads) {
    static_for<0, PER>([&](auto n) {
      const int it = min((int)threadIdx.x + n * THREADS, ITEMS - 1);
      const int l = it & 63, piece = (it >> 6) % PIECES, g = it / (64 * PIECES);
      const int head = 4 * g + (l & 3), e = (l >> 2) & 7;
      v[n] = *(const score_u32x4*)(qs + min(head, heads - 1) * D + e * CH + piece * 8);
    });
  }

  __device__ __forceinline__ void store(unsigned char* qlds, int heads) const {
    static_for<0, PER>([&](auto n) {
      const int it = threadIdx.x + n * THREADS;
      const int l = it & 63, piece = (it >> 6) % PIECES, g = it / (64 * PIECES);
      if (ITEMS % THREADS != 0 && it >= ITEMS) return;
      const bool live = 4 * g + (l & 3) < heads;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w = live ? v[n][i] : 0u;
        const uint32_t lo = w & 0xffffu, hi = w >> 16;  // channels 2i and 2i+1 of the piece
        const uint32_t qa0 = (lo & 0x8000u) ? lo : lo << 16;
        const uint32_t qa1 = (hi & 0x8000u) ? hi : hi << 16;
        const int c = piece * 8 + 2 * i;
        *(score_u32x2*)(qlds + (size_t)((g * CH + c) * 64 + l) * 8) = score_u32x2{qa0, 0u};
        *(score_u32x2*)(qlds + (size_t)((g * CH + c + 1) * 64 + l) * 8) = score_u32x2{0u, qa1};
      }
    });
  }
};

// Scores tiles t0 + wave, t0 + wave + WAVES, ... < t1 of one stream.  `base` = the stream's
// tiles + lane; out = the stream's score row(s).  DEPTH tiles of the wavefront are requested
// ahead (DEPTH - 1 in flight behind the one being computed); STREAM: with loads that leave the
// caches alone.  `prologue` is run by every thread
// once the first tiles have been requested: it stores the operand table (ScoreQuery, whose loads the
// caller has made) and synchronises the workgroup.
// Heads from `heads` on count for nothing.
template <int D, int R, bool PER_HEAD, int WAVES, int DEPTH = 2, bool STREAM = false,
          class Prologue>
__device__ __forceinline__ void score_tile_range(const score_u32x4* __restrict__ base,
                                                 float* __restrict__ out, int NP, int t0, int t1,
                                                 const unsigned char* qlds, int wave, int lane,
                                                 Prologue prologue, int heads = R) {
  constexpr int CH = D / 8, NJ = CH / 4, NG = (R + 3) / 4, T16 = NJ * 64;
  const int tlast = t1 - 1;
  uint32_t qoff = lane * 8;
  auto load_tile = [&](score_u32x4 (&dst)[NJ], int tt) {
    const score_u32x4* pt = base + (size_t)min(tt, tlast) * T16;  // past the range: last tile again
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      dst[j] = STREAM ? __builtin_nontemporal_load(pt + j * 64) : pt[j * 64];
  };
  auto score_tile = [&](const score_u32x4 (&cur)[NJ], int tt) {
    float best = 0.f;
    // the operand table is read anew for every tile: an address the compiler cannot see through
    // keeps its loads inside the tile loop instead of pinning every operand in a register
    asm volatile("" : "+v"(qoff));
    const unsigned char* ql = qlds + qoff;
    const int page = tt * kBoundsTilePages + 4 * (lane >> 5) + (lane & 3);
    const bool writer = (lane & 0x1c) == kChunkSumLanes && page < NP;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const score_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      score_f32x4 u[NJ];  // per 16-byte unit: sum of its four channels, per head row
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const score_bf16x4 b01 = __builtin_bit_cast(score_bf16x4, score_u32x2{cur[j].x, cur[j].y});
        const score_bf16x4 b23 = __builtin_bit_cast(score_bf16x4, score_u32x2{cur[j].z, cur[j].w});
        score_f32x4 t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const score_bf16x4 a =
              *(const score_bf16x4*)(ql + (size_t)((g * CH + 4 * j + k) * 64) * 8);
          t[k] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, k < 2 ? b01 : b23, zero, 0, 0, 0);
        }
        u[j] = (t[0] + t[1]) + (t[2] + t[3]);
      }
#pragma unroll
      for (int w = 1; w < NJ; w *= 2)
#pragma unroll
        for (int j = 0; j < NJ; j += 2 * w) u[j] += u[j + w];
      const int rows = (R - 4 * g) < 4 ? (R - 4 * g) : 4;
#pragma unroll
      for (int i = 0; i < rows; ++i) {
        const float s = chunk_tree_sum(u[0][i]);
        if (PER_HEAD) {
          if (writer && 4 * g + i < heads)
            out[(size_t)(4 * g + i) * NP + page] = s == 0.f ? 0.f : s;
        } else if (4 * g + i < heads) {
          best = (g == 0 && i == 0) ? s : fmaxf(best, s);
        }
      }
    }
    if (!PER_HEAD && writer) out[page] = best == 0.f ? 0.f : best;
  };

  int t = t0 + wave;
  const bool any = t < t1;  // wave-uniform
  score_u32x4 d[DEPTH][NJ];
  __builtin_amdgcn_sched_barrier(0);  // behind the query loads
  if (any) static_for<0, DEPTH>([&](auto k) { load_tile(d[k], t + k * WAVES); });
  __builtin_amdgcn_sched_barrier(0);  // the tile requests go out before anything is waited for
  prologue();
  if (!any) return;
  for (; t < t1; t += DEPTH * WAVES) {
    static_for<0, DEPTH>([&](auto k) {
      if (k == 0 || t + k * WAVES < t1) {
        score_tile(d[k], t + k * WAVES);
        load_tile(d[k], t + (k + DEPTH) * WAVES);
      }
    });
  }
}

}  // namespace stc
