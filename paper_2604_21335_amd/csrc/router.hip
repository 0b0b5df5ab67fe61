// Value-group router (App. B.1): one linear projection from the layer-input hidden state of a
// token to its G group logits, logits[t, g] = sum_c h[t, c] * W[g, c] (+ bias[g]).
//
// The masks are integer decisions taken on these logits, so the float summation order is
// fixed: d_model is cut into chunks of 128 adjacent channels, a chunk is summed as a balanced
// tree over adjacent channels, and the chunk sums are accumulated left to right; the bias is
// added last.
//
// The products and the first level of the tree come from the matrix cores, exactly.
// v_mfma_f32_4x4x4_16b_bf16 multiplies, per block, a 4x4 A (rows = 4 groups, 4 k-slots) with a
// 4x4 B (k-slots, columns = 4 tokens).  A B register pair holds 4 adjacent channels of the
// lane's token as loaded; the A row holds the weight of ONE even channel in its slot and zeros
// in the other three, so every output is a single product of two bf16 values (exact in float)
// plus exact zeros, whatever rounding the unit applies to longer sums.
// v_mfma_f32_4x4x1_16b_f32 then adds the odd neighbour's product: it has one k-slot, takes float
// operands and rounds once, like fmaf (4 M random cases agree bit for bit, subnormal
// products among them), and the product of two bf16 values is exact, so what it rounds is
// the sum of the two products.  The other additions are ordinary float additions in the
// fixed order.  The float unit does not read subnormal operands as zero as the bf16 unit does,
// so they are replaced by zero on the way.
//
// Lane l of a wavefront: token 4*(l/32) + l%4 of a group of 8 tokens, channels
// 16*((l/4)%8) .. +16 of the current chunk (two 16-byte loads of h).  The 16 blocks of the MFMA
// are the 16 (token quad, 16-channel piece) pairs; the lane supplies the A row of group l%4
// (+4 per further MFMA group) for its block's channels.  Per (token, group) the 16 products of
// a lane are summed as a pair tree in the lane.  The 8 pieces are summed across lanes, several
// groups at a time: a level of that tree needs a result in only half of the lanes, so after
// each level two registers are merged into one.  In the end a lane carries the accumulator of
// its token and the group that lane bits 2, 3 (and 4) name.  A wavefront works on TG groups of
// 8 tokens per chunk, so the weights of a chunk are fetched and masked once for 8*TG tokens.
//
// Bound by memory and by the additions together.  Measured on 16 x 32768 tokens of 3584
// channels, 8 groups (3.77 GB): 760 us (5.0 TB/s; 683 on constant data, which draw less power) against 915 with all additions on the vector
// ALUs, a reduction of its own per group and half as many tokens per wavefront.  Streaming loads
// are slower here (834 against 749 in an earlier form): the two requests of a chunk take
// turns within each line.
//
// Inputs are zero or normal bf16 numbers (the matrix cores read subnormal bf16 inputs as
// zero), with products in the normal float range.
#include "stc_common.hpp"
#include "stc_kernels.hpp"

namespace stc {

typedef __attribute__((ext_vector_type(4))) short bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t router_u32x4;

__device__ __forceinline__ bf16x4 router_bf16x4(uint32_t w0, uint32_t w1) {
  return __builtin_bit_cast(bf16x4, (u32x2){w0, w1});
}

// TG groups of 8 tokens per wavefront.  SPLIT: the wavefronts of a workgroup work on the same
// tokens and take the chunks in turn, for launches of few tokens; their chunk sums meet in LDS and
// are accumulated there in the same order.
constexpr int kSplitWaves = 8;
constexpr int kSplitChunks = 64;  // chunk sums held in LDS at a time
template <int G, int TG, bool SPLIT>
struct RouterCfg {
  static constexpr int NH = (G + 3) / 4;        // MFMA row groups of 4 router outputs
  static constexpr int NA = (NH + 1) / 2;       // accumulators per lane and token group
  static constexpr int WAVES = SPLIT ? kSplitWaves : 4;
  static constexpr int WAVE_TOKENS = 8 * TG;
  static constexpr int BLOCK_TOKENS = (SPLIT ? 1 : WAVES) * WAVE_TOKENS;
  static_assert(!SPLIT || TG * NA <= kSplitWaves, "one wavefront per accumulator");
};

// The odd channel of a dword of two bf16 values as float, zero if it is subnormal (class bits:
// zeros and subnormals of either sign; the even channel below it makes a zero a subnormal).
__device__ __forceinline__ float odd_channel(uint32_t w) {
  const bool zero = __builtin_amdgcn_classf(__uint_as_float(w), 0xf0);
  return zero ? 0.f : bf16_hi(w);
}

// First two levels of the sum over the 4 lanes that share lane bits 0, 1, 4 and 5 (pieces
// (0,1)(2,3), then both) for the four router outputs v[0..3]: the lane with bit 2 set holds
// outputs 0 / 2, the other 1 / 3; bit 3 set: 0 / 1, clear: 2 / 3.  Of fewer than four outputs only
// the sums that the lanes of an output hold are taken.
template <int OUTPUTS>
__device__ __forceinline__ float fold_four(const float (&v)[4], bool bit2, bool bit3) {
  // (every sum is taken in all lanes: a lane cannot read from one that a branch switched off)
  const float s0 = v[0] + dpp_f32<0x124>(v[0]);  // row_ror:4, the piece before
  if constexpr (OUTPUTS == 1) return s0 + dpp_f32<0x128>(s0);
  const float s1 = v[1] + dpp_f32<0x12c>(v[1]);  // row_ror:12, the piece behind
  if constexpr (OUTPUTS == 2) {
    const float x = bit2 ? s0 : s1;
    return x + dpp_f32<0x128>(x);
  }
  const float s2 = v[2] + dpp_f32<0x124>(v[2]);
  const float s3 = v[3] + dpp_f32<0x12c>(v[3]);
  const float x01 = bit2 ? s0 : s1, x23 = bit2 ? s2 : s3;
  const float y01 = x01 + dpp_f32<0x128>(x01), y23 = x23 + dpp_f32<0x128>(x23);
  return bit3 ? y01 : y23;
}

template <int G, int TG, bool SPLIT>
__global__ __launch_bounds__((RouterCfg<G, TG, SPLIT>::WAVES * 64)) void router_logits_kernel(
                                                            const router_u32x4* __restrict__ h,
                                                            const router_u32x4* __restrict__ W,
                                                            const float* __restrict__ bias,
                                                            float* __restrict__ logits, int N,
                                                            int d_model, int Hkv,
                                                            int bias_stride) {
  using C = RouterCfg<G, TG, SPLIT>;
  constexpr int NH = C::NH, NA = C::NA;
  constexpr int STEP = SPLIT ? kSplitWaves : 1;
  __shared__ float s_sum[SPLIT ? kSplitChunks * TG * NA * 64 : 1];
  const int b = blockIdx.y;
  if (bias) bias += (size_t)b * bias_stride;  // 0: one bias for the batch; G: one per element
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 3, dp = (lane >> 2) & 7, tq = lane >> 5;
  const bool bit2 = lane & 4, bit3 = lane & 8;
  const int t_first = blockIdx.x * C::BLOCK_TOKENS + (SPLIT ? 0 : wave * C::WAVE_TOKENS) +
                      4 * tq + j;
  if constexpr (!SPLIT)  // a wavefront behind the last token (no barriers in this form)
    if (blockIdx.x * C::BLOCK_TOKENS + wave * C::WAVE_TOKENS >= N) return;
  const int nc = d_model / 128;
  const int row16 = d_model / 8;  // 16-byte pieces per row

  // rows past the end repeat the last token (never stored)
  const router_u32x4* hp[TG];
#pragma unroll
  for (int g8 = 0; g8 < TG; ++g8)
    hp[g8] = h + ((size_t)b * N + min(t_first + 8 * g8, N - 1)) * row16 + dp * 2;
  // the A rows this lane supplies: router output 4*hh + j (none beyond G: zeros)
  const router_u32x4* wp[NH];
#pragma unroll
  for (int hh = 0; hh < NH; ++hh) wp[hh] = W + (size_t)min(4 * hh + j, G - 1) * row16 + dp * 2;

  float acc[TG][NA];
#pragma unroll
  for (int g8 = 0; g8 < TG; ++g8)
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[g8][a] = 0.f;

  router_u32x4 hx[TG][2], wx[NH][2];
  const int c_first = SPLIT ? min(wave, nc - 1) : 0;
#pragma unroll
  for (int g8 = 0; g8 < TG; ++g8)
    hx[g8][0] = hp[g8][c_first * 16], hx[g8][1] = hp[g8][c_first * 16 + 1];
#pragma unroll
  for (int hh = 0; hh < NH; ++hh)
    wx[hh][0] = wp[hh][c_first * 16], wx[hh][1] = wp[hh][c_first * 16 + 1];

  for (int base = 0; base < nc; base += SPLIT ? kSplitChunks : nc) {
  const int cend = SPLIT ? min(base + kSplitChunks, nc) : nc;
  for (int c = base + (SPLIT ? wave : 0); c < cend; c += STEP) {
    // A operands of this chunk, per dword of two channels: the even channel's weight alone in
    // the low half, the odd channel's as float
    uint32_t we[NH][8];
    float wo[NH][8];
#pragma unroll
    for (int hh = 0; hh < NH; ++hh)
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const uint32_t w = (G % 4 == 0 || 4 * hh + j < G) ? wx[hh][d / 4][d % 4] : 0u;
        we[hh][d] = w & 0xffffu;
        wo[hh][d] = odd_channel(w);
      }
    router_u32x4 cur[TG][2];
#pragma unroll
    for (int g8 = 0; g8 < TG; ++g8) cur[g8][0] = hx[g8][0], cur[g8][1] = hx[g8][1];
    if (c + STEP < nc) {  // next chunk's requests go out before this chunk's arithmetic
#pragma unroll
      for (int g8 = 0; g8 < TG; ++g8)
        hx[g8][0] = hp[g8][(c + STEP) * 16], hx[g8][1] = hp[g8][(c + STEP) * 16 + 1];
#pragma unroll
      for (int hh = 0; hh < NH; ++hh)
        wx[hh][0] = wp[hh][(c + STEP) * 16], wx[hh][1] = wp[hh][(c + STEP) * 16 + 1];
    }
#pragma unroll
    for (int g8 = 0; g8 < TG; ++g8) {
      float ho[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) ho[d] = odd_channel(cur[g8][d / 4][d % 4]);
      float y[NH];
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) {
        // node[d][i] = sum over channels 2d, 2d+1 for router output 4*hh + i, then the next two
        // levels per 8 channels
        f32x4 half[2];
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          f32x4 node[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int d = 4 * q + k;
            const bf16x4 bb = router_bf16x4(cur[g8][q][k & ~1], cur[g8][q][k | 1]);
            const bf16x4 aa = (k & 1) ? router_bf16x4(0u, we[hh][d]) : router_bf16x4(we[hh][d], 0u);
            node[k] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(aa, bb, zero, 0, 0, 0);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
            node[k] = __builtin_amdgcn_mfma_f32_4x4x1f32(wo[hh][4 * q + k], ho[4 * q + k], node[k],
                                                         0, 0, 0);
          half[q] = (node[0] + node[1]) + (node[2] + node[3]);
        }
        const f32x4 s = half[0] + half[1];
        const float v[4] = {s[0], s[1], s[2], s[3]};
        y[hh] = fold_four<(G < 4 ? G : 4)>(v, bit2, bit3);
      }
      // pieces 0..3 and 4..7 sit in lanes with bit 4 clear and set: two row groups at a time
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const float ya = y[2 * a], yb = 2 * a + 1 < NH ? y[2 * a + 1] : y[2 * a];
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(ya), __float_as_uint(yb),
                                                        false, false);
        const float sum = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if constexpr (SPLIT) s_sum[((c - base) * TG * NA + g8 * NA + a) * 64 + lane] = sum;
        else acc[g8][a] += sum;
      }
    }
  }
  if constexpr (SPLIT) {  // wavefront i carries accumulator i
    __syncthreads();
    if (wave < TG * NA)
      for (int c = base; c < cend; ++c) acc[0][0] += s_sum[((c - base) * TG * NA + wave) * 64 + lane];
    __syncthreads();
  }
  }

  // accumulator a of a lane: router output 8*a + 4*(bit 4) + 2*(bit 3 clear) + (bit 2 clear)
  const int sub = (bit3 ? 0 : 2) + (bit2 ? 0 : 1);
  const int up = (lane >> 4) & 1;
  if (NH == 1 && up) return;  // both hold the same
  auto store = [&](float sum, int g8, int a) {
    const int g = 8 * a + 4 * up + sub, t = t_first + 8 * g8;
    if (g >= G || t >= N) return;
    const float v = sum + (bias ? bias[g] : 0.f);
    for (int kvh = 0; kvh < Hkv; ++kvh) logits[(((size_t)b * Hkv + kvh) * N + t) * G + g] = v;
  };
  if constexpr (SPLIT) {
    if (wave < TG * NA) store(acc[0][0], wave / NA, wave % NA);
  } else {
#pragma unroll
    for (int g8 = 0; g8 < TG; ++g8)
#pragma unroll
      for (int a = 0; a < NA; ++a) store(acc[g8][a], g8, a);
  }
}

// Tokens per wavefront and who shares them.  Measured, us, as split 8 / split 16 / own 16 / own 32:
//   channels tokens     4 groups                     8 groups                     16 groups
//   3584       1000    6.3/  8.1/ 21 / 34           8.1/ 11  / 28 / 51         12.2/ 16  / 51 / 88
//              6000   13.4/ 13.6/ 21 / 35          19.0/ 20.4/ 29 / 51         34  / 32  / 51 / 89
//             12000   23  / 19  / 21 / 34          34  / 29.8/ 29 / 51         65  / 47  / 51 / 89
//             24000   40  / 33  / 40 / 35          59  / 56  / 52 / 51        126  / 92  / 89 / 90
//             32768   56  / 45  / 42 / 38          83  / 78  / 55 / 54        170  /125  / 92 / 92
//        64 x   576   62  / 51  / 61 / 69          91  / 86  / 81 / 87        191  /140  /131 /152
//             65536  120  / 95  / 92 / 87         166  /158  /132 /100        336  /253  /193 /167
//            524288  883  /698  /676 /642        1218  /1202 /906 /790       2644  /1972 /1387/1220
//   1024       6000    5.5/  5.7/7.8/ 12           7.7/  8.8/ 10 / 17         14.2/ 12.7/ 17 / 29
//             12000    8.8/  7.7/8.4/ 12          13.5/ 12.6/ 11 / 17         26  / 18.5/ 18 / 29
//             24000   17  / 15  / 14 / 13          26  / 25  / 17 / 18         49  / 37  / 29 / 29
//    512      12000    7.8/  6.7/5.4/ 7.9         11.5/ 9.3/6.6/10.4           19  / 13.4/ 11 / 17
// Few tokens are bound by the chain of chunks of a wavefront, which the split form cuts to an eighth
// (the more chunks there are, the longer it wins); many by the weights' preparation per wavefront,
// which more tokens share.  The last form's wavefronts fill a SIMD each (64 x 576 tokens are a second
// round of an eighth).  A wavefront's tokens are of one batch element: elements of few tokens take the
// form that they fill (1024 channels, 8 groups, elements of 1 token: 32768 of them 201 / 408 / 232 /
// 545; of 13: 2048 of them 33 / 31 / 21 / 43; of 40: 3000 of them 116 / 132 / 72 / 117; of 65: 512 of
// them 37 / 39 / 38 / 27).
RouterForm router_form(int B, int N, int d_model, int G) {
  const long long tokens = (long long)B * N;
  const int chunks = d_model / 128;
  if (tokens < 3000 || N <= 8) return kSplit8;
  const int split_max = G <= 4 ? min(24000, 1600 * chunks)
                               : min(12000, 4000 + (G == 8 ? 600 : 1200) * chunks);
  if (tokens < split_max) return kSplit16;
  constexpr int kSimds = 1024;
  const long long waves = (long long)B * ((N + 31) / 32);  // of the last form
  const bool many = waves >= kSimds * 4 / 3;               // no short second round
  if (G <= 4) {
    if (N >= 64 && tokens >= 24000 && waves <= kSimds) return kOwn32;
    if (N >= 64 && chunks >= 16 && waves < kSimds * 7 / 4) return kSplit16;
  }
  return N >= 64 && many ? kOwn32 : kOwn16;
}

int launch_router_logits(const void* h, const void* W, const float* bias, int bias_stride,
                         float* logits, int B, int Hkv, int N, int d_model, int G,
                         hipStream_t st) {
#define STC_ROUTER_GO(GG, TG, SPLIT)                                                            \
  router_logits_kernel<GG, TG, SPLIT>                                                           \
      <<<dim3((N + RouterCfg<GG, TG, SPLIT>::BLOCK_TOKENS - 1) /                                \
                  RouterCfg<GG, TG, SPLIT>::BLOCK_TOKENS, B),                                   \
         RouterCfg<GG, TG, SPLIT>::WAVES * 64, 0, st>>>(                                        \
          (const router_u32x4*)h, (const router_u32x4*)W, bias, logits, N, d_model, Hkv,        \
          bias_stride)
  const RouterForm form = router_form(B, N, d_model, G);
#define STC_ROUTER_CASE(GG)                                                                     \
  case GG:                                                                                      \
    if (form == kSplit8) STC_ROUTER_GO(GG, 1, true);                                            \
    else if (form == kSplit16) STC_ROUTER_GO(GG, 2, true);                                      \
    else if (form == kOwn16) STC_ROUTER_GO(GG, 2, false);                                       \
    else STC_ROUTER_GO(GG, 4, false);                                                           \
    break;
  switch (G) {
    STC_ROUTER_CASE(1)
    STC_ROUTER_CASE(2)
    STC_ROUTER_CASE(4)
    STC_ROUTER_CASE(8)
    STC_ROUTER_CASE(16)
    default:
      return -1;
  }
#undef STC_ROUTER_CASE
#undef STC_ROUTER_GO
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace stc
