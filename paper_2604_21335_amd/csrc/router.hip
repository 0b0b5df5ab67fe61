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
//   3584       4096   10.7/  9.4/ 22 / 35          14.5/ 12.2/ 29 / 51         25.1/ 18.9/ 52 / 90
//             12000   24  / 20  / 22 / 35          35  / 31  / 30 / 51         67  / 49  / 52 / 90
//             20000   36  / 29  / 40 / 35          53  / 49  / 52 / 51        109  / 78  / 88 / 90
//             32768   56  / 45  / 42 / 38          81  / 78  / 55 / 55        171  /124  / 92 / 93
//             40000   69  / 57  / 64 / 71         103  / 98  / 82 / 88        212  /160  /132 /154
//             65536  118  / 92  / 92 / 87         164  /159  /134 / 99        340  /254  /184 /161
//            524288  883  /698  /676 /642        1218  /1202 /906 /790       2644  /1972 /1387/1220
//   1024       4096    5.1/  4.9/8.4/ 13           6.3/  6.0/ 11 / 18         10.6/  7.9/ 18 / 29
//              8000    7.1/  6.3/8.8/ 13          10.1/  9.7/ 11 / 18         19.0/ 13.7/ 18 / 29
//             16384   12.4/ 10.4/9.2/ 13          18.3/ 17.4/ 12 / 18           35  / 26  / 19 / 30
//             40000   25  / 23  / 20 / 23          42  / 40  / 27 / 29          82  / 60  / 44 / 50
//         500 x  40   14.7/ 14.7/ 12 / 17          23  / 25  / 16 / 26          42  / 37  / 29 / 45
//        5000 x   1   18.9/ 29  / 24 / 36          31  / 63  / 33 / 60          76  /103  / 63 /104
// The time goes in rounds of one workgroup to a CU (a wavefront that has its workgroup for itself: to
// a SIMD).  Of the first round the split forms see next to nothing, being bound by latency there: the
// chain of chunks of a wavefront is an eighth of the other two forms'.  Later rounds cost the chunks
// times a constant of form and groups, which falls with the tokens that share a preparation of the
// weights.  The switch is where these lines cross: over 792 sizes (700 to 140000 tokens in elements of
// 1 to 98304, 256 to 8192 channels, 1 to 16 groups) the form taken is 1 % above the best in the mean,
// and 10 % and more above it in 19.
RouterForm router_form(int B, int N, int d_model, int G) {
  // per round and chunk: G <= 4, 8, 16
  static constexpr int kCost[4][3] = {{58, 90, 183}, {94, 188, 307}, {55, 72, 138}, {98, 132, 235}};
  const int chunks = d_model / 128, groups = G <= 4 ? 0 : G == 8 ? 1 : 2;
  auto blocks = [&](int tokens) { return (long long)B * ((N + tokens - 1) / tokens); };
  auto rounds = [](long long n, int at_once) { return (n + at_once - 1) / at_once; };
  auto split = [&](RouterForm f, int tokens) {
    return 10 * (max(chunks, 8) + 10) * kCost[f][groups] * (rounds(blocks(tokens), 256) - 1);
  };
  auto own = [&](RouterForm f, int tokens, int tenths) {
    const long long n = N <= tokens ? rounds(B, 1024) : rounds(blocks(4 * tokens), 256);
    return 8 * (chunks + 3) * kCost[f][groups] * (10 * n - tenths);
  };
  RouterForm form = kSplit8;
  long long cost = split(kSplit8, 8);
  auto take = [&](RouterForm f, long long c) {
    if (c < cost) form = f, cost = c;
  };
  take(kSplit16, split(kSplit16, 16));
  take(kOwn16, own(kOwn16, 16, 3));
  // (few groups of long rows are bound by the reads: 64 chunks of 4 groups, 131072 tokens: 477 / 392 /
  // 437 / 493)
  if (G > 4 || chunks <= 32) take(kOwn32, own(kOwn32, 32, 0));
  return form;
}

int launch_router_logits(const void* h, const void* W, const float* bias, int bias_stride,
                         float* logits, int B, int Hkv, int N, int d_model, int G,
                         hipStream_t st) {
  // a batch element of fewer tokens than a workgroup's has no wavefronts behind its last token
  auto waves = [&](int tokens) { return min(4, (N + tokens - 1) / tokens); };
#define STC_ROUTER_GO(GG, TG, SPLIT)                                                            \
  router_logits_kernel<GG, TG, SPLIT>                                                           \
      <<<dim3((N + RouterCfg<GG, TG, SPLIT>::BLOCK_TOKENS - 1) /                                \
                  RouterCfg<GG, TG, SPLIT>::BLOCK_TOKENS, B),                                   \
         (SPLIT ? kSplitWaves : waves(RouterCfg<GG, TG, SPLIT>::WAVE_TOKENS)) * 64, 0, st>>>(  \
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
