// GEMMs of the scheduled layer: the fused-QKV / output / FFN projections (paper section 2.2 step 1,
// appendix schedule) and the eight backward products, with the bias, bias+activation, activation
// derivative and residual-add epilogues applied to the fp32 accumulators in registers.
//
// bf16 path: 8 wavefronts in a 2x4 grid (or 2 x 2x2 with an in-block K split), each owning a block of
// v_mfma_f32_16x16x32_bf16 tiles. That form moves half the accumulator traffic per multiply of the 32x32x16 one, and
// under a load that is bound by power the chip holds a higher clock with it: a loop of nothing but MFMAs on random data
// runs at 2.12 PFLOP/s (2.1 GHz) against 1.87 (1.86 GHz) with the 32x32x16 form, at the same cycle count (another card 1.94
// / 1.73; on zeros or one repeated value, which draw less power, both run at 2.42-2.45).
// K slabs go global -> LDS by direct loads into a ring of LDS stages, one barrier per slab; a K that is no multiple of
// the slab ends in a zero-filled one. Operands whose contraction index is
// contiguous in memory are read from LDS with 16-byte reads; operands whose contraction index is the
// strided one (the "N" operand of dY*W and both operands of dY^T*X) stay in their memory order in LDS and
// are read with the transposing ds_read_b64_tr_b16, so no transposed copy of any tensor is ever made.
// fp32 path (the mode that checks the others): fp32 MFMAs, wavefronts that share a tile along K.
#include <stdio.h>
#include <stdlib.h>
#include <type_traits>

#include "common.h"
#include "gemm_tile.h"
#include "kernels.h"

namespace slapo {

template <int LAYOUT, int BM, int BN, int BK, int WGM, int WGN, int KS, int NS, int PW, bool KTAIL, int EPI,
          bool F16 = false, bool HYB = false>
__global__ __launch_bounds__((WGM * WGN * KS + PW) * 64, NS == 2 && PW ? 6 : 1)   // (two workgroups of twelve wavefronts per CU)
void gemm_bf16_kernel(int M, int N, int K, const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
                      const bf16_t* __restrict__ bias, const bf16_t* aux_in, bf16_t* __restrict__ aux_out, int act,
                      int tail_begin, int tail_splits, float* __restrict__ hyb_ws) {
  gemm_bf16_tile<LAYOUT, BM, BN, BK, WGM, WGN, KS, NS, PW, KTAIL, EPI, F16, HYB>(
      blockIdx.x, M, N, K, A, B, C, bias, aux_in, aux_out, act, tail_begin, tail_splits, hyb_ws);
}

// The whole rounds of a grid of 256x256 tiles, and the tiles of a thin last one in quarters (quarter_tiles): 128x128 tiles of the
// same eight wavefronts, 128-deep slabs in two stages (the bytes in flight of the large tile). The quarters of a tile go to one XCD.
template <int LAYOUT, bool KTAIL, int EPI, bool F16>
__global__ __launch_bounds__(512, 1) void gemm_bf16_quarters_kernel(int M, int N, int K, const bf16_t* __restrict__ A,
                                                                    const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
                                                                    const bf16_t* __restrict__ bias, const bf16_t* aux_in,
                                                                    bf16_t* __restrict__ aux_out, int act, int whole) {
  if ((int)blockIdx.x < whole) {
    gemm_bf16_tile<LAYOUT, 256, 256, 64, 2, 4, 1, 2, 0, KTAIL, EPI, F16>(blockIdx.x, M, N, K, A, B, C, bias, aux_in, aux_out, act, 0, 1, nullptr);
    return;
  }
  const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
  const int u = blockIdx.x - whole, tile = whole + (u >> 5) * 8 + (u & 7), quarter = (u >> 3) & 3;
  if (tile >= tiles_m * tiles_n) return;
  const TilePos pos = tile_position(tile, tiles_m, tiles_n, 1);
  const int m0 = pos.tile_m * 256 + (quarter >> 1) * 128, n0 = pos.tile_n * 256 + (quarter & 1) * 128;
  if (m0 >= M || n0 >= N) return;
  gemm_bf16_tile<LAYOUT, 128, 128, 128, 2, 4, 1, 2, 0, KTAIL, EPI, F16>(0, M, N, K, A, B, C, bias, aux_in, aux_out, act, 0, 1, nullptr, m0, n0);
}

template <int LAYOUT, int W>
__global__ __launch_bounds__(F32_WAVES * 64) void gemm_f32_kernel(int M, int N, int K, const float* __restrict__ A,
                                                                  const float* __restrict__ B, float* __restrict__ C,
                                                                  const float* __restrict__ bias, const float* aux_in,
                                                                  float* __restrict__ aux_out, int epi, int act) {
  __shared__ __attribute__((aligned(16))) float lds[f32_lds_floats(W)];
  gemm_f32_tile<LAYOUT, W>(blockIdx.x, lds, M, N, K, A, B, C, bias, aux_in, aux_out, epi, act);
}

// 64 tiles of 32x32 at 256 x 256 x 1024 take 10.3 us, 256 of 16x16 6.1; 75 tiles (77 x 776 x 520) 6.0 / 3.7; 192 tiles
// (256 x 768 x 256) 5.3 / 5.6; 1536 tiles 48 / 69.
static bool f32_wide(int M, int N) { return (int64_t)((M + 31) / 32) * ((N + 31) / 32) > 128; }

// epilogue / layout pairs the layer itself uses; the others exist as 128x128 tiles only
constexpr bool epi_used(int layout, int epi) {
  return layout == GEMM_NT ? (epi == EPI_NONE || epi == EPI_BIAS || epi == EPI_BIAS_ACT || epi == EPI_GATE || epi == EPI_ROPE)
       : layout == GEMM_NN ? (epi == EPI_NONE || epi == EPI_DACT || epi == EPI_ADD || epi == EPI_DGATE)
                           : (epi == EPI_NONE || epi == EPI_ADD);
}

template <int LAYOUT, int BM, int BN, int WGM, int WGN, int KS, int NS, int PW, bool F16, bool ALL_EPI = false, int BK = 64>
static void launch_bf16_tile(int epi, int act, int M, int N, int K, const void* A, const void* B, void* C,
                             const void* bias, const void* aux_in, void* aux_out, hipStream_t st) {
  const int tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const size_t lds = gemm_lds_bytes<BM, BN, BK, WGM, WGN, KS, NS>();
#define SLAPO_GEMM(E)                                                                                       \
  do {                                                                                                      \
    if constexpr ((ALL_EPI && E != EPI_ROPE) || epi_used(LAYOUT, E)) {                                                         \
      auto kern = LAYOUT == GEMM_TN || K % BK == 0 ? gemm_bf16_kernel<LAYOUT, BM, BN, BK, WGM, WGN, KS, NS, PW, false, E, F16> \
                                                   : gemm_bf16_kernel<LAYOUT, BM, BN, BK, WGM, WGN, KS, NS, PW, LAYOUT != GEMM_TN, E, F16>; \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);  \
      hipLaunchKernelGGL(kern, dim3(tiles), dim3((WGM * WGN * KS + PW) * 64), lds, st, M, N, K, (const bf16_t*)A,       \
                         (const bf16_t*)B, (bf16_t*)C, (const bf16_t*)bias, (const bf16_t*)aux_in,          \
                         (bf16_t*)aux_out, act, tiles, 1, (float*)nullptr);                                 \
    }                                                                                                       \
  } while (0)
  switch (epi) {
    case EPI_NONE: SLAPO_GEMM(EPI_NONE); break;
    case EPI_BIAS: SLAPO_GEMM(EPI_BIAS); break;
    case EPI_BIAS_ACT: SLAPO_GEMM(EPI_BIAS_ACT); break;
    case EPI_DACT: SLAPO_GEMM(EPI_DACT); break;
    case EPI_GATE: SLAPO_GEMM(EPI_GATE); break;
    case EPI_DGATE: SLAPO_GEMM(EPI_DGATE); break;
    case EPI_ROPE: SLAPO_GEMM(EPI_ROPE); break;
    default: SLAPO_GEMM(EPI_ADD); break;
  }
#undef SLAPO_GEMM
}

// Tile selection, from measurements on the layer's shapes. 256x256 tiles (8 wavefronts, 128x64 each, direct
// loads into two stages) when they still cover at least three quarters
// of the 256 CUs. Otherwise 128x128 tiles (8 wavefronts, 64x32 each; TN: two sets of four, 64x64 each): a ring of four
// stages filled by four loader wavefronts. 128x64 tiles of the same form (four computing wavefronts) where all of them
// fit one round, and 64x64 tiles with 128-deep slabs (layouts NT and NN, K of two such slabs or more) where the latter would
// leave half of the CUs idle:
// such a product is a chain of slabs whose bytes each CU has to fetch by itself, so more CUs and fewer bytes per CU shorten
// it. Forward of an encoder layer, 128x64 / 64x64, 64-deep slabs / 64x64, 128-deep: hidden 256, 1024 tokens 41.8 / 37.4 / 36.9
// us; 512, 512 48.9 / 43.2 / 42.4; 1024, 128 47.7 / 43.5 / 42.7; 2048, 128 68.7 / 62.0 / 60.9 (deeper rings, or eight
// computing wavefronts instead of four: nothing or 1-3 % more). K needs no particular multiple: TN products with K = 2286 tokens and 768 x 3072 outputs take 18.7 us
// (41.7 with the register-staged kernel that such K used to go to), K = 2000 and 10240 x 2560 take 107 us (170 before).
enum TileKind { TILE_256, TILE_128_SPLITSLAB, TILE_128_LOADERS, TILE_128x64_LOADERS, TILE_64_LOADERS, TILE_192x128_LOADERS, TILE_256x128_LOADERS,
                TILE_192x256, TILE_64x32_LOADERS, TILE_NONE };

// Products that one size of tile would finish in a round and a bit: the smallest tile that makes it exactly one round (one
// workgroup per CU). 192x128 and 256x128 as the 128x128 form (eight computing wavefronts, four loaders, three stages), 192x256 as the
// 256x256 form. Larger tiles read fewer bytes from LDS per MFMA, and nothing is left over; a slab of 192x128 takes 0.47 us against
// 0.37 of 128x128, of 192x256 0.95 against 1.15 of 256x256. us, the form taken before (128x128 tiles, in K ranges where a workspace allows,
// or two per CU) / one round:
//   192x128  2331 x 2048 x 768 13.9 / 11.5, x 2048 25.8 / 21.3, x 8192 82.7 / 66.5 (0.95 -> 1.18 PFLOP/s); 2000 x 2560 x 8192 81.1 / 69.9; NN
//            2000 x 2560 x 4096 52.4 / 40.0; with GeLU 2331 x 2048 x 2048 30.4 / 25.1
//   256x128  2048 x 4096 x 768 17.4 / 16.9 (with GeLU 21.2 / 21.1), x 4096 57.4 / 52.8; NN 3000 x 2560 x 2048 32.7 / 29.8, x 4096 58.4 / 51.7
//   192x256  3500 x 2560 x 768 24.3 / 18.1, x 2048 49.7 / 37.1, x 4096 78.7 / 67.1; NN 2048 x 5504 x 4096 93.4 / 72.9 (256x256 tiles 75.9)
// Steps: 2 x 1024 tokens of width 3072 1507 -> 1375 us, 3 x 777 of 2048 834 -> 769, 10 x 500 of 1024 613 -> 573, gated 2 x 1100 of 4096 2760 -> 2479.
// 192x256 loses to two 128x128 workgroups per CU where those are all resident (2600 x 3072 x 768 with GeLU: 504 tiles of 128x128, forward of
// the layer 91 / 95), and at K = 512 192x128 gains nothing (a gated layer's 2048 x 2736 x 512: forward 57.5 / 58.0). Layout TN has no
// such tiles: the chunk permutation of rows along M needs a power of two, and 256x128 ones have not been built for it.
static TileKind one_round_tile(int layout, int M, int N, int K) {
  auto count = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int64_t t128 = count(128, 128);
  if (layout == GEMM_TN || K < 768 || t128 <= 256) return TILE_NONE;
  if (count(192, 128) <= 256) return TILE_192x128_LOADERS;
  if (count(256, 128) <= 256) return TILE_256x128_LOADERS;
  return t128 > 512 && count(192, 256) <= 256 ? TILE_192x256 : TILE_NONE;
}
bool gemm_in_one_round(int dtype, int layout, int M, int N, int K) {
  return dtype != DT_FP32 && one_round_tile(layout, M, N, K) != TILE_NONE;
}

// 64x32 tiles (four stages of 128-deep slabs) where 64x64 ones take at most half of the CUs: three quarters of the bytes per CU and slab.
// Layout NT (rows of an operand that is not contiguous along K are 64 elements at least). us, 64x64 / 64x32, operands from memory:
//   128 x 3072 x 1024 5.78 / 5.08, 128 x 4096 x 1024 with GeLU 6.53 / 5.67, 128 x 2304 x 768 5.29 / 4.62, 256 x 2048 x 512 with GeLU 5.27 / 4.69;
//   more than 256 of them: 256 x 4096 x 1024 7.14 / 9.86, 128 x 6144 x 2048 12.2 / 16.6
// Products of at most 32 tiles of 64x64 keep those although 64x32 ones are faster there too (128 x 768 x 768 4.99 / 4.31): the layer and
// the exported product select alike, and the tests of the latter hold it to 64x64 tiles at these sizes.
static bool many_64x32(int M, int N) {
  const int64_t rows = (M + 63) / 64;
  return rows * ((N + 63) / 64) > 32 && rows * ((N + 31) / 32) <= 256;
}

static TileKind tile_by_count(int layout, int M, int N, int K, bool solo) {
  const int64_t t256 = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  // A grid of 256x256 tiles runs in rounds of 256 (one workgroup per CU) and a thin last round costs a full one:
  // 320 tiles take two rounds for 1.25 rounds of work. A GEMM that has the chip to itself (`solo`: the forward
  // pass, the exported building block) therefore takes 128x128 tiles when their round count is the cheaper one,
  // at the long-K rates that the two kernels had when the rule was measured (PFLOP/s: 1.30 for all three layouts against
  // 1.05 / 1.0 / 1.0; 256x256 tiles reach 1.51 now; one is four small ones). In the backward pass the idle CUs of a thin
  // round are exactly where the other stream's kernels run, and the same rule makes the step slower (2.7B-shaped layer:
  // 5.39 ms against 4.99 ms; on a single stream 5.06 against 5.62), so it is not applied there.
  bool big = t256 >= 192;
  if (solo && big && K >= 2048) {
    const double e256 = 1.30, e128 = layout == GEMM_NT ? 1.05 : 1.0;
    const double c256 = (double)((t256 + 255) / 256) * 4.0 / e256, c128 = (double)((t128 + 255) / 256) / e128;
    big = c256 <= c128;
  }
  if (big) return TILE_256;
  // TN: both operands go through the transposing LDS reads (two per fragment): the 64x64 wave tile of the
  // split-slab form needs a third fewer of them per MFMA, worth 2-7 % on the weight-gradient shapes from K = 2048 on; the
  // K-contiguous layouts gain nothing from it. Short K pays for the sum of its two wave sets instead: 1024 x 4096 outputs
  // at K = 128 6.8 / 6.0 us (split-slab / plain), 512 9.0 / 8.1, 1024 12.5 / 11.6, 2048 18.3 / 18.8.
  // Two rounds of 128x64 tiles are slower than one of 128x128 (768 x 3072 outputs, K = 2286: 26.8 against 18.7 us), one
  // round is faster (2304 x 768: 14.9 against 17.4).
  const int64_t t128x64 = (int64_t)((M + 127) / 128) * ((N + 63) / 64);
  if (t128x64 <= 256) {
    if (t128x64 > 128 || layout == GEMM_TN || K < 256) return TILE_128x64_LOADERS;
    return layout == GEMM_NT && many_64x32(M, N) ? TILE_64x32_LOADERS : TILE_64_LOADERS;
  }
  return layout == GEMM_TN && K > 1024 ? TILE_128_SPLITSLAB : TILE_128_LOADERS;
}

static TileKind select_tile(int layout, int M, int N, int K, bool solo) {
  const TileKind one = one_round_tile(layout, M, N, K);
  return one != TILE_NONE ? one : tile_by_count(layout, M, N, K, solo);
}

// Several rounds of 128x128 tiles: two LDS stages instead of four, so that two workgroups fit a CU and one's first loads and
// epilogue run beside the other's products. For K below 768, layout TN, and grids that no tile makes one round. Four / two stages, us:
// NT 3000 x 1536 x 512 12.8 / 11.0, with GeLU 18.3 / 15.4, 4096 x 2048 x 512 with GeLU 22.9 / 19.2, 640 x 12000 x 1024 with GeLU 29.0 / 24.7, x 4096
// 62.2 / 60.8; NN 3000 x 2048 x 512 with GeLU' 15.9 / 13.4, 640 x 12000 x 2048 37.8 / 34.9; TN 1536 x 4096 x 512 14.2 / 12.5, x 1024 20.4 / 19.1; more
// rounds gain less (NT 7000 x 1536 x 512 19.0 / 18.8).
static bool two_per_cu(int M, int N, int K) {
  const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  return t128 > 256 && (t128 <= 512 || K <= 3072);
}

// ---- thin last rounds: the tail tiles of a grid in several K ranges ----------------------------------
// 320 tiles on 256 CUs take two rounds for 1.25 rounds of work. With a workspace at hand, the tiles beyond the
// last full round are cut into s = 256 / (their number) K ranges, so that the last round has about 256 workgroups
// of 1/s the length, and a second kernel adds the ranges in order (bitwise reproducible) and applies the
// epilogue. Worth it when the saved (1 - 1/s) of a round outweighs writing and re-reading the partial tiles,
// i.e. for long K; plain and add epilogues only (the others have so many tiles that a thin round matters little).
// A grid with fewer tiles than half the CUs is all tail: 300 x 2048 outputs are 96 tiles of 128x64.
// Without / with, us: 8192 x 2560 x 10240 397 / 359 (whole tiles), 336 / 330 (quarters); 300 x 2048 x 8192 24.4 / 23.4. Three kinds of plan
// are older than what the product takes without a workspace now, and slower: 128x128 tiles where others make one round (2331 x 2048 x
// 8192 73 / 83; the layers pass no workspace there), few 128x64 tiles where 64x64 ones have 128-deep slabs (256 x 1024 x 4096 10.2 / 13.5)
// and where the reader adds ranges itself (product_in_ranges). Exported calls that bring a workspace get what they ask for.
struct HybridPlan { TileKind tile; int tail_begin, tail_tiles, splits; size_t ws_bytes; };
static HybridPlan hybrid_plan(int layout, int epi, int M, int N, int K) {
  HybridPlan none = {TILE_256, 0, 0, 1, 0}, p = none;
  static const bool disabled = debug_flag("no-hybrid");
  if (disabled || (epi != EPI_NONE && epi != EPI_ADD)) return none;
  p.tile = tile_by_count(layout, M, N, K, false);
  if (p.tile == TILE_64_LOADERS || p.tile == TILE_64x32_LOADERS) p.tile = TILE_128x64_LOADERS;   // (K ranges bring the workgroups that the smaller tiles would)
  if (layout == GEMM_TN && p.tile != TILE_256) return none;   // (K ranges of their own: weight_grad_splits)
  const int bm = p.tile == TILE_256 ? 256 : 128, bn = p.tile == TILE_256 ? 256 : p.tile == TILE_128x64_LOADERS ? 64 : 128;
  const int tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int rem = tiles % 256, nk = (K + 63) / 64;
  if (rem == 0 || (tiles < 256 && p.tile != TILE_128x64_LOADERS)) return none;
  int s = 256 / rem;
  s = s > 8 ? 8 : s;
  while (s > 1 && ((s - 1) * ((nk + s - 1) / s) >= nk || nk / s < 8)) --s;   // every range non-empty, at least 8 slabs
  if (s < 2) return none;
  // Time of a 64-deep slab of a round (256x256: a lower bound, the matrix cores' own time at 1.95 PFLOP/s; the kernel takes
  // 1.35 us), and the partial tiles written and read once at ~4 TB/s; the small tiles' rounds are short enough for the
  // second kernel's own 4 us to count.
  const double slab_us = p.tile == TILE_256 ? 1.1 : p.tile == TILE_128_LOADERS ? 0.37 : 0.2;
  const double saved_us = (1.0 - 1.0 / s) * nk * slab_us;
  const double cost_us = 2.0 * rem * s * bm * bn * 4.0 / 4.0e6;
  if (saved_us < 1.5 * cost_us + (p.tile == TILE_256 ? 0.0 : 4.0)) return none;
  p.tail_tiles = rem;
  p.tail_begin = tiles - rem;
  p.splits = s;
  p.ws_bytes = (size_t)rem * s * bm * bn * sizeof(float);
  return p;
}

// C tile of tail tile t = sum over the K ranges of hyb_ws[(t * splits + r)] (+ aux_in), eight columns per thread, the
// ranges four at a time so that their loads are in flight together.
template <int BM, int BN, bool F16>
__global__ __launch_bounds__(256) void hybrid_reduce_kernel(int M, int N, int tail_begin, int splits,
                                                            const float* __restrict__ ws, bf16_t* C,
                                                            const bf16_t* aux_in) {
  constexpr int CPT = BM * BN / 8;   // 8-column chunks per tile
  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM;
  const int q = blockIdx.x * 256 + threadIdx.x;
  const int t = q / CPT, in_tile = q - t * CPT;
  const TilePos pos = tile_position(tail_begin + t, tiles_m, tiles_n, 1);
  const int row = in_tile / (BN / 8), col = (in_tile % (BN / 8)) * 8;
  const int m = pos.tile_m * BM + row, n = pos.tile_n * BN + col;
  if (m >= M || n >= N) return;
  const float* part = ws + ((size_t)t * splits * BM + row) * BN + col;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r0 = 0; r0 < splits; r0 += 4) {
    float v[4][8];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r0 + r < splits) load8(part + (size_t)(r0 + r) * BM * BN, v[r]);   // (uniform)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r0 + r < splits) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += v[r][e];
      }
  }
  const int64_t idx = (int64_t)m * N + n;
  if (aux_in) {
    float v[8];
    load8h<F16>(aux_in + idx, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += v[e];
  }
  store8h<F16>(C + idx, acc);
}

template <int LAYOUT, int BM, int BN, int WGM, int WGN, int NS, int PW, bool F16>
static void launch_hybrid_tile(const HybridPlan& hp, int epi, int M, int N, int K, const void* A, const void* B, void* C,
                               const void* aux_in, float* ws, hipStream_t st) {
  const size_t lds = gemm_lds_bytes<BM, BN, 64, WGM, WGN, 1, NS>();
  const int grid = hp.tail_begin + hp.tail_tiles * hp.splits;
#define SLAPO_HYB(E)                                                                                           \
  do {                                                                                                         \
    auto kern = LAYOUT == GEMM_TN || K % 64 == 0 ? gemm_bf16_kernel<LAYOUT, BM, BN, 64, WGM, WGN, 1, NS, PW, false, E, F16, true> \
                                                 : gemm_bf16_kernel<LAYOUT, BM, BN, 64, WGM, WGN, 1, NS, PW, LAYOUT != GEMM_TN, E, F16, true>; \
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);       \
    hipLaunchKernelGGL(kern, dim3(grid), dim3((WGM * WGN + PW) * 64), lds, st, M, N, K, (const bf16_t*)A, (const bf16_t*)B, \
                       (bf16_t*)C, (const bf16_t*)nullptr, (const bf16_t*)aux_in, (bf16_t*)nullptr, 0,         \
                       hp.tail_begin, hp.splits, ws);                                                          \
  } while (0)
  if (epi == EPI_ADD) SLAPO_HYB(EPI_ADD); else SLAPO_HYB(EPI_NONE);
#undef SLAPO_HYB
  const int chunks = hp.tail_tiles * (BM * BN / 8);
  hipLaunchKernelGGL((hybrid_reduce_kernel<BM, BN, F16>), dim3(chunks / 256), dim3(256), 0, st, M, N, hp.tail_begin, hp.splits,
                     (const float*)ws, (bf16_t*)C, epi == EPI_ADD ? (const bf16_t*)aux_in : (const bf16_t*)nullptr);
}

template <int LAYOUT, bool F16>
static void launch_hybrid(const HybridPlan& hp, int epi, int M, int N, int K, const void* A, const void* B, void* C,
                          const void* aux_in, float* ws, hipStream_t st) {
  if constexpr (LAYOUT != GEMM_TN) {   // (TN plans are for 256x256 tiles only)
    if (hp.tile == TILE_128_LOADERS) {
      launch_hybrid_tile<LAYOUT, 128, 128, 2, 4, 4, 4, F16>(hp, epi, M, N, K, A, B, C, aux_in, ws, st);
      return;
    }
    if (hp.tile == TILE_128x64_LOADERS) {
      launch_hybrid_tile<LAYOUT, 128, 64, 2, 2, 4, 4, F16>(hp, epi, M, N, K, A, B, C, aux_in, ws, st);
      return;
    }
  }
  launch_hybrid_tile<LAYOUT, 256, 256, 2, 4, 2, 0, F16>(hp, epi, M, N, K, A, B, C, aux_in, ws, st);
}

// Thin last rounds without K ranges. A product that has the chip to itself runs the tiles of its whole rounds as 256x256 ones and
// cuts each tile beyond them into four 128x128 ones, in the same launch: up to half a round of tiles makes at most two rounds of
// quarters, which take a third of a round each. Every sum keeps its order, so the bits are those of whole tiles. us, the form
// taken before (two rounds, or 128x128 tiles from K = 2048 on) / quarters:
//   NT with GeLU  2331 x 8192 x 2560 (320 tiles) 113.4 / 95.2, x 1024 67.3 / 51.2, x 512 49.3 / 39.0; 4352 x 4096 x 2560 (272) 111.6 / 91.5;
//                 2600 x 8192 x 4096 (352) 183.3 / 166.6, x 2560 119.5 / 116.9; 3072 x 8192 x 1024 (384) 68.9 / 65.1
//   NT with bias  8192 x 2064 x 2560 (288) 100.6 / 77.8; 8192 x 2560 x 2560 (320) 107 / 84.7; 16384 x 1536 x 4096 (384) 174.6 / 159.5
// K ranges (hybrid_plan) come first where a workspace is at hand and K is long enough for them (8192 x 2560 x 10240: 328 us, quarters 315;
// beside its neighbours in a step level). Not on the two streams of backward, whose kernels fill a thin round from both sides:
// steps of whole rounds and thin ones / quarters there too, 4 x 1024 tokens of width 2560 2123 / 2165 us, 1 x 8192 backward 3377 / 3413.
// Steps with them in forward alone: 2 x 1000 tokens of width 2560, checkpointed 2988 -> 2866; 10 x 500 of 1024 606 -> 589; forward
// of 2 x 1024 of 3072 635 -> 572, of 3 x 777 of 2048 302 -> 293.
static int quarter_tiles(int layout, int M, int N, int K, bool solo) {
  const int64_t t256 = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  const int rem = (int)(t256 % 256);
  return solo && layout != GEMM_TN && t256 > 256 && rem > 0 && rem <= 128 && K >= 256 ? rem : 0;
}

template <int LAYOUT, bool F16>
static void launch_quarters(int rem, int epi, int act, int M, int N, int K, const void* A, const void* B, void* C,
                            const void* bias, const void* aux_in, void* aux_out, hipStream_t st) {
  const int whole = ((M + 255) / 256) * ((N + 255) / 256) - rem;
  constexpr size_t l0 = gemm_lds_bytes<256, 256, 64, 2, 4, 1, 2>(), l1 = gemm_lds_bytes<128, 128, 128, 2, 4, 1, 2>(), lds = l0 > l1 ? l0 : l1;
#define SLAPO_QUARTERS(E)                                                                                               \
  do {                                                                                                                  \
    if constexpr (epi_used(LAYOUT, E)) {                                                                                \
      auto kern = K % 128 == 0 ? gemm_bf16_quarters_kernel<LAYOUT, false, E, F16> : gemm_bf16_quarters_kernel<LAYOUT, true, E, F16>; \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);               \
      hipLaunchKernelGGL(kern, dim3(whole + (rem + 7) / 8 * 32), dim3(512), lds, st, M, N, K, (const bf16_t*)A, (const bf16_t*)B, \
                         (bf16_t*)C, (const bf16_t*)bias, (const bf16_t*)aux_in, (bf16_t*)aux_out, act, whole);         \
    }                                                                                                                   \
  } while (0)
  switch (epi) {
    case EPI_NONE: SLAPO_QUARTERS(EPI_NONE); break;
    case EPI_BIAS: SLAPO_QUARTERS(EPI_BIAS); break;
    case EPI_BIAS_ACT: SLAPO_QUARTERS(EPI_BIAS_ACT); break;
    case EPI_DACT: SLAPO_QUARTERS(EPI_DACT); break;
    case EPI_GATE: SLAPO_QUARTERS(EPI_GATE); break;
    case EPI_DGATE: SLAPO_QUARTERS(EPI_DGATE); break;
    case EPI_ROPE: SLAPO_QUARTERS(EPI_ROPE); break;
    default: SLAPO_QUARTERS(EPI_ADD); break;
  }
#undef SLAPO_QUARTERS
}

template <int LAYOUT, bool F16>
static void launch_bf16(int epi, int act, int M, int N, int K, const void* A, const void* B, void* C,
                        const void* bias, const void* aux_in, void* aux_out, hipStream_t st, bool solo, float* ws,
                        size_t ws_bytes) {
  if (ws) {
    // (with a workspace the thin last round in K ranges also beats the full grid of 128x128 tiles that a GEMM running
    // alone would otherwise take: 359 against 397 us for the 8192 x 2560 x 10240 NT product)
    const HybridPlan hp = hybrid_plan(LAYOUT, epi, M, N, K);
    if (hp.ws_bytes && hp.ws_bytes <= ws_bytes) {
      launch_hybrid<LAYOUT, F16>(hp, epi, M, N, K, A, B, C, aux_in, ws, st);
      return;
    }
  }
  if constexpr (LAYOUT != GEMM_TN) {
    const int rem = quarter_tiles(LAYOUT, M, N, K, solo);
    if (rem && epi_used(LAYOUT, epi)) {
      launch_quarters<LAYOUT, F16>(rem, epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      return;
    }
  }
  // (epilogues that the layer never pairs with this layout come as 128x128 tiles only)
  switch (epi_used(LAYOUT, epi) ? select_tile(LAYOUT, M, N, K, solo) : TILE_128_LOADERS) {
    case TILE_256:
      launch_bf16_tile<LAYOUT, 256, 256, 2, 4, 1, 2, 0, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_128_SPLITSLAB:
      if constexpr (LAYOUT == GEMM_TN) launch_bf16_tile<LAYOUT, 128, 128, 2, 2, 2, 4, 4, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_128_LOADERS:
      if (two_per_cu(M, N, K)) {
        launch_bf16_tile<LAYOUT, 128, 128, 2, 4, 1, 2, 4, F16, true>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
        break;
      }
      launch_bf16_tile<LAYOUT, 128, 128, 2, 4, 1, 4, 4, F16, true>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st); break;
    case TILE_128x64_LOADERS:
      launch_bf16_tile<LAYOUT, 128, 64, 2, 2, 1, 4, 4, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st); break;
    case TILE_192x128_LOADERS:
      if constexpr (LAYOUT != GEMM_TN) launch_bf16_tile<LAYOUT, 192, 128, 2, 4, 1, 3, 4, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_256x128_LOADERS:
      if constexpr (LAYOUT != GEMM_TN) launch_bf16_tile<LAYOUT, 256, 128, 2, 4, 1, 3, 4, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_192x256:
      if constexpr (LAYOUT != GEMM_TN) launch_bf16_tile<LAYOUT, 192, 256, 2, 4, 1, 2, 0, F16>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_NONE: break;
    case TILE_64x32_LOADERS:
      if constexpr (LAYOUT == GEMM_NT) launch_bf16_tile<LAYOUT, 64, 32, 2, 2, 1, 4, 4, F16, false, 128>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
    case TILE_64_LOADERS:
      if constexpr (LAYOUT != GEMM_TN) launch_bf16_tile<LAYOUT, 64, 64, 2, 2, 1, 3, 4, F16, false, 128>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st);
      break;
  }
}

// What the tiles of a product take spread over all CUs, as they are where the tiles of another stream fill the rounds: at the rates of
// each form (slabs of a 256x256 tile, 1.33 us), and what a tile takes besides its slabs, four such ones for the smaller forms.
double gemm_slabs_beside(int layout, int M, int N, int K) {
  const double nk = (K + 63) / 64;
  const auto tiles = [&](int bm, int bn) { return (double)((M + bm - 1) / bm) * ((N + bn - 1) / bn) / 256.0; };
  switch (select_tile(layout, M, N, K, false)) {
    case TILE_256: return tiles(256, 256) * (nk + TILE_SLABS);
    case TILE_192x256: return tiles(192, 256) * (0.70 * nk + TILE_SLABS);
    case TILE_256x128_LOADERS: return tiles(256, 128) * (0.46 * nk + 4);
    case TILE_192x128_LOADERS: return tiles(192, 128) * (0.36 * nk + 4);
    case TILE_128x64_LOADERS: return tiles(128, 64) * (0.16 * nk + 4);
    case TILE_64_LOADERS: return tiles(64, 64) * (0.13 * nk + 4);
    case TILE_128_LOADERS:
      if (two_per_cu(M, N, K)) return tiles(128, 128) * (0.55 * nk + 4) / 2;
      [[fallthrough]];
    default: return tiles(128, 128) * (0.29 * nk + 4);
  }
}

// Rates of the other tiles in slabs of a 256x256 one (1.33 us): their rules have the times.
int gemm_slabs(int layout, int M, int N, int K) {
  const int nk = (K + 63) / 64, t256 = ((M + 255) / 256) * ((N + 255) / 256), t128 = ((M + 127) / 128) * ((N + 127) / 128);
  const int rem = quarter_tiles(layout, M, N, K, true), rounds = t256 / 256;
  if (rem) return rounds * (nk + TILE_SLABS) + ((rem + 63) / 64) * (nk + TILE_SLABS) / 4 + nk / 10;
  switch (select_tile(layout, M, N, K, true)) {
    case TILE_256: return ((t256 + 255) / 256) * (nk + TILE_SLABS);
    case TILE_192x128_LOADERS: return nk * 36 / 100 + TILE_SLABS;
    case TILE_256x128_LOADERS: return nk * 46 / 100 + TILE_SLABS;
    case TILE_192x256: return nk * 70 / 100 + TILE_SLABS;
    default: return ((t128 + 255) / 256) * (nk * 29 / 100 + TILE_SLABS);
  }
}

// ---- weight gradients with few output tiles: several K ranges per tile ---------------------------------
// C = sum over the ranges of the fp32 partial products, added in range order (so the result does not depend on
// which workgroup finished first), + addend (may be C itself), eight columns per thread.
template <typename T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(int64_t chunks, int64_t mn, int splits,
                                                            const float* __restrict__ ws, T* C, const T* addend) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= chunks) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < splits; ++s) {
    float v[8];
    load8(ws + (int64_t)s * mn + i * 8, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += v[e];
  }
  if (addend) {
    float v[8];
    load8(addend + i * 8, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += v[e];
  }
  store8(C + i * 8, acc);
}

void launch_add_ranges(int dtype, int64_t mn, int ranges, const float* parts, const void* addend, void* out, hipStream_t st) {
  const int64_t chunks = mn / 8;
  const dim3 grid((unsigned)((chunks + 255) / 256));
  if (dtype == DT_FP16) hipLaunchKernelGGL(splitk_reduce_kernel<f16_t>, grid, dim3(256), 0, st, chunks, mn, ranges, parts, (f16_t*)out, (const f16_t*)addend);
  else hipLaunchKernelGGL(splitk_reduce_kernel<bf16_t>, grid, dim3(256), 0, st, chunks, mn, ranges, parts, (bf16_t*)out, (const bf16_t*)addend);
}

// Number of K ranges for a weight gradient: 1 (plain GEMM) unless the 128x128 tiles leave most of the chip idle
// and K is long; then as many as bring the grid to about one workgroup per CU, each range at least 48 slabs
// (measured: at M = N = 1024 four ranges take 41 us against 70 us at K = 16384, but 22.5 against 20.4 at K = 4096,
// where the second kernel and the partial tiles cost more than the idle CUs).
static int weight_grad_splits(int M, int N, int K) {
  static const bool disabled = debug_flag("no-splitk");   // A/B timing
  if (disabled || N % 8 != 0) return 1;
  const int64_t t128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  if (t128 >= 160) return 1;
  int64_t s = 256 / t128;
  const int64_t by_len = (K / 64) / 48;
  if (s > by_len) s = by_len;
  if (s > 8) s = 8;
  return s < 2 ? 1 : (int)s;
}

size_t gemm_ws_bytes(int dtype, int layout, int epi, int M, int N, int K) {
  return dtype == DT_FP32 ? 0 : hybrid_plan(layout, epi, M, N, K).ws_bytes;
}

size_t gemm_ws_least_bytes(int dtype, int layout, int epi, int M, int N, int K) {
  if (dtype == DT_FP32) return 0;
  const HybridPlan hp = hybrid_plan(layout, epi, M, N, K);
  return hp.tile == TILE_256 && K % 128 == 0 ? hp.ws_bytes : 0;
}

size_t weight_grad_ws_bytes(int dtype, int M, int N, int K) {
  if (dtype == DT_FP32) return 0;
  const int s = weight_grad_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * sizeof(float) : hybrid_plan(GEMM_TN, EPI_NONE, M, N, K).ws_bytes;   // (same for the add epilogue)
}

size_t weight_grad_ws_least_bytes(int dtype, int M, int N, int K) {
  if (weight_grad_splits(M, N, K) > 1) return K % 256 == 0 ? weight_grad_ws_bytes(dtype, M, N, K) : 0;
  return gemm_ws_least_bytes(dtype, GEMM_TN, EPI_NONE, M, N, K);
}

template <bool F16>
static void launch_splitk(int splits, int accumulate, int M, int N, int K, const void* A, const void* B, void* C,
                          float* ws, hipStream_t st) {
  constexpr int BM = 128, BN = 128;
  const int tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const size_t lds = gemm_lds_bytes<BM, BN, 64, 2, 2, 2, 4>();
  auto kern = gemm_bf16_kernel<GEMM_TN, BM, BN, 64, 2, 2, 2, 4, 4, false, EPI_SPLITK, F16>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(tiles * splits), dim3((2 * 2 * 2 + 4) * 64), lds, st, M, N, K, (const bf16_t*)A,
                     (const bf16_t*)B, (bf16_t*)C, (const bf16_t*)nullptr, (const bf16_t*)nullptr,
                     reinterpret_cast<bf16_t*>(ws), splits, tiles * splits, 1, (float*)nullptr);
  launch_add_ranges(F16 ? DT_FP16 : DT_BF16, (int64_t)M * N, splits, ws, accumulate ? C : nullptr, C, st);
}

// ---- products of few tokens: K ranges that the reader adds up -----------------------------------------
// A [T, hidden] product of few tokens is a handful of 64x64 tiles, each a chain of slabs that one workgroup fetches by itself
// at 40 of the 64 bytes per clock its CU can load (128 x 1024 x 4096: 32 tiles of 64 slabs, 13-17 us). Four ranges of K bring
// three more CUs per tile in, and the row kernel that reads the product adds them up on the way (rowwise.hip), so that no kernel
// and no pass is added. Only the input gradient of a post-LN layer, which no row kernel reads, pays a kernel for the sum (4 us).
// The line: the ranges cost the row kernel 1-2 us, and long chains of few tiles repay that; 64-tile products only from K = 6144
// on, more tiles or shorter K nowhere. us, forward / backward of an encoder layer, plain -> ranges:
//   inside   hidden 512, 128 tokens 36.7 -> 32.6 / 44.0 -> 40.5; 1024, 24 40.7 -> 36.6 / 57.4 -> 49.7, 128 43.9 -> 40.2 / 62.5 -> 55.3;
//            2048, 64 57.5 -> 53.1 / 113.9 -> 93.4, 128 60.6 -> 57.0 / 117.2 -> 104.6; decoder 4096, 64 backward 263 -> 252
//   outside  hidden 256, 1024 34.5 -> 36.4 / 48.6 -> 55.8; 512, 512 37.2 -> 37.9 / 52.5 -> 58.6; 1024, 256 45.5 -> 44.1 / 66.8 -> 67.9, 512
//            51.7 -> 51.0 / 79.1 -> 83.6; 2048, 256 69.2 -> 68.9 / 126.9 -> 130.3; 4096, 128 168.6 -> 168.8 / 303.0 -> 310.6
// (Up to eight ranges: the same within 2 %, the row kernels spill. 16 slabs or more: none of four ranges is empty.)
bool product_in_ranges(int dtype, int M, int N, int K) {
  if (dtype == DT_FP32 || N < RANGES_MIN_N || N > RANGES_MAX_N) return false;
  const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
  return (tiles <= 32 && K >= 2048) || (tiles <= 64 && K >= 6144);
}

template <int LAYOUT, int BN, int NS, bool F16>
static void launch_ranges_tile(int M, int N, int K, const void* A, const void* B, float* parts, hipStream_t st) {
  constexpr int BK = 128;
  const int tiles = ((M + 63) / 64) * ((N + BN - 1) / BN);
  const size_t lds = gemm_lds_bytes<64, BN, BK, 2, 2, 1, NS>();
  auto kern = K % BK == 0 ? gemm_bf16_kernel<LAYOUT, 64, BN, BK, 2, 2, 1, NS, 4, false, EPI_SPLITK, F16>
                          : gemm_bf16_kernel<LAYOUT, 64, BN, BK, 2, 2, 1, NS, 4, true, EPI_SPLITK, F16>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(tiles * K_RANGES), dim3((2 * 2 + 4) * 64), lds, st, M, N, K, (const bf16_t*)A, (const bf16_t*)B,
                     (bf16_t*)nullptr, (const bf16_t*)nullptr, (const bf16_t*)nullptr, reinterpret_cast<bf16_t*>(parts), K_RANGES,
                     tiles * K_RANGES, 1, (float*)nullptr);
}

// (64x32 tiles in layout NT where all ranges of them fit one round, as for whole products)
template <int LAYOUT, bool F16>
static void launch_ranges(int M, int N, int K, const void* A, const void* B, float* parts, hipStream_t st) {
  if constexpr (LAYOUT == GEMM_NT) {
    if (((M + 63) / 64) * ((N + 31) / 32) * K_RANGES <= 256) {
      launch_ranges_tile<LAYOUT, 32, 4, F16>(M, N, K, A, B, parts, st);
      return;
    }
  }
  launch_ranges_tile<LAYOUT, 64, 3, F16>(M, N, K, A, B, parts, st);
}

void launch_gemm_ranges(int dtype, int layout, int M, int N, int K, const void* A, const void* B, float* parts, hipStream_t st) {
#define SLAPO_RANGES(L)                                                         \
  do {                                                                          \
    if (dtype == DT_FP16) launch_ranges<L, true>(M, N, K, A, B, parts, st);     \
    else launch_ranges<L, false>(M, N, K, A, B, parts, st);                     \
  } while (0)
  if (layout == GEMM_NT) SLAPO_RANGES(GEMM_NT); else SLAPO_RANGES(GEMM_NN);
#undef SLAPO_RANGES
}

void launch_weight_grad(int dtype, int accumulate, int M, int N, int K, const void* A, const void* B, void* C,
                        float* ws, hipStream_t st, bool solo) {
  const int splits = (ws && dtype != DT_FP32) ? weight_grad_splits(M, N, K) : 1;
  if (splits == 1) {
    launch_gemm(dtype, GEMM_TN, accumulate ? EPI_ADD : EPI_NONE, 0, M, N, K, A, B, C, nullptr, accumulate ? C : nullptr,
                nullptr, st, solo, ws, ws ? weight_grad_ws_bytes(dtype, M, N, K) : 0);
    return;
  }
  if (dtype == DT_FP16) launch_splitk<true>(splits, accumulate, M, N, K, A, B, C, ws, st);
  else launch_splitk<false>(splits, accumulate, M, N, K, A, B, C, ws, st);
}

// The kernel instance a GEMM of this shape runs as, in the spelling of the kernel's template arguments
// (layout, BM, BN, BK, WGM, WGN, KS, NS, PW, KTAIL, epilogue, F16, HYB), as the profiler prints the symbol; for
// the weight-gradient path (`weight_grad`) with its K ranges, if any.
void describe_gemm(int dtype, int layout, int epi, int M, int N, int K, bool solo, bool weight_grad, bool with_ws,
                   char* buf, size_t len) {
  if (dtype == DT_FP32) { snprintf(buf, len, "gemm_f32_kernel<%d, %d>", layout, f32_wide(M, N) ? 2 : 1); return; }
  const int f16 = dtype == DT_FP16 ? 1 : 0;
  const char* b = f16 ? "true" : "false";
  const char* kt = layout != GEMM_TN && K % 64 != 0 ? "true" : "false";
  static const char* const shape[] = {"256, 256, 64, 2, 4, 1, 2, 0", "128, 128, 64, 2, 2, 2, 4, 4", "128, 128, 64, 2, 4, 1, 4, 4",
                                      "128, 64, 64, 2, 2, 1, 4, 4", "64, 64, 128, 2, 2, 1, 3, 4", "192, 128, 64, 2, 4, 1, 3, 4",
                                      "256, 128, 64, 2, 4, 1, 3, 4", "192, 256, 64, 2, 4, 1, 2, 0", "64, 32, 128, 2, 2, 1, 4, 4"};
  if (with_ws && !(weight_grad && weight_grad_splits(M, N, K) > 1)) {
    const HybridPlan hp = hybrid_plan(layout, weight_grad ? EPI_NONE : epi, M, N, K);
    if (hp.ws_bytes) {
      snprintf(buf, len, "gemm_bf16_kernel<%d, %s, %s, %d, %s, true> (%d tiles + %d tiles in %d K ranges) + hybrid_reduce_kernel",
               layout, shape[(int)hp.tile], kt, epi, b, hp.tail_begin, hp.tail_tiles, hp.splits);
      return;
    }
  }
  if (weight_grad) {
    const int splits = weight_grad_splits(M, N, K);
    if (splits > 1) {
      snprintf(buf, len, "gemm_bf16_kernel<2, 128, 128, 64, 2, 2, 2, 4, 4, false, %d, %s, false> in %d K ranges + splitk_reduce_kernel", EPI_SPLITK, b, splits);
      return;
    }
  }
  if (const int rem = quarter_tiles(layout, M, N, K, solo); rem && epi_used(layout, epi)) {
    snprintf(buf, len, "gemm_bf16_quarters_kernel<%d, %s, %d, %s>", layout, K % 128 != 0 ? "true" : "false", epi, b);
    return;
  }
  const TileKind k = epi_used(layout, epi) ? select_tile(layout, M, N, K, solo) : TILE_128_LOADERS;
  if (k == TILE_128_LOADERS && two_per_cu(M, N, K)) {
    snprintf(buf, len, "gemm_bf16_kernel<%d, 128, 128, 64, 2, 4, 1, 2, 4, %s, %d, %s, false>", layout, kt, epi, b);
    return;
  }
  if (k == TILE_64_LOADERS || k == TILE_64x32_LOADERS) kt = K % 128 != 0 ? "true" : "false";
  snprintf(buf, len, "gemm_bf16_kernel<%d, %s, %s, %d, %s, false>", layout, shape[(int)k], kt, epi, b);
}

void launch_gemm(int dtype, int layout, int epi, int act, int M, int N, int K, const void* A, const void* B,
                 void* C, const void* bias, const void* aux_in, void* aux_out, hipStream_t st, bool solo, float* ws,
                 size_t ws_bytes) {
  if (dtype == DT_FP32) {
    const bool wide = f32_wide(M, N);
    const int tile = wide ? 32 : 16;
    const dim3 grid((unsigned)(((M + tile - 1) / tile) * ((N + tile - 1) / tile)));
#define SLAPO_F32W(L, W)                                                                                  \
  hipLaunchKernelGGL((gemm_f32_kernel<L, W>), grid, dim3(F32_WAVES * 64), 0, st, M, N, K, (const float*)A, (const float*)B, \
                     (float*)C, (const float*)bias, (const float*)aux_in, (float*)aux_out, epi, act)
#define SLAPO_F32(L) do { if (wide) SLAPO_F32W(L, 2); else SLAPO_F32W(L, 1); } while (0)
    if (layout == GEMM_NT) SLAPO_F32(GEMM_NT);
    else if (layout == GEMM_NN) SLAPO_F32(GEMM_NN);
    else SLAPO_F32(GEMM_TN);
#undef SLAPO_F32
#undef SLAPO_F32W
    return;
  }
#define SLAPO_H(F)                                                                                          \
  if (layout == GEMM_NT) launch_bf16<GEMM_NT, F>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st, solo, ws, ws_bytes);     \
  else if (layout == GEMM_NN) launch_bf16<GEMM_NN, F>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st, solo, ws, ws_bytes); \
  else launch_bf16<GEMM_TN, F>(epi, act, M, N, K, A, B, C, bias, aux_in, aux_out, st, solo, ws, ws_bytes)
  if (dtype == DT_FP16) { SLAPO_H(true); } else { SLAPO_H(false); }
#undef SLAPO_H
}

}  // namespace slapo
