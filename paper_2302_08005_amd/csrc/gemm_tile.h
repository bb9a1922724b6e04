// The product of one output tile, as device functions: main loops, LDS layouts and epilogues of the GEMM kernels
// (gemm.hip), which also run inside the launches that hold several products (grads.hip).
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace slapo {

enum { ACT_GELU = 0, ACT_RELU = 1 };
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float act_fwd(float u, int act) {
  if (act == ACT_RELU) return u > 0.f ? u : 0.f;
  return 0.5f * u * (1.f + erff(u * 0.70710678118654752f));
}
__device__ __forceinline__ float act_grad(float u, int act) {
  if (act == ACT_RELU) return u > 0.f ? 1.f : 0.f;
  const float cdf = 0.5f * (1.f + erff(u * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * __expf(-0.5f * u * u);
  return cdf + u * pdf;
}

// GeLU for the bf16 epilogues. Phi(u) = 0.5 (1 + erf(u / sqrt 2)) with the erf of Abramowitz & Stegun 7.1.26
// (|error| <= 1.5e-7, far below one bf16 rounding): for x >= 0, erf(x) = 1 - t (a1 + t (a2 + ... a5 t)) exp(-x^2),
// t = 1 / (1 + 0.3275911 x). Written for h = 0.5 * poly * exp(-u^2/2): Phi(-|u|) = h, Phi(|u|) = 1 - h, so the
// negative tail has no cancellation. One exp2, one reciprocal and a dozen FMAs, about half the cost of erff.
struct GeluTerms { float phi, e; };   // Phi(u) and exp(-u^2 / 2)
__device__ __forceinline__ GeluTerms gelu_terms(float u) {
  const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(u), 0.3275911f * 0.70710678118654752f, 1.0f));
  const float e = __builtin_amdgcn_exp2f(u * u * (-0.5f * 1.4426950408889634f));
  float p = fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);
  p = fmaf(t, p, 0.5f * 1.421413741f);
  p = fmaf(t, p, 0.5f * -0.284496736f);
  p = fmaf(t, p, 0.5f * 0.254829592f);
  const float h = p * t * e;
  GeluTerms g;
  g.phi = u < 0.f ? h : 1.0f - h;
  g.e = e;
  return g;
}

template <typename T>
__device__ __forceinline__ void epilogue_store(int epi, int act, float acc, int64_t m, int64_t n, int64_t ldc,
                                               T* __restrict__ C, const T* __restrict__ bias,
                                               const T* aux_in, T* __restrict__ aux_out) {
  const int64_t idx = m * ldc + n;
  float v = acc;
  if (epi == EPI_BIAS) {
    v += to_f32(bias[n]);
  } else if (epi == EPI_BIAS_ACT) {
    v += to_f32(bias[n]);
    if (aux_out) from_f32(aux_out[idx], act_grad(v, act));   // all that backward needs of the pre-activation
    v = act_fwd(v, act);
  } else if (epi == EPI_DACT) {
    const float u = to_f32(aux_in[idx]);
    v = act == ACT_RELU ? (u > 0.f ? v : 0.f) : v * u;
  } else if (epi == EPI_ADD) {
    v += to_f32(aux_in[idx]);
  }
  from_f32(C[idx], v);
}

// Turns PAIRS adjacent pairs of row m, from column n of the packed queries and keys on, by the angles of the row's position
// (act = rope_act: sequence length and head width 64 or 128).
template <int PAIRS, int N>
__device__ __forceinline__ void rope_turn(float (&v)[N], const float* __restrict__ table, int act, int m, int n) {
  const int seq = act >> 1, half = act & 1 ? 64 : 32;
  const float* t = table + ((int64_t)(m % seq) * half + ((n & (2 * half - 1)) >> 1)) * 2;
#pragma unroll
  for (int e = 0; e < PAIRS; e += 2) {
    const float4 w = *reinterpret_cast<const float4*>(t + 2 * e);   // cos, sin of two pairs
    turn_pair(v[2 * e], v[2 * e + 1], w.x, w.y);
    turn_pair(v[2 * e + 2], v[2 * e + 3], w.z, w.w);
  }
}

// silu(u) = u * sigmoid(u) and the two factors the gated feed-forward block keeps for backward
struct GateTerms { float out, dgate, dup; };   // silu(u) * w, w * silu'(u), silu(u)
template <bool FAST>
__device__ __forceinline__ GateTerms gate_terms(float u, float w) {
  const float sg = FAST ? __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u * -1.4426950408889634f))
                        : 1.0f / (1.0f + expf(-u));
  const float s = u * sg;
  GateTerms g;
  g.out = s * w;
  g.dgate = w * (sg + s * (1.0f - sg));   // silu'(u) = sigmoid(u) (1 + u (1 - sigmoid(u)))
  g.dup = s;
  return g;
}

// Sum over the lanes whose number is the same modulo EVERY (4, 8 or 16), in all of them.
template <int EVERY>
__device__ __forceinline__ float sum_of_lanes(float x) {
  auto rotated = [](float v, auto by) {   // within 16 lanes
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + decltype(by)::value, 0xf, 0xf, false));
  };
  if constexpr (EVERY <= 4) x += rotated(x, std::integral_constant<int, 4>{});
  if constexpr (EVERY <= 8) x += rotated(x, std::integral_constant<int, 8>{});
  const unsigned a = __builtin_bit_cast(unsigned, x);
  const auto p = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const unsigned b = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return __builtin_bit_cast(float, (unsigned)q[0]) + __builtin_bit_cast(float, (unsigned)q[1]);
}

// LDS layouts. Every tile sits in LDS unpadded and in memory order, 16 bytes of thread t of a slab at byte
// 16 t of the stage, as the direct global -> LDS loads of gfx950 write it (one wave-level load fills 1 KB of
// consecutive LDS, lane l at byte 16 l).
// Bank conflicts are avoided by permuting, inside each tile row, which 16-byte chunk of global memory a
// thread fetches. The LDS has 64 banks of 4 B: 16 lanes of a 16-byte access, and 32 lanes of a transposing
// 8-byte read, are checked against each other for conflicts. Measured peak rates per CU with conflict-free
// addresses and 8 or 16 wavefronts: 16-byte reads 257 B per clock, plain 8-byte reads 164, transposing
// 8-byte reads 120 (about the same instruction rate as the 16-byte read, half the bytes).
//  - K-contiguous tile [rows][BK]: position p of row r holds chunk p ^ swzK(r), swzK(r) = (r / RP) % (BK/8),
//    RP = rows per 256 B (2 at a depth of 64, 1 at 128). A fragment read (one chunk of 16 consecutive rows) then lands in 16 different
//    16-byte bank groups. swzK depends on the lane only (wave tiles start at multiples of 32 rows), so a
//    fragment address is a per-lane base plus (2*ks ^ per-lane constant).
//  - M-contiguous tile [BK][W]: position p of k-row r holds chunk p ^ (swzM(r) << 1), i.e. 32-byte granules
//    are permuted by swzM(r) (defined in the kernel). A transposing 8-byte read is served 32 lanes at a time:
//    one granule of four consecutive k-rows and of the four that lie 8 further, whose 8 pieces the permutation
//    spreads over the 8 bank groups.
//  The conflict counter reads 1-4 % of the LDS cycles in all three layouts (6 % where K = 1024 leaves the epilogue's
//  staging a larger share).
//
// Why direct loads: a ds_write moves 64 B per clock and keeps the LDS busy meanwhile, so writing a slab
// costs as much LDS time as reading it three times; measured on the chip, fragment reads running beside
// register-staged stores take the sum of both times, beside direct loads the maximum.

// NS: LDS stages.
// PW: extra wavefronts that do nothing but issue the direct loads. A
//     vector-memory instruction holds its wavefront at issue while the address unit is busy, and the 32 KB
//     a 128x128 tile needs per slab keep that unit (64 B per clock) busy for as long as the slab's MFMAs
//     take; with the loads on wavefronts of their own, that wait never stands in front of an MFMA.
//     0 = every wavefront loads its share, spread between its MFMAs (256x256 tiles, which have twice the MFMAs per byte).
// KTAIL: K is no multiple of BK and an operand is contiguous along it.
// F16: the 16-bit elements are IEEE half instead of bf16 (same data movement; MFMA and conversions differ).
// Position of workgroup `bid` of a grid of tiles_m x tiles_n tiles. Workgroups are handed to the 8 XCDs round-robin;
// the ids are renumbered so that each XCD (own L2) gets a run of consecutive tile ids, and the ids are ordered in
// groups of 4 tile rows walked column by column, so that the tiles an XCD works on at the same time form a compact
// block: its workgroups walk K in step, and every A (B) slab that reaches the L2 is used by all tiles of its row
// (column) in the block. `copies`: the grid holds that many copies of the tile set (K ranges), copy after copy.
struct TilePos { int tile_m, tile_n, copy; };
__device__ __forceinline__ TilePos tile_in_order(int id, int tiles_m, int tiles_n) {
  TilePos t;
  t.copy = 0;
  constexpr int GROUP_M = 4;
  const int group = id / (GROUP_M * tiles_n);
  const int first_m = group * GROUP_M;
  const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
  const int in_group = id - group * GROUP_M * tiles_n;
  t.tile_m = first_m + in_group % gsz;
  t.tile_n = in_group / gsz;
  return t;
}
__device__ __forceinline__ TilePos tile_position(int bid, int tiles_m, int tiles_n, int copies) {
  const int nblk = tiles_m * tiles_n;
  const int per_xcd = (nblk * copies) / 8;
  if (bid < per_xcd * 8) bid = (bid & 7) * per_xcd + (bid >> 3);
  const int copy = bid / nblk;
  TilePos t = tile_in_order(bid - copy * nblk, tiles_m, tiles_n);
  t.copy = copy;
  return t;
}

// Byte offset behind the last piece of any operand: fewer than 2^31 elements, a multiple of 8 of them.
constexpr unsigned BEYOND_OPERANDS = 0xfffffff0u;

// HYB: a grid whose tile count is not a multiple of the 256 CUs ends in a thin round that costs a full one. A
// hybrid launch runs the tiles of the full rounds as usual (workgroups below tail_begin) and cuts each tile of
// the remainder into tail_splits K ranges, one workgroup each, so that the last round is short instead of
// thin: workgroup tail_begin + r * (tiles in the tail) + t covers range r of tail tile t and leaves its fp32
// accumulators as a full tile in hyb_ws[(t * tail_splits + r)][BM][BN]; hybrid_reduce_kernel adds the ranges in
// order and applies the epilogue. Plain launches pass tail_begin = number of tiles.
// BY_AUX (EPI_ADD): whether there is a sum to add to is told by aux_in, not by the instance.
// `block`: this workgroup's position in the grid of the product (not blockIdx.x where a launch holds several products).
// m_at >= 0: the tile's origin (m_at, n_at) in place of a position.
template <int LAYOUT, int BM, int BN, int BK, int WGM, int WGN, int KS, int NS, int PW, bool KTAIL, int EPI,
          bool F16 = false, bool HYB = false, bool BY_AUX = false>
__device__ __forceinline__ void gemm_bf16_tile(int block, int M, int N, int K, const bf16_t* __restrict__ A,
                                               const bf16_t* __restrict__ B, bf16_t* __restrict__ C,
                                               const bf16_t* __restrict__ bias, const bf16_t* aux_in,
                                               bf16_t* __restrict__ aux_out, int act, int tail_begin, int tail_splits,
                                               float* __restrict__ hyb_ws, int m_at = -1, int n_at = 0) {
  constexpr bool A_KC = (LAYOUT != GEMM_TN);  // A operand contiguous along K
  constexpr bool B_KC = (LAYOUT == GEMM_NT);
  // KS == 2: two sets of WGM x WGN wavefronts share the output tile; set g multiplies the g-th half of
  // every K slab and the two accumulator sets are added through LDS before the epilogue. This doubles the
  // wavefronts per SIMD without shrinking the per-wave tile (LDS traffic per flop stays that of the
  // larger wave tile).
  constexpr int NCOMP = WGM * WGN * KS * 64;         // threads that compute
  constexpr int NTHR = PW ? PW * 64 : NCOMP;         // threads that load
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  constexpr int A_LOADS = BM * BK / 8 / NTHR, B_LOADS = BN * BK / 8 / NTHR;
  static_assert(A_LOADS >= 1 && B_LOADS >= 1, "tile too small for the thread count");
  static_assert(BK == 64 || BK == 128, "swizzles and fragment addresses written for 128- and 256-byte tile rows");
  static_assert(TM % 2 == 0, "tile rows are multiplied in pairs");
  static_assert((A_KC || BM >= 64) && (B_KC || BN >= 64), "at least four 32-byte granules per row of an M-contiguous tile");
  static_assert(NS >= 2 && NS <= 10, "stage count");
  constexpr int PA = A_KC ? BK : BM;        // row pitch of the A tile in elements (unpadded)
  constexpr int PB = B_KC ? BK : BN;
  constexpr int SA = BM * BK, SB = BN * BK;  // elements per stage
  auto swzK = [](int row) { return BK == 64 ? (row / 2) % 8 : row % 16; };
  auto swzM = [](int krow, auto width) {
    constexpr int W = decltype(width)::value;
    constexpr int RPM = W >= 128 ? 1 : 128 / W;   // k-rows per 256 bytes of LDS
    const int q = krow / RPM;
    // One transposing read covers, per group of 32 lanes, one granule of k-rows r..r+3 and r+8..r+11: eight 32-byte
    // pieces that must land in eight different bank groups. The k-row picks bits 1-2 of the granule position (bit 1
    // only for 64-wide tiles, whose rows alternate between the two halves of the 256 bytes by themselves); rows 8 apart
    // differ in bit 0.
    return W >= 128 ? (((q & 3) << 1) ^ ((q >> 3) & 1)) : (((q & 1) << 1) ^ ((q >> 2) & 1));
  };
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* sA = smem;               // [NS][SA]
  bf16_t* sB = smem + NS * SA;   // [NS][SB]

  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM;
  const int nblk = tiles_m * tiles_n;
  // Split-K instances: `act` K ranges per tile, every (range, tile) pair a workgroup; consecutive ids walk the
  // tiles of one range, so the blocks an XCD holds still share operand panels.
  constexpr bool SPLITK = (EPI == EPI_SPLITK);
  static_assert(!(HYB && SPLITK), "one kind of K range at a time");
  int bid = block;
  bool is_tail = false;          // (uniform for the workgroup)
  int tail_range = 0, tail_tile = 0;
  if (HYB && bid >= tail_begin) {
    const int t = bid - tail_begin, tail_tiles = nblk - tail_begin;
    tail_range = t / tail_tiles;
    tail_tile = t - tail_range * tail_tiles;
    bid = tail_begin + tail_tile;
    is_tail = true;
  }
  const TilePos pos = tile_position(bid, tiles_m, tiles_n, SPLITK ? act : 1);
  const int splits = SPLITK ? act : (is_tail ? tail_splits : 1);
  const int split = SPLITK ? pos.copy : tail_range;
  const int tile_m = pos.tile_m, tile_n = pos.tile_n;
  const int m0 = m_at >= 0 ? m_at : tile_m * BM, n0 = m_at >= 0 ? n_at : tile_n * BN;

  const int lane = threadIdx.x & 63;
  const bool is_loader = PW ? threadIdx.x >= NCOMP : true;
  const int tid = PW ? (is_loader ? threadIdx.x - NCOMP : 0) : threadIdx.x;   // index among the loading threads
  const int cw = threadIdx.x >> 6;                                            // wavefront index
  const int kgroup = cw / (WGM * WGN), wave = cw % (WGM * WGN);
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;

  // Each loading thread moves A_LOADS + B_LOADS 16-byte pieces per slab: thread t owns position t of the slab (tile
  // row t / CA, chunk position t % CA), piece i sits NTHR positions (RSA tile rows) further. Pieces outside M or N are
  // whatever the buffer holds there (zero past its end) and never reach a stored output.
  constexpr int CA = A_KC ? BK / 8 : BM / 8, CB = B_KC ? BK / 8 : BN / 8;   // pieces per tile row
  constexpr int RSA = NTHR / CA, RSB = NTHR / CB;                            // tile rows between pieces
  const int ar = tid / CA, br = tid / CB;
  // column (in elements) of the chunk fetched for the position in tile row r
  auto col_a = [&](int r) {
    return A_KC ? ((tid % CA) ^ swzK(r)) * 8 : ((tid % CA) ^ (swzM(r, std::integral_constant<int, BM>{}) << 1)) * 8;
  };
  auto col_b = [&](int r) {
    return B_KC ? ((tid % CB) ^ swzK(r)) * 8 : ((tid % CB) ^ (swzM(r, std::integral_constant<int, BN>{}) << 1)) * 8;
  };
  const int lda = A_KC ? K : M, ldb = B_KC ? K : N;
  const int64_t stepA = A_KC ? BK : (int64_t)BK * lda, stepB = B_KC ? BK : (int64_t)BK * ldb;

  // slabs of this workgroup: all of them, or the split's range (the host makes every range non-empty)
  const int nk_all = (K + BK - 1) / BK;
  const int nk_per = (nk_all + splits - 1) / splits;
  const int ks0 = split * nk_per;   // (split = 0, splits = 1 for workgroups that walk all of K)
  const int nk = nk_all - ks0 < nk_per ? nk_all - ks0 : nk_per;
  // The pieces are written by the memory system straight into LDS (wave-uniform LDS base,
  // lane l lands 16 l bytes behind it). Completion is tracked by the vector-memory counter. The loads are
  // buffer loads: resource = the operand from the tile's origin on, per-lane byte offset fixed for the whole
  // K loop, the K step in the scalar offset. Issuing a slab then takes no vector-ALU instruction at all,
  // which matters because the vector ALU is where the MFMAs run: address arithmetic of a loading wavefront
  // queues behind the MFMAs of the wavefronts that share its SIMD (measured: 64-bit per-lane addresses make
  // load time and MFMA time add up; this form overlaps them). Reads beyond the operand's end return zero.
  // A row beyond K may lie more than 32 bits of bytes away (rows of over 34 million elements): its offset stops at one
  // that is beyond the end of every operand, instead of wrapping back into it.
  auto byte_offset = [](int row, int ld, int col) {
    const uint64_t b = 2 * ((uint64_t)row * ld + col);
    return b < BEYOND_OPERANDS ? (unsigned)b : BEYOND_OPERANDS;
  };
  unsigned voa[A_LOADS], vob[B_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; ++i) voa[i] = byte_offset(ar + i * RSA, lda, col_a(ar + i * RSA));
#pragma unroll
  for (int i = 0; i < B_LOADS; ++i) vob[i] = byte_offset(br + i * RSB, ldb, col_b(br + i * RSB));
  const int64_t origin_a = A_KC ? (int64_t)m0 * lda : m0, origin_b = B_KC ? (int64_t)n0 * ldb : n0;
  auto records = [](int64_t elems) { const int64_t b = elems * 2; return (unsigned)(b < 0xffffffffll ? b : 0xffffffffll); };
  const bf16_t* base_a = A + origin_a;
  const bf16_t* base_b = B + origin_b;
  const unsigned bytes_a = records((int64_t)M * K - origin_a), bytes_b = records((int64_t)N * K - origin_b);
  const int lw = __builtin_amdgcn_readfirstlane(PW ? cw - NCOMP / 64 : cw);   // index among the loading wavefronts
  // Fragments of an operand that is not contiguous along K come through transposing reads, which the compiler would
  // hold back behind every direct load this wavefront has in flight (common.h): wavefronts that also compute issue
  // their loads where it does not see them.
  constexpr bool UNTRACKED = PW == 0;
  auto dma16 = [](const bf16_t* base, unsigned bytes, bf16_t* lds, unsigned voffset, unsigned soffset) {
    if constexpr (UNTRACKED) buffer_load_lds_16_untracked(base, bytes, lds, voffset, soffset);
    else buffer_load_lds_16(base, bytes, lds, voffset, soffset);
  };
  // A K that is no multiple of BK ends in a partial slab. Operands whose rows run along the other dimension end with
  // the buffer there (zeros by the bounds above); the pieces of a K-contiguous row that lie at or beyond K would read
  // the next row, so the last slab sends them out of bounds (K % 8 == 0: a piece lies on one side as a whole). KTAIL:
  // instances for such K of their own, because the test alone costs the others 1.5 % (loads issued by computing waves).
  auto load_piece = [&](int kstep, int stage, int i) {   // piece i of the A (i < A_LOADS) or B tile of a slab
    const int left = K - (ks0 + kstep) * BK;   // (uniform)
    const bool last = KTAIL && (A_KC || B_KC) && left < BK;
    if (i < A_LOADS) {
      bf16_t* a = sA + stage * SA + lw * 512;
      const unsigned soa = (unsigned)(ks0 + kstep) * (unsigned)(stepA * 2);
      dma16(base_a, bytes_a, a + i * NTHR * 8, !last || !A_KC || col_a(ar + i * RSA) < left ? voa[i] : BEYOND_OPERANDS, soa);
    } else {
      i -= A_LOADS;
      bf16_t* b = sB + stage * SB + lw * 512;
      const unsigned sob = (unsigned)(ks0 + kstep) * (unsigned)(stepB * 2);
      dma16(base_b, bytes_b, b + i * NTHR * 8, !last || !B_KC || col_b(br + i * RSB) < left ? vob[i] : BEYOND_OPERANDS, sob);
    }
  };
  auto load_direct = [&](int kstep, int stage) {
#pragma unroll
    for (int i = 0; i < A_LOADS + B_LOADS; ++i) load_piece(kstep, stage, i);
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // Per-lane fragment addressing (stage 0, k-step 0). A fragment is 16 rows x 32 k: lane l holds k 8 (l / 16) .. + 7 of
  // row l % 16.
  // K-contiguous: chunk 4*ks + lane/16 of the row, stored at position (4*ks + lane/16) ^ swzK = (4*ks ^ fsw) with the two
  // low bits folded into the base.
  const int fsw = swzK(lane & 15) & (BK / 8 - 4);
  const int kc_low = (((lane >> 4) ^ swzK(lane & 15)) & 3) << 3;
  const int fa_base = (wm0 + (lane & 15)) * PA + kc_low;
  const int fb_base = (wn0 + (lane & 15)) * PB + kc_low;
  // M-contiguous: the lane reads 4 elements at k-row krow_l (+4 for the upper half of the fragment), column 4*(lane%4) of
  // the 16-wide granule g, which is stored at g ^ swzM.
  const int krow_l = 8 * (lane >> 4) + ((lane & 15) >> 2);
  int ma_lo[2], ma_sw[2], mb_lo[2], mb_sw[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ma_lo[h] = (krow_l + 4 * h) * PA + 4 * (lane & 3);
    mb_lo[h] = (krow_l + 4 * h) * PB + 4 * (lane & 3);
    ma_sw[h] = swzM(krow_l + 4 * h, std::integral_constant<int, BM>{});
    mb_sw[h] = swzM(krow_l + 4 * h, std::integral_constant<int, BN>{});
  }
  auto frag_kc = [&](const bf16_t* tile, int base, int pitch, int t, int ks) -> bf16x8_t {
    return *reinterpret_cast<const bf16x8_t*>(tile + base + t * 16 * pitch + (((4 * ks) ^ fsw) << 3));
  };
  auto frag_mc = [&](const bf16_t* tile, const int (&lo)[2], const int (&sw)[2], int pitch, int g, int ks) -> bf16x8_t {
    typedef s16x4_t __attribute__((address_space(3))) * lds4_t;
    const bf16_t* p = tile + ks * 32 * pitch;
    s16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(p + lo[0] + ((g ^ sw[0]) << 4)));
    s16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(p + lo[1] + ((g ^ sw[1]) << 4)));
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    s16x8_t v = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  };
  // The operands are swapped (the instruction's rows are the columns of C), so a lane holds four consecutive columns of
  // one row of C.
  constexpr int KQ = BK / 32 / KS;
  auto read_a = [&](int stage, int kq, int i) {
    const bf16_t* a = sA + stage * SA;
    const int ks = kq + kgroup * KQ;
    return A_KC ? frag_kc(a, fa_base, PA, i, ks) : frag_mc(a, ma_lo, ma_sw, PA, (wm0 >> 4) + i, ks);
  };
  auto read_b = [&](int stage, int kq, int j) {
    const bf16_t* b = sB + stage * SB;
    const int ks = kq + kgroup * KQ;
    return B_KC ? frag_kc(b, fb_base, PB, j, ks) : frag_mc(b, mb_lo, mb_sw, PB, (wn0 >> 4) + j, ks);
  };
  constexpr int LPS = A_LOADS + B_LOADS;   // loads per slab and loading wavefront

  if constexpr (PW == 0) {
    // Two stages, every wavefront loads its share. The slab is a stream of pairs of tile rows (2 TN MFMAs each): the next
    // pair's two A fragments are requested in front of the first two MFMAs of this one, and a B fragment of the next
    // k-step right behind its last use in this one, six MFMAs ahead of its first use, so 32 registers of fragments are
    // enough. The barrier that hands over the next slab stands in front of the LAST pair, whose operands are in registers
    // by then: its MFMAs cover the barrier and the LDS round trip of the next slab's first fragments. From there on
    // this slab's stage is free, so the loads of the slab after the next one start in the last pair, one every LOAD_GAP
    // MFMAs (a vector-memory instruction holds its wavefront while the address unit is busy).
    // Same card, against the 32x32x16 form with its barrier between two slabs: NT 8192 x 2048 x 8192 202 -> 182.5 us (1.51
    // PFLOP/s), NN 207 -> 183, TN 2048 x 8192 x 8192 209 -> 186; the change of MFMA form alone gives 189 / 188 / 194.
    // What is left is the clock (1.8 GHz under this load) and, per tile, 8-11 us of first loads and last stores.
    static_assert(NS == 2 && KS == 1, "alternating stages");
    constexpr int PAIRS = TM / 2, NPAIR = KQ * PAIRS, MPP = 2 * TN;
    // Epilogues that move two values per product element put bursts of stores between the other workgroups' loads: the
    // earlier request pays there (4096 x 22016 x 4096 gated: 574 us at a gap of 2, 598 at 4, 627 at 6), the even spread
    // everywhere else (8192 x 2048 x 8192: 187.7 / 182.5 / 186.2).
    // (Tiles of 128x128 have half the MFMAs per load.)
    constexpr int LOAD_GAP = BM == 128 || EPI == EPI_GATE || EPI == EPI_DGATE || EPI == EPI_BIAS_ACT ? 2 : 4;
    static_assert(LOAD_GAP * (LPS - 1) < NPAIR * MPP - MPP, "all loads issued in front of the wait");
    constexpr int EARLY = (MPP + LOAD_GAP - 1) / LOAD_GAP;   // loads issued in the last pair of the slab before
#pragma unroll
    for (int i = 0; i < LPS; ++i) load_piece(0, 0, i);
    if (nk > 1) {
#pragma unroll
      for (int i = 0; i < EARLY; ++i) load_piece(1, 1, i);
      wait_loads_and_lds<EARLY>();
    } else {
      wait_loads_and_lds<0>();
    }
    block_barrier();
    bf16x8_t fa[2][2], fb[TN];
    fa[0][0] = read_a(0, 0, 0);
    fb[0] = read_b(0, 0, 0);
    fa[0][1] = read_a(0, 0, 1);
#pragma unroll
    for (int j = 1; j < TN; ++j) fb[j] = read_b(0, 0, j);
    for (int k0 = 0; k0 < nk; k0 += 2) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = k0 + s;
        if (k >= nk) break;   // uniform
        static_assert(NPAIR % 2 == 0, "register sets alternate across slabs");
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) {
          const int kq = p / PAIRS, ip = p % PAIRS;
          const bool last = p + 1 == NPAIR;
          if (last) {
            wait_loads_and_lds<0>();
            block_barrier();
          }
          // (behind the last slab the requests read a stage whose contents nobody uses)
          const int nstage = last ? s ^ 1 : s, np = last ? 0 : p + 1;
#pragma unroll
          for (int m = 0; m < MPP; ++m) {
            const int j = m >> 1, h = m & 1;
            if (m < 2) fa[(p + 1) & 1][m] = read_a(nstage, np / PAIRS, 2 * (np % PAIRS) + m);
            if (m == 0 && ip == 0) fb[TN - 1] = read_b(s, kq, TN - 1);
            if (h == 0 && j > 0 && ip == PAIRS - 1) fb[j - 1] = read_b(nstage, last ? 0 : kq + 1, j - 1);
            const int n = last ? m : MPP + p * MPP + m;   // MFMAs since the barrier
            if (n % LOAD_GAP == 0 && n / LOAD_GAP < LPS) {
              if (last) {
                if (k + 2 < nk) load_piece(k + 2, s, n / LOAD_GAP);
              } else if (k + 1 < nk) {
                load_piece(k + 1, s ^ 1, n / LOAD_GAP);
              }
            }
            acc[2 * ip + h][j] = mfma16_16<F16>(fb[j], fa[p & 1][h], acc[2 * ip + h][j]);
            __builtin_amdgcn_sched_barrier(0);   // keep this order (the scheduler would sink the requests)
          }
        }
      }
    }
  } else {
    // Pipeline over a ring of NS stages, slab j in stage j % NS. Step k issues the loads of slab k + NS - 1
    // into the stage that step k - 1 computed from (free
    // since the barrier that ended step k - 1), computes slab k, then waits until its own loads of slab
    // k + 1 have landed (the younger ones stay in flight) and meets the other wavefronts at the barrier.
    auto compute = [&](int stage) {
      // Scheduling hint for the slab: interleave the LDS reads with the MFMAs. With two transposing reads per fragment of
      // both operands the plain order is the faster one (same card: 2048 x 2048 x 8192 60.9 us, 64.4 and 66.0 with the
      // interleaving and its second variant, 1024 x 4096 x 16384 115.8 / 122.3 / 125.7); elsewhere 0-3 % the other way.
      if constexpr (LAYOUT != GEMM_TN) __builtin_amdgcn_iglp_opt(0);
#pragma unroll
      for (int kq = 0; kq < KQ; ++kq) {
        bf16x8_t fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = read_a(stage, kq, i);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = read_b(stage, kq, j);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma16_16<F16>(fb[j], fa[i], acc[i][j]);
      }
    };
    if (is_loader) {
#pragma unroll
      for (int j = 0; j < NS - 1; ++j)
        if (j < nk) load_direct(j, j);   // (uniform)
    }
    if (nk >= NS - 1) wait_loads_and_lds<(NS - 2) * LPS>();
    else wait_loads_and_lds<0>();
    block_barrier();
    if (is_loader) {
      // loader wavefronts: issue, wait for the oldest slab, meet the others; nothing else
      for (int k0 = 0; k0 < nk; k0 += NS) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (k0 + s >= nk) break;                  // uniform (slab counts that are no multiple of NS)
          const bool more = k0 + s + NS - 1 < nk;   // uniform
          if (more) load_direct(k0 + s + NS - 1, (s + NS - 1) % NS);
          if (more) wait_loads_and_lds<(NS - 2) * LPS>();
          else wait_loads_and_lds<0>();
          block_barrier();
        }
      }
    } else {
      for (int k0 = 0; k0 < nk; k0 += NS) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (k0 + s >= nk) break;                   // uniform
          compute(s);
          wait_loads_and_lds<63>();                  // LDS reads done (no loads of its own)
          block_barrier();
        }
      }
    }
  }

  if (PW && is_loader) return;   // every load has landed (the last steps drain them); the rest is compute only

  // Epilogue. The accumulators (element r of a 16x16 tile: row lane%16, column 4*(lane/16) + r) go, one 32-row slab at a
  // time, through a per-wave fp32 staging area in LDS so that every global access of the epilogue (bias, auxiliary
  // input, both outputs) is a 16-byte access of 8 consecutive columns of one row. The stages are free: every wavefront
  // has met the others behind its last read that counts (alternating stages: the reads behind the last slab's barrier
  // fetch what nobody uses).
  if (KS == 2) {   // add the second wave set's accumulators to the first; then only the first goes on
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem) + wave * (TM * TN * 64) + lane;
    if (kgroup == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) red[(i * TN + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (kgroup == 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const f32x4_t other = red[(i * TN + j) * 64];
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] += other[r];
        }
    }
    __syncthreads();
    if (kgroup == 1) return;
  }
  constexpr int SM = WM / 32;   // 32-row slabs of the wave tile
  constexpr int LDP = WN + 4;
  float* stage = reinterpret_cast<float*>(smem) + wave * (32 * LDP);
  constexpr int CPR = WN / 8;         // 8-column chunks per staged row
  constexpr int RPP = 64 / CPR;       // rows covered by one pass of the wave
  const int cc = lane % CPR, rr = lane / CPR;
  const int n = n0 + wn0 + cc * 8;
  float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if ((EPI == EPI_BIAS || EPI == EPI_BIAS_ACT) && n < N) load8h<F16>(bias + n, bv);
  // The auxiliary input of a 32-row slab is fetched one slab ahead (clamped addresses, so the loads are
  // unconditional): its latency passes while the slab before it is staged and written out.
  constexpr bool AUX = (EPI == EPI_DACT || EPI == EPI_ADD || EPI == EPI_DGATE);
  constexpr int NP = 32 / RPP;
  constexpr int NAUX = EPI == EPI_DGATE ? 2 : 1;   // 16-byte pieces of auxiliary input per 8 product columns
  u32x4_t au[SM][NP * NAUX];
  auto aux_fetch = [&](int i, u32x4_t (&dst)[NP * NAUX]) {
    const int nc = n < N ? n : N - 8;
#pragma unroll
    for (int pass = 0; pass < NP; ++pass) {
      int m = m0 + wm0 + i * 32 + pass * RPP + rr;
      m = m < M ? m : M - 1;
      if constexpr (EPI == EPI_DGATE) {   // the factor pairs of product columns nc..nc+7 sit in columns 2nc..2nc+15 of [M,2N]
        const bf16_t* q = aux_in + (int64_t)m * (2 * N) + 2 * nc;
        dst[2 * pass] = *reinterpret_cast<const u32x4_t*>(q);
        dst[2 * pass + NAUX - 1] = *reinterpret_cast<const u32x4_t*>(q + 8);
      } else {
        dst[pass] = *reinterpret_cast<const u32x4_t*>(aux_in + (int64_t)m * N + nc);
      }
    }
  };
  auto aux_get = [](const u32x4_t& w, float (&u)[8]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) { u[2 * e] = unpack_lo<F16>(w[e]); u[2 * e + 1] = unpack_hi<F16>(w[e]); }
  };
  // EPI_DACT: aux_out takes the column sums of every 32 rows of C, [M / 32 rounded up][N] floats (NULL: none), from which the bias
  // gradient in front of the activation comes without another pass over C. The sums are of the unrounded values; a value that the
  // storage type holds as an infinity counts as one (IEEE half, from 65520 on; bf16 reaches as far as the sums do).
  static_assert(EPI != EPI_DACT || CPR == 4 || CPR == 8 || CPR == 16, "sum_of_lanes");
  float* col_sums = EPI == EPI_DACT ? reinterpret_cast<float*>(aux_out) : nullptr;
  const bool aux_here = AUX && !is_tail && (!BY_AUX || aux_in != nullptr);   // (uniform)
  if (aux_here) aux_fetch(0, au[0]);
#pragma unroll
  for (int i = 0; i < SM; ++i) {
    if (aux_here && i + 1 < SM) aux_fetch(i + 1, au[i + 1]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        *reinterpret_cast<f32x4_t*>(stage + (h * 16 + (lane & 15)) * LDP + j * 16 + 4 * (lane >> 4)) = acc[2 * i + h][j];
    __builtin_amdgcn_wave_barrier();
    float sums[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int pass = 0; pass < 32 / RPP; ++pass) {
      const int row = pass * RPP + rr;
      const int m = m0 + wm0 + i * 32 + row;
      float v[8];
      const float4 lo = *reinterpret_cast<const float4*>(stage + row * LDP + cc * 8);
      const float4 hi = *reinterpret_cast<const float4*>(stage + row * LDP + cc * 8 + 4);
      v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
      if (HYB && is_tail) {   // one K range of a tail tile: the bare accumulators, as a full tile of the workspace
        float* part = hyb_ws + ((size_t)(tail_tile * tail_splits + tail_range) * BM + (wm0 + i * 32 + row)) * BN + wn0 + cc * 8;
        *reinterpret_cast<float4*>(part) = lo;
        *reinterpret_cast<float4*>(part + 4) = hi;
      } else if (m < M && n < N) {
        const int64_t idx = (int64_t)m * N + n;
        if (EPI == EPI_BIAS) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += bv[e];
        } else if (EPI == EPI_BIAS_ACT) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += bv[e];
          // Activation and its derivative from the same fp32 pre-activation; the derivative is what is kept
          // for backward (the activation terms are at hand here, and backward is then one multiply).
          float dv[8];
          if (act == ACT_RELU) {
#pragma unroll
            for (int e = 0; e < 8; ++e) { dv[e] = v[e] > 0.f ? 1.f : 0.f; v[e] = v[e] > 0.f ? v[e] : 0.f; }
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const GeluTerms g = gelu_terms(v[e]);
              dv[e] = fmaf(v[e] * g.e, 0.39894228040143268f, g.phi);
              v[e] *= g.phi;
            }
          }
          if (aux_out) store8h<F16>(aux_out + idx, dv);   // (a ReLU layer keeps nothing: its gate is read off the output)
        } else if (EPI == EPI_DACT) {
          float u[8];
          aux_get(au[i][pass], u);
          if (act == ACT_RELU) {   // aux_in is the activation output (or the stored 0/1 derivative): gate = [aux_in > 0]
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = u[e] > 0.f ? v[e] : 0.f;
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= u[e];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) sums[e] += !F16 || fabsf(v[e]) < 65520.f ? v[e] : v[e] * __builtin_inff();
        } else if (EPI == EPI_ADD) {
          if (!BY_AUX || aux_here) {
            float u[8];
            aux_get(au[i][pass], u);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += u[e];
          }
        } else if constexpr (EPI == EPI_ROPE) {
          if (n < 2 * (N / 3)) {
            round_pairs<F16>(v);   // what a kernel that turns the stored product would read
            rope_turn<4>(v, reinterpret_cast<const float*>(bias), act, m, n);
          }
        } else if (EPI == EPI_GATE) {
          // columns come as (gate, up) pairs: four gated values go to C [M,N/2], the backward factors stay [M,N]
          float f[8], o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const GateTerms g = gate_terms<true>(v[2 * e], v[2 * e + 1]);
            o[e] = g.out; f[2 * e] = g.dgate; f[2 * e + 1] = g.dup;
          }
          store8h<F16>(aux_out + idx, f);
          uint2 w;
          w.x = pack2<F16>(o[0], o[1]);
          w.y = pack2<F16>(o[2], o[3]);
          *reinterpret_cast<uint2*>(C + (int64_t)m * (N / 2) + n / 2) = w;
        } else if constexpr (EPI == EPI_DGATE) {
          float fa[8], fb[8], o0[8], o1[8];
          aux_get(au[i][2 * pass], fa);
          aux_get(au[i][2 * pass + NAUX - 1], fb);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o0[2 * e] = v[e] * fa[2 * e]; o0[2 * e + 1] = v[e] * fa[2 * e + 1];
            o1[2 * e] = v[4 + e] * fb[2 * e]; o1[2 * e + 1] = v[4 + e] * fb[2 * e + 1];
          }
          bf16_t* q = C + (int64_t)m * (2 * N) + 2 * n;
          store8h<F16>(q, o0);
          store8h<F16>(q + 8, o1);
        }
        else if (EPI == EPI_SPLITK) {
          float* part = reinterpret_cast<float*>(aux_out) + (int64_t)split * M * N + idx;
          *reinterpret_cast<float4*>(part) = make_float4(v[0], v[1], v[2], v[3]);
          *reinterpret_cast<float4*>(part + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
        if (EPI != EPI_GATE && EPI != EPI_DGATE && EPI != EPI_SPLITK) store8h<F16>(C + idx, v);
      }
    }
    if (EPI == EPI_DACT && col_sums) {   // (uniform)
#pragma unroll
      for (int e = 0; e < 8; ++e) sums[e] = sum_of_lanes<CPR>(sums[e]);
      const int first = m0 + wm0 + i * 32;
      if (rr == 0 && first < M && n < N) store8(col_sums + (int64_t)(first / 32) * N + n, sums);
    }
  }
}

template <int BM, int BN, int BK, int WGM, int WGN, int KS, int NS>
constexpr size_t gemm_lds_bytes() {
  constexpr size_t main_bytes = (size_t)NS * (BM + BN) * BK * sizeof(bf16_t);
  constexpr size_t epi_bytes = (size_t)WGM * WGN * 32 * (BN / WGN + 4) * sizeof(float);
  constexpr size_t red_bytes = KS == 2 ? (size_t)BM * BN * sizeof(float) : 0;
  constexpr size_t m1 = main_bytes > epi_bytes ? main_bytes : epi_bytes;
  return m1 > red_bytes ? m1 : red_bytes;
}

// fp32: 32x32 tiles (W = 2), or 16x16 (W = 1) where the larger ones would leave half of the CUs idle, eight wavefronts
// that take the 16-deep K chunks of the tile in turn, so that a product with few tiles (256 tokens, 256 columns: 64) still
// has 512 wavefronts' loads in flight; such products are bound by the chain of load latencies, not by the 157 TFLOP/s of
// the fp32 MFMAs. Operands go from memory to registers in the shape of
// v_mfma_f32_16x16x4_f32 fragments (nothing is shared between wavefronts that do not share K), the next chunk requested
// ahead of the one that is multiplied; the partial tiles meet in LDS. Inputs, products and sums are fp32 as in a plain FMA
// loop. (Two or four chunks ahead need 150-250 registers and lose more to the fewer wavefronts: 512 x 3072 x 768 takes 52
// and 67 us.)
// A fragment element belongs to k = k0 + 4 (lane/16) + s in step s for either operand; lane%16 counts rows.
//  - contiguous along K: one 16-byte load per 16 rows gives the four steps
//  - contiguous along rows: one load of W floats per step gives the rows W (lane%16) .. + W - 1 of the W 16-row tiles
// Against one 64x64 tile of plain FMAs per workgroup: 256 x 256 x 1024 142 -> 6 us, 512 x 3072 x 768 157 -> 48 us.
constexpr int F32_WAVES = 8;
constexpr int f32_lds_floats(int W) { return F32_WAVES * 16 * W * (16 * W + 4); }
template <int LAYOUT, int W>
__device__ __forceinline__ void gemm_f32_tile(int block, float* lds, int M, int N, int K, const float* __restrict__ A,
                                              const float* __restrict__ B, float* __restrict__ C,
                                              const float* __restrict__ bias, const float* aux_in,
                                              float* __restrict__ aux_out, int epi, int act) {
  constexpr bool A_KC = LAYOUT != GEMM_TN, B_KC = LAYOUT == GEMM_NT;
  constexpr int TILE = 16 * W, PITCH = TILE + 4;   // floats per staged row
  float(*part)[TILE * PITCH] = reinterpret_cast<float(*)[TILE * PITCH]>(lds);   // [F32_WAVES]
  const int tiles_n = (N + TILE - 1) / TILE;
  const int m0 = (block / tiles_n) * TILE, n0 = (block % tiles_n) * TILE;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;

  struct Frag { float v[W][4]; };   // [16-row tile][step]
  // rows beyond the operand are clamped (their products are never stored), k beyond K is zero in both operands
  auto load = [&](auto kc, const float* X, int r0, int rows, int k0) {
    Frag f;
    if constexpr (decltype(kc)::value) {
      const int k = k0 + 4 * g;
#pragma unroll
      for (int t = 0; t < W; ++t) {
        const int r = r0 + 16 * t + i < rows ? r0 + 16 * t + i : rows - 1;
        float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < K) w = *reinterpret_cast<const float4*>(X + (int64_t)r * K + k);   // (K % 8 == 0)
        f.v[t][0] = w.x; f.v[t][1] = w.y; f.v[t][2] = w.z; f.v[t][3] = w.w;
      }
    } else {
      const int r = r0 + W * i < rows ? r0 + W * i : rows - W;                      // (rows % 8 == 0)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + 4 * g + s;
        if constexpr (W == 2) {
          float2 w = make_float2(0.f, 0.f);
          if (k < K) w = *reinterpret_cast<const float2*>(X + (int64_t)k * rows + r);
          f.v[0][s] = w.x; f.v[1][s] = w.y;
        } else {
          f.v[0][s] = k < K ? X[(int64_t)k * rows + r] : 0.f;
        }
      }
    }
    return f;
  };
  f32x4_t acc[W][W] = {};
  const int chunks = (K + 15) / 16;
  Frag fa[2], fb[2];
  auto fetch = [&](int buf, int c) {
    if (c >= chunks) return;   // (uniform)
    fa[buf] = load(std::integral_constant<bool, A_KC>{}, A, m0, M, c * 16);
    fb[buf] = load(std::integral_constant<bool, B_KC>{}, B, n0, N, c * 16);
  };
  auto multiply = [&](int buf, int c) {
    if (c >= chunks) return;   // (uniform)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int tm = 0; tm < W; ++tm)
#pragma unroll
        for (int tn = 0; tn < W; ++tn)   // operands swapped: a lane holds four columns of one row
          acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[buf].v[tn][s], fa[buf].v[tm][s], acc[tm][tn], 0, 0, 0);
  };
  fetch(0, wave);
  for (int c = wave; c < chunks; c += 2 * F32_WAVES) {
    fetch(1, c + F32_WAVES);
    multiply(0, c);
    fetch(0, c + 2 * F32_WAVES);
    multiply(1, c + F32_WAVES);
  }
  // element (tm, tn, r) of the lane: row i of A tile tm, row 4 g + r of B tile tn
  float* mine = part[wave];
#pragma unroll
  for (int tm = 0; tm < W; ++tm) {
    float* row = mine + (A_KC ? 16 * tm + i : W * i + tm) * PITCH;
    if constexpr (B_KC) {
#pragma unroll
      for (int tn = 0; tn < W; ++tn) *reinterpret_cast<f32x4_t*>(row + 16 * tn + 4 * g) = acc[tm][tn];
    } else {
#pragma unroll
      for (int tn = 0; tn < W; ++tn)
#pragma unroll
        for (int r = 0; r < 4; ++r) row[W * (4 * g + r) + tn] = acc[tm][tn][r];
    }
  }
  __syncthreads();
  // four columns of one row per thread, the partial tiles added in order
  constexpr int TPR = TILE / 4;   // threads per row
  if (threadIdx.x >= TILE * TPR) return;
  const int row = (int)threadIdx.x / TPR, col = ((int)threadIdx.x % TPR) * 4, m = m0 + row, n = n0 + col;
  if (m >= M || n >= N) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < F32_WAVES; ++w) {
    const float4 x = *reinterpret_cast<const float4*>(part[w] + row * PITCH + col);
    v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
  }
  if (epi == EPI_GATE) {          // (gate, up) pairs in adjacent columns
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const GateTerms t = gate_terms<false>(v[j], v[j + 1]);
      C[(int64_t)m * (N / 2) + (n + j) / 2] = t.out;
      aux_out[(int64_t)m * N + n + j] = t.dgate;
      aux_out[(int64_t)m * N + n + j + 1] = t.dup;
    }
  } else if (epi == EPI_ROPE) {
    if (n < 2 * (N / 3)) rope_turn<2>(v, bias, act, m, n);
#pragma unroll
    for (int j = 0; j < 4; ++j) C[(int64_t)m * N + n + j] = v[j];
  } else if (epi == EPI_DGATE) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t q = (int64_t)m * (2 * N) + 2 * (n + j);
      C[q] = v[j] * aux_in[q];
      C[q + 1] = v[j] * aux_in[q + 1];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) epilogue_store<float>(epi, act, v[j], m, n + j, N, C, bias, aux_in, aux_out);
  }
}

}  // namespace slapo
