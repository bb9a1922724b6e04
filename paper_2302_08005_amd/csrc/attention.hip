// Fused softmax attention, forward and backward (paper section 2.2 step 2: attention computed block
// by block so that the S x S matrix never reaches memory; the appendix schedule swaps it in for the
// matched scaled-dot-product pattern). Works in place on the packed projection [B,S,3H] = Q | K | V,
// so no head transposes are materialised.
//
// 16-bit path. A workgroup of four wavefronts owns 128 query rows (forward, dQ) or 128 key rows (dK/dV) of one (sample,
// head), or 64 in small grids, whose wavefronts then form two groups that share the walk (group_slot); each wavefront
// owns 32 of them and walks the other sequence dimension in 64-row tiles brought into two LDS stages by direct global -> LDS loads (one barrier per tile). All products run on
// v_mfma_f32_32x32x16_bf16 and are arranged "transposed" (S^T = K Q^T, O^T = V^T P^T, ...), because
// then the accumulator layout of the score tile already is the B-operand layout of the next product
// and the per-row softmax state (max, sum, logsumexp, delta) is one scalar per lane; a row's maximum
// and sum need the lane's own 16..32 registers plus a single exchange with lane^32. The operand whose
// contraction index is the strided one in LDS is fetched with the transposing ds_read_b64_tr_b16.
// Backward recomputes the probabilities from the saved logsumexp and is split in two kinds of blocks (dK/dV
// per key tile, dQ per query tile) so that no floating-point atomics are needed: two kernels, or one launch of both kinds
// where neither fills the chip (attn_bwd_both_kernel).
//
// fp32 path (correctness mode): up to 1024 tokens fp32 MFMAs on 16 rows per workgroup, whose scores stay in LDS; longer
// sequences one wavefront per row, plain loops.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace slapo {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// ---- LDS tile [64 rows][D] of bf16, unpadded, 16-byte chunks permuted inside each row ---------------
// The LDS serves 256 B per clock (64 banks of 4 B): 16 lanes of a 16-byte read, 32 lanes of a transposing 8-byte read.
// The same tile is read both ways: 16 consecutive rows x one chunk (operand with the contraction along D), and 4
// consecutive rows x 4 chunks with the transposing read (operand with the contraction along the rows). Position p of
// row r holds chunk p ^ f(r); f is a bijection of the rows that share a chunk position (16 rows at D = 128; 8 pairs of
// rows at D = 64, whose rows are half as long as the banks), so the first kind of read meets every bank group once,
// and the bits of f that choose a group of four chunks come from the lowest bits of r, so the four rows of the second
// kind lie in different groups. (Rows padded by 16 bytes, the layout before, are conflict-free for the first kind
// only: the four rows of a transposing read overlapped in 12 of 16 banks at D = 128, and the LDS spent 50-59 % of its
// cycles on conflicts there.) A fragment address is a per-lane base with a compile-time XOR and a compile-time offset.
template <int D>
struct Tile {
  static constexpr int P = D;              // row pitch in elements
  static constexpr int ELEMS = 64 * P;     // one 64-row tile
  static __device__ __forceinline__ int f(int row) {   // of rows that are equal modulo 16 the same
    return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
  }
};
// per-lane bases, computed once per kernel
template <int D>
__device__ __forceinline__ int rows_base(int lane) {
  const int row = lane & 31;
  return row * Tile<D>::P + ((Tile<D>::f(row) ^ (lane >> 5)) << 3);
}
template <int D>
__device__ __forceinline__ int tr_base(int lane) {
  const int j = lane & 15, g = lane >> 4, row = 4 * (g >> 1) + (j >> 2);
  return row * Tile<D>::P + ((Tile<D>::f(row) ^ (2 * (g & 1) + ((j >> 1) & 1))) << 3) + 4 * (j & 1);
}
// MFMA operand whose 32 rows are tile rows r0.. (a multiple of 16) and whose contraction runs along D (step s of 16)
template <int D>
__device__ __forceinline__ bf16x8_t frag_rows(const bf16_t* tile, int base, int r0, int s) {
  return *reinterpret_cast<const bf16x8_t*>(tile + (base ^ (16 * s)) + r0 * Tile<D>::P);
}
// MFMA operand whose 32 rows are tile COLUMNS t*32.. and whose contraction runs over tile rows
// c0 + {4kc..4kc+3, 8+4kc..8+4kc+3} (kc = lane/32; c0 a multiple of 16): the order in which a 32x32 accumulator holds
// them. Eight rows further f differs in bit 1.
template <int D>
__device__ __forceinline__ bf16x8_t frag_tr(const bf16_t* tile, int base, int c0, int t) {
  const bf16_t* p0 = tile + (base ^ (32 * t)) + c0 * Tile<D>::P;
  const bf16_t* p1 = tile + (base ^ (32 * t + 16)) + (c0 + 8) * Tile<D>::P;
  s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)p0);
  s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)p1);
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, v);
}
// eight accumulator registers 8h..8h+7 as a bf16 operand
template <bool F16>
__device__ __forceinline__ bf16x8_t pack8(const f32x16_t& v, int h) {
  uint4 w;
  w.x = pack2<F16>(v[8 * h + 0], v[8 * h + 1]); w.y = pack2<F16>(v[8 * h + 2], v[8 * h + 3]);
  w.z = pack2<F16>(v[8 * h + 4], v[8 * h + 5]); w.w = pack2<F16>(v[8 * h + 6], v[8 * h + 7]);
  return __builtin_bit_cast(bf16x8_t, w);
}
// (mfma16_agpr, common.h: the dK/dV kernel of 128-wide heads needs 128 registers for its two output accumulators
// alone; as ordinary registers they leave so few for operands that fragments and the K/V operands are shuttled in
// and out of spill registers inside the loop. The operands of these accumulations are packed by vector
// instructions right before, hence the default two wait states in front.)
// The value exists in ordinary registers at this point of the program: an ordering anchor for operations that
// have no side effects of their own (nothing is emitted).
__device__ __forceinline__ void pin_here(f32x16_t& v) { asm volatile("" : "+v"(v)); }
// Backward of the rotary embedding on four consecutive columns (two pairs) of a head of width d: turned by the negative
// angles of the row's position. (16-bit gradients are rounded first, like the array that a pass of its own would read.)
// The table loads at the end of a block cost a fraction of what the pass would (4 x 1024 tokens, 32 heads of 128: 53 us saved
// with the forward pass); read by lanes of 32 rows, before the rows left through LDS, they cost as much where a block has few steps.
__device__ __forceinline__ void rope_back(float (&v)[4], const float* __restrict__ table, int pos, int d, int col) {
  const float4 w = *reinterpret_cast<const float4*>(table + (int64_t)pos * d + col);
  turn_pair(v[0], v[1], w.x, -w.y);
  turn_pair(v[2], v[3], w.z, -w.w);
}
// row index inside a 32x32 accumulator tile of register r
__device__ __forceinline__ int acc_row(int r, int lane) { return (r >> 2) * 8 + 4 * (lane >> 5) + (r & 3); }

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// A 64 x D tile is brought in by direct global -> LDS loads (no staging registers, no ds_write). One
// wave-level load fills 1 KB of consecutive LDS, lane l at byte 16 l: the lane fetches the chunk that the permutation
// puts there. The D/8 loads of a tile are dealt out to the four wavefronts. Rows past the end of the sequence are whatever
// follows in memory (the next sample's rows, zero past the end of the tensor: the buffer bounds): finite
// values that only ever meet masked scores.
template <int D>
struct TileDirect {
  static constexpr int SPR = D / 8;                // 16-byte chunks per row = wave-level loads per tile
  static constexpr int MINE = SPR / 4;             // loads per tile of one wavefront
  unsigned voff[MINE];
  int wave;                                        // wave-uniform
  __device__ __forceinline__ void init(int lane, int wave_uniform, unsigned row_stride_bytes) {
    wave = wave_uniform;
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
      const int slot = (wave + 4 * k) * 64 + lane, row = slot / SPR, pos = slot % SPR;
      voff[k] = (unsigned)row * row_stride_bytes + (unsigned)(pos ^ Tile<D>::f(row)) * 16u;
    }
  }
  // tile rows row0.. of the operand that starts at `base` (`bytes` long from there) -> LDS tile
  __device__ __forceinline__ void issue(const bf16_t* base, unsigned bytes, bf16_t* tile, unsigned row0_bytes) const {
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
      buffer_load_lds_16_untracked(base, bytes, tile + (wave + 4 * k) * 512, voff[k], row0_bytes);
    }
  }
};

// The tile loop of the forward kernel: a ring of NSTG LDS stages, tiles t+1 .. t+NSTG-1 on their way while
// tile t is computed, one barrier per tile. LPT = loads every wavefront issues per tile step:
// waiting until at most (NSTG-2)*LPT loads are outstanding leaves only younger tiles in flight (loads
// complete in issue order). On the last steps nothing is issued any more and the wait is for everything.
template <int NSTG, int LPT, typename Issue, typename Compute>
__device__ __forceinline__ void tile_ring(int n_tiles, Issue&& issue_tile, Compute&& compute) {
  static_assert(NSTG >= 2, "ring");
  if (n_tiles <= 0) return;
#pragma unroll
  for (int t = 0; t < NSTG - 1; ++t)
    if (t < n_tiles) issue_tile(t, t);
  if (n_tiles >= NSTG - 1) wait_loads_and_lds<(NSTG - 2) * LPT>();
  else wait_loads_and_lds<0>();
  block_barrier();
  for (int it0 = 0; it0 < n_tiles; it0 += NSTG) {
#pragma unroll
    for (int s = 0; s < NSTG; ++s) {   // (stages at compile time: a fragment address is a per-lane base plus an offset in the instruction)
      const int it = it0 + s;
      if (it >= n_tiles) break;        // uniform
      const bool more = it + NSTG - 1 < n_tiles;
      if (more) issue_tile((s + NSTG - 1) % NSTG, it + NSTG - 1);   // that stage was last read before the barrier that ended step it - 1
      compute(s, it);
      if (more) wait_loads_and_lds<(NSTG - 2) * LPT>();
      else wait_loads_and_lds<0>();
      block_barrier();
    }
  }
}

// The walk of a sequence that is one tile (SHORT): nothing is on its way during anything.
template <typename Issue, typename Compute>
__device__ __forceinline__ void one_tile(int n_tiles, Issue&& issue_tile, Compute&& compute) {
  if (n_tiles <= 0) return;
  issue_tile(0, 0);
  wait_loads_and_lds<0>();
  block_barrier();
  compute(0, 0);
}

// Small grids (few heads, few rows) leave most of the chip idle while each block walks its tiles one after the other. Their
// blocks own 128 / G rows instead of 128 and their wavefronts form G groups that take every G-th tile of the walk (a step
// brings in G tiles); the groups' results meet in LDS. G = 2: twice the blocks, half the steps.
// Per-lane values of groups 1.. -> LDS, and back in group 0: slot [group - 1][row wavefront][register][lane].
template <int G, int REGS>
__device__ __forceinline__ float* group_slot(void* smem, int grp, int row_wave, int lane) {
  return reinterpret_cast<float*>(smem) + ((grp - 1) * (4 / G) + row_wave) * (REGS * 64) + lane;
}

// A wavefront's 32 rows of output, [32][D] in its accumulators, on their way out. A lane has four columns of one row at a time, 8
// bytes: stored as they are, an instruction touches 32 rows with 16 bytes each, and the L2 sees every 128-byte line eight times.
// Through LDS (the stages are free by then) each 8 bytes of a lane join those of its neighbours to whole rows. us, as they are ->
// whole rows, forward / backward (samples x tokens, heads): 64-wide 64 x 64, 16 7.8 -> 7.3 / 29.3 -> 26.9; 6 x 381, 12 9.5 -> 9.4 / 20.0 -> 18.9; 8 x
// 512, 16 16.4 -> 15.2 / 43.5 -> 40.0; 8 x 1024, 32 causal 57.6 -> 55.4 / 174 -> 162; 128-wide causal 4 x 1024, 32 56.4 -> 53.4 / 184 -> 166; 4 x 2048, 20
// 111 -> 107 / 360 -> 338; the longer the walk the less: 1 x 8192, 20 451 -> 449 / 1277 -> 1274.
// As they are where that is faster: where a wavefront has fewer than 32 rows (the last, and in causal grids longest, block of 1 x 152, 19,
// causal, forward 64-wide 5.8 / 6.0, 128-wide 7.2 / 7.6), and where no other wavefront of the block has any (SHORT, sequences up to 32:
// 16 x 32, 8 forward 64-wide 4.1 / 4.4, 128-wide 5.0 / 5.5, backward 5.4 / 5.6, 8.1 / 8.3; 8 x 64, 8 3.9 / 3.9, 6.0 / 5.6).
// Gradients that are turned on the way always take their rows through LDS, because the table then is read in whole rows too
// (backward of a gated layer, 16 x 16 tokens, hidden 768: 128-wide 64.5 / 63.2; 6 x 40, hidden 512 61.2 / 59.9).
// SHORT instances hold what one tile with one sub-tile of keys and of queries needs and nothing else (62-143 registers where the others
// take 118-256). Against both sub-tiles and the ring of tiles, forward / backward: 64-wide 16 x 32, 8 4.1 -> 3.5 / 5.4 -> 4.3, 128 x 32, 8 6.7
// -> 5.4 / 20.7 -> 14.4; 128-wide 64 x 16, 8 6.1 -> 4.9 / 19.8 -> 13.3. All attention kernels together 2.0 -> 1.65 MB of code.
template <int D, bool F16, bool SHORT>
struct RowsOut {
  static constexpr int P = D + 4;          // row pitch in elements: 8 bytes more, so that the 8-byte writes of 32 rows meet every bank once
  static constexpr int ELEMS = 32 * P;
  bf16_t* stage;                           // of this wavefront
  int lane, first, rows;                   // first row; of the 32 from there on, so many exist
  __device__ __forceinline__ RowsOut(bf16_t* stage, int lane, int first, int seq) : stage(stage), lane(lane), first(first), rows(seq - first) {}
  // What the lanes of this wavefront have written is there for its other lanes, and they are done with what was there before
  // (its LDS accesses are executed in order; this binds the compiler).
  static __device__ __forceinline__ void meet() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  static __device__ __forceinline__ uint2 turned(uint2 w, const float* __restrict__ table, int pos, int col) {
    float v[4] = {unpack_lo<F16>(w.x), unpack_hi<F16>(w.x), unpack_lo<F16>(w.y), unpack_hi<F16>(w.y)};
    rope_back(v, table, pos, D, col);
    return make_uint2(pack2<F16>(v[0], v[1]), pack2<F16>(v[2], v[3]));
  }
  // value(t, e): column 32 t + 8 (e / 4) + 4 (lane / 32) + e % 4 of row lane % 32. out: the first row, the others `stride` apart.
  // table: the rows are turned back by the rotary angles of their positions.
  template <class Value>
  __device__ __forceinline__ void store(Value&& value, bf16_t* out, int64_t stride, const float* __restrict__ table = nullptr) const {
    const int row = lane & 31, col = 4 * (lane >> 5);
    if (SHORT || (rows < 32 && !table)) {   // (uniform)
      if (row < rows) {
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<uint2*>(out + (row * stride + t * 32 + g * 8 + col)) =
                make_uint2(pack2<F16>(value(t, 4 * g), value(t, 4 * g + 1)), pack2<F16>(value(t, 4 * g + 2), value(t, 4 * g + 3)));
      }
      return;
    }
    if constexpr (!SHORT) {
      meet();
#pragma unroll
      for (int t = 0; t < D / 32; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<uint2*>(stage + row * P + t * 32 + g * 8 + col) =
              make_uint2(pack2<F16>(value(t, 4 * g), value(t, 4 * g + 1)), pack2<F16>(value(t, 4 * g + 2), value(t, 4 * g + 3)));
      meet();
      constexpr int CPR = D / 8, RPI = 64 / CPR;   // 16-byte chunks per row, rows per access
      const int c = (lane % CPR) * 8;
      const auto move = [&](int r) {
        const uint2* p = reinterpret_cast<const uint2*>(stage + r * P + c);
        uint2 w0 = p[0], w1 = p[1];
        if (table) { w0 = turned(w0, table, first + r, c); w1 = turned(w1, table, first + r, c + 4); }   // (uniform)
        *reinterpret_cast<uint4*>(out + (r * stride + c)) = make_uint4(w0.x, w0.y, w1.x, w1.y);
      };
      if (rows >= 32) {   // (uniform)
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) move(i * RPI + lane / CPR);
      } else {
#pragma unroll 1
        for (int r = lane / CPR; r < rows; r += RPI) move(r);
      }
    }
  }
};

__device__ __forceinline__ int visible_keys(const AttnShape& sh, const int32_t* seqlens, int b) {
  int n = sh.seq;
  if (seqlens) { const int v = seqlens[b]; n = v < n ? v : n; n = n < 0 ? 0 : n; }
  return n;
}

// Workgroups are handed to the 8 XCDs round-robin in launch order. The 128-row blocks of one (batch, head)
// all read that head's K and V (or Q and dO), so they are renumbered to sit on the same XCD, next to each
// other in time, and share the tiles through its L2 instead of each fetching them from memory.
// With a causal mask the blocks of a head differ in work by a factor of the block count (query block x sees
// x + 1 key blocks, key block x is seen by nx - x query blocks). `descending` walks a head's blocks from its
// last to its first, for the kernels whose last block is the longest, so that in every kernel the long
// blocks of a head start first and the grid ends on short ones instead of waiting for a long straggler.
struct BlockId { int x, a, b; };
// lpt_heads > 1 (causal shapes): the heads an XCD owns are taken in groups of that many, and a group's blocks are
// walked longest-first ACROSS its heads (all heads' longest blocks, then all second-longest, ...) instead of head by
// head: with head-by-head order a slot that has just finished a short block picks up the next head's longest one
// late, and the grid ends on a ragged tail of long blocks (a list-scheduling estimate puts the head-by-head order
// at 1.15-1.5x the balanced makespan for the causal benchmark shapes, the grouped order at 1.0-1.14x).
// `w`: position in a grid of nx x ny x nz blocks (the launch's own grid unless it holds several).
__device__ __forceinline__ BlockId xcd_local_block(int w, int nx, int ny, int nz, bool descending = false, int lpt_heads = 0) {
  const int total = nx * ny * nz;
  if (total % 8 == 0) w = (w & 7) * (total >> 3) + (w >> 3);
  int xi = w % nx, head = w / nx;
  if (lpt_heads > 1 && total % 8 == 0 && (total >> 3) % nx == 0) {
    const int per_xcd = total >> 3, hpx = per_xcd / nx;   // workgroups and heads of one XCD
    const int xcd = w / per_xcd, wl = w - xcd * per_xcd;
    const int grp = wl / (lpt_heads * nx);
    const int gs = hpx - grp * lpt_heads < lpt_heads ? hpx - grp * lpt_heads : lpt_heads;   // heads in this group
    const int j = wl - grp * lpt_heads * nx;
    xi = j / gs;
    head = xcd * hpx + grp * lpt_heads + j % gs;
  }
  BlockId id;
  id.x = descending ? nx - 1 - xi : xi;
  id.a = head % ny;
  id.b = head / ny;
  return id;
}

// ---- dropout on the attention probabilities ---------------------------------------------------------
// One Philox call yields the 16-bit draws of 8 consecutive keys of one query row (element index
// ((b*heads + a)*S + i)*S + j, block = index >> 3; S % 8 == 0 keeps a block inside a row).
//
// Kernels whose lanes own a query (forward, dQ): a lane holds, per 32-key sub-tile, keys 8g + 4*(lane/32) + e
// (g, e = 0..3) of its query, i.e. half of each of four blocks; lane^32 holds the other halves of the same
// query. Each of the two computes two of the four blocks and hands the partner its half (two words per
// block through the lane exchange). Returns bit r = element r of the 16-element accumulator is kept.
__device__ __forceinline__ uint32_t keep16_query_lane(const DropoutParams& dp, uint64_t row_blk, int kvs, int kc) {
  uint32_t lo[4], hi[4];   // per block g: the word holding e = 0,1 and the word holding e = 2,3 of this lane's half
#pragma unroll
  for (int gg = 0; gg < 2; ++gg) {
    uint32_t o[4];
    const uint64_t blk = row_blk + (uint64_t)((kvs >> 3) + 2 * kc + gg);
    philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), dp.site, dp.layer, dp.key0, dp.key1, o);
    const uint32_t mine0 = kc ? o[2] : o[0], mine1 = kc ? o[3] : o[1];
    const uint32_t send0 = kc ? o[0] : o[2], send1 = kc ? o[1] : o[3];
    const uint32_t rcv0 = (uint32_t)__shfl_xor((int)send0, 32, 64), rcv1 = (uint32_t)__shfl_xor((int)send1, 32, 64);
    lo[gg] = kc ? rcv0 : mine0;          // blocks 0, 1 are computed by the lanes with kc == 0
    hi[gg] = kc ? rcv1 : mine1;
    lo[2 + gg] = kc ? mine0 : rcv0;      // blocks 2, 3 by the lanes with kc == 1
    hi[2 + gg] = kc ? mine1 : rcv1;
  }
  uint32_t bits = 0;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    bits |= ((lo[g] & 0xffffu) >= dp.thr ? 1u : 0u) << (4 * g);
    bits |= ((lo[g] >> 16) >= dp.thr ? 1u : 0u) << (4 * g + 1);
    bits |= ((hi[g] & 0xffffu) >= dp.thr ? 1u : 0u) << (4 * g + 2);
    bits |= ((hi[g] >> 16) >= dp.thr ? 1u : 0u) << (4 * g + 3);
  }
  return bits;
}

// The dK/dV kernel's lanes own a key: element r of a 32-query sub-tile is query qs + 8*(r/4) + 4*(lane/32) + r%4
// against the lane's key, so every element sits in a different block, and the 8 lanes whose keys share a block
// (consecutive lanes) need the same 16 calls. Lane t of such a group computes the calls of elements 2t and
// 2t+1, all eight exchange them through `xch` (per wavefront: [2 halves][4 groups][16 elements][4 words]), and
// every lane picks the draw of its own key out of each call.
__device__ __forceinline__ uint32_t keep16_key_lane(const DropoutParams& dp, uint64_t head_blk, int S8, int qs, int my_kv,
                                                    int lane, uint32_t* xch) {
  const int kc = lane >> 5, t = lane & 7, grp = (lane >> 3) & 7;   // grp: 4 groups per half, halves apart by 4
  uint32_t* slot = xch + grp * 64;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int r = 2 * t + u;
    const int q = qs + 8 * (r >> 2) + 4 * kc + (r & 3);
    uint32_t o[4];
    const uint64_t blk = head_blk + (uint64_t)q * (uint64_t)S8 + (uint64_t)(my_kv >> 3);
    philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), dp.site, dp.layer, dp.key0, dp.key1, o);
    *reinterpret_cast<uint4*>(slot + r * 4) = make_uint4(o[0], o[1], o[2], o[3]);
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS writes of this wavefront done (lgkmcnt 0)
  __builtin_amdgcn_wave_barrier();
  const int word = (my_kv & 7) >> 1, sh16 = 16 * (my_kv & 1);
  uint32_t bits = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) bits |= (((slot[r * 4 + word] >> sh16) & 0xffffu) >= dp.thr ? 1u : 0u) << r;
  __builtin_amdgcn_wave_barrier();      // the next call overwrites the slots
  return bits;
}

__device__ __forceinline__ BlockId xcd_local_block(bool descending, int lpt_heads) {
  return xcd_local_block(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x, gridDim.y, gridDim.z, descending, lpt_heads);
}

// =================================== forward =====================================================
// LDS stages of the forward kernel's K/V ring. Two: with three or four the forward pass is 10-40 % slower on
// every shape with more than two workgroups per CU (the LDS footprint costs resident workgroups, and those,
// not the depth of the prefetch, are what hides the latencies here) and unchanged on the others.
template <int D> constexpr int FWD_STAGES = 2;

template <int D, bool DROP, bool F16, int G, bool SHORT>
__global__ __launch_bounds__(256) void attn_fwd_bf16_kernel(AttnShape sh, const bf16_t* __restrict__ qkv,
                                                            const int32_t* __restrict__ seqlens,
                                                            bf16_t* __restrict__ out, float* __restrict__ lse) {
  constexpr int NS = D / 16, NT = D / 32;
  constexpr int TE = Tile<D>::ELEMS;
  constexpr int RB = 128 / G;   // rows of the block
  constexpr int SUBS = SHORT ? 1 : 2;   // sub-tiles of 32 keys that hold any
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];  // [2][G][K tile | V tile]
  const int S = sh.seq, H = sh.hidden;
  const BlockId blk = xcd_local_block(sh.causal != 0, sh.lpt_heads);
  const int b = blk.b, a = blk.a, q_base = blk.x * RB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kc = lane >> 5;
  const int row_wave = wave % (4 / G), grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / (4 / G));
  const int fr_base = rows_base<D>(lane), ft_base = tr_base<D>(lane);
  const int64_t rs = 3 * (int64_t)H;
  const bf16_t* base = qkv + (int64_t)b * S * rs + a * D;
  const int kv_len = visible_keys(sh, seqlens, b);
  int kv_end = kv_len;
  if (sh.causal && q_base + RB < kv_end) kv_end = q_base + RB;
  const int n_tiles = (kv_end + 63) / 64;
  const int my_q = q_base + 32 * row_wave + (lane & 31);
  const int q_ld = my_q < S ? my_q : S - 1;
  const int wave_q_min = q_base + 32 * row_wave, wave_q_max = wave_q_min + 31;
  const float scale = rsqrtf((float)D), sl2 = LOG2E * scale;

  bf16x8_t qf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) qf[s] = *reinterpret_cast<const bf16x8_t*>(base + q_ld * rs + 16 * s + 8 * kc);

  f32x16_t o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
  float m = -INFINITY, l = 0.f;   // running maximum (raw score units) and sum of this lane's half row
  // G > 1: the groups tell each other the maxima of a step's tiles, so that every tile's probabilities are taken (and
  // rounded) against the maximum of all keys up to it, as if one group walked the tiles in order. `seen`: of all steps so far.
  float seen = -INFINITY;
  float* maxima = reinterpret_cast<float*>(smem + FWD_STAGES<D> * G * 2 * TE) + row_wave * 32 + (lane & 31);   // [G][RB]
  const uint64_t row_blk = ((((uint64_t)b * sh.heads + a) * S + (uint64_t)q_ld) * (uint64_t)S) >> 3;   // DROP: block of key 0

  // K and V tiles of 64 keys: direct loads into two LDS stages, tile t+1 on its way while tile t is computed
  TileDirect<D> td;
  td.init(lane, __builtin_amdgcn_readfirstlane(wave), (unsigned)(rs * 2));
  const bf16_t* kbase = base + H;
  const bf16_t* vbase = base + 2 * H;
  const int64_t total_elems = (int64_t)sh.batch * S * rs;
  const unsigned kbytes = (unsigned)((total_elems - (kbase - qkv)) * 2), vbytes = (unsigned)((total_elems - (vbase - qkv)) * 2);
  auto issue_step = [&](int stage, int step) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int t = step * G + g;
      if (t >= n_tiles) break;   // uniform
      const unsigned row0_bytes = (unsigned)t * 64u * (unsigned)(rs * 2);
      td.issue(kbase, kbytes, smem + (stage * G + g) * 2 * TE, row0_bytes);
      td.issue(vbase, vbytes, smem + (stage * G + g) * 2 * TE + TE, row0_bytes);
    }
  };
  auto compute = [&](int stage, int step) {
    const int t = step * G + grp, kv0 = t * 64;
    const bool mine = !((G > 1 && t >= n_tiles) || (sh.causal && kv0 > wave_q_max));   // else every key of the tile lies in this wave's future
    if (G == 1 && !mine) return;
    const bf16_t* kt = smem + (stage * G + grp) * 2 * TE;
    const bf16_t* vt = kt + TE;
    f32x16_t sc[SUBS];
    float mx = -INFINITY;
    if (mine) {
#pragma unroll
      for (int i = 0; i < SUBS; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[i][r] = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s)
          sc[i] = mfma16<F16>(frag_rows<D>(kt, fr_base, i * 32, s), qf[s], sc[i]);
      }
      if ((kv0 + 64 > kv_len) || (sh.causal && kv0 + 63 > wave_q_min)) {   // tile crosses a mask boundary
#pragma unroll
        for (int i = 0; i < SUBS; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int kv = kv0 + i * 32 + acc_row(r, lane);
            const bool hide = (kv >= kv_len) | ((sh.causal != 0) & (kv > my_q));
            sc[i][r] = hide ? -INFINITY : sc[i][r];
          }
      }
#pragma unroll
      for (int i = 0; i < SUBS; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[i][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    }
    float before = m;   // maximum of all keys in front of this tile
    if constexpr (G > 1) {
      if (kc == 0) maxima[grp * RB] = mx;
      wait_loads_and_lds<63>();
      block_barrier();
      before = seen;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float v = maxima[g * RB];
        before = g < grp ? fmaxf(before, v) : before;
        seen = fmaxf(seen, v);
      }
      if (!mine) return;
    }
    const float m_new = fmaxf(before, mx);
    if (__any(m_new > m)) {   // some row's maximum grew: rescale what has been accumulated
      const float alpha = __builtin_amdgcn_exp2f((m - m_new) * sl2);   // m = -inf gives 0; m = m_new gives 1
      const float al = (m_new == -INFINITY) ? 0.f : alpha;             // avoids inf - inf for rows still empty
      l *= al;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= al;
      m = m_new;
    }
    const float mb = (m == -INFINITY) ? 0.f : m * sl2;
#pragma unroll
    for (int i = 0; i < SUBS; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sc[i][r], sl2, -mb));
        sc[i][r] = p;
        l += p;
      }
    if (DROP) {   // the row sum above is the softmax denominator: dropout acts on the normalised probabilities
#pragma unroll
      for (int i = 0; i < SUBS; ++i) {
        const uint32_t keep = keep16_query_lane(sh.drop, row_blk, kv0 + 32 * i, kc);
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[i][r] = ((keep >> r) & 1u) ? sc[i][r] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < SUBS; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bf16x8_t pf = pack8<F16>(sc[i], h);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          o[t] = mfma16<F16>(frag_tr<D>(vt, ft_base, i * 32 + 16 * h, t), pf, o[t]);
      }
  };
  if constexpr (SHORT) one_tile(n_tiles, issue_step, compute);
  else tile_ring<FWD_STAGES<D>, G * 2 * TileDirect<D>::MINE>((n_tiles + G - 1) / G, issue_step, compute);
  if constexpr (G > 1) {   // (the ring ends behind a barrier: the stages are free)
    static_assert(FWD_STAGES<D> == 2, "partly filled steps are waited for as a whole");
    constexpr int REGS = NT * 16 + 2;
    if (grp > 0) {
      float* p = group_slot<G, REGS>(smem, grp, row_wave, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) p[(t * 16 + r) * 64] = o[t][r];
      p[NT * 16 * 64] = m;
      p[(NT * 16 + 1) * 64] = l;
    }
    __syncthreads();
    if (grp > 0) return;
    for (int g = 1; g < G; ++g) {
      const float* p = group_slot<G, REGS>(smem, g, row_wave, lane);
      const float m2 = p[NT * 16 * 64], m_new = fmaxf(m, m2);
      const float mine = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - m_new) * sl2);
      const float theirs = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m2 - m_new) * sl2);
      l = l * mine + p[(NT * 16 + 1) * 64] * theirs;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] = o[t][r] * mine + p[(t * 16 + r) * 64] * theirs;
      m = m_new;
    }
  }

  const float l_tot = l + __shfl_xor(l, 32, 64);
  const float inv = l_tot > 0.f ? (DROP ? sh.drop.scale : 1.f) / l_tot : 0.f;
  // (a group's wavefront writes over its own slot of what the groups handed it)
  const RowsOut<D, F16, SHORT> rows(smem + row_wave * (G > 1 ? (NT * 16 + 2) * 128 : RowsOut<D, F16, SHORT>::ELEMS), lane, wave_q_min, S);
  if (rows.rows <= 0) return;
  rows.store([&](int t, int e) { return o[t][e] * inv; }, out + ((int64_t)b * S + rows.first) * H + a * D, H);
  if (my_q < S) {
    if (kc == 0) lse[((int64_t)b * sh.heads + a) * S + my_q] = l_tot > 0.f ? m * scale + __logf(l_tot) : -INFINITY;
  }
}

// ============================ backward: delta = rowsum(dO * O) ===================================
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_delta_kernel(AttnShape sh, const T* __restrict__ o,
                                                         const T* __restrict__ dout, float* __restrict__ delta) {
  // 8 lanes per (token, head); each lane D/8 elements
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t item = gid >> 3;
  const int sub = (int)(gid & 7);
  const int64_t total = (int64_t)sh.batch * sh.seq * sh.heads;
  float s = 0.f;
  int64_t tok = 0;
  int a = 0;
  if (item < total) {
    tok = item / sh.heads;
    a = (int)(item % sh.heads);
    const int64_t off = tok * sh.hidden + a * D + sub * (D / 8);
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
      float x[8], y[8];
      load8(o + off + i * 8, x);
      load8(dout + off + i * 8, y);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += x[j] * y[j];
    }
  }
  s += __shfl_xor(s, 1, 64);
  s += __shfl_xor(s, 2, 64);
  s += __shfl_xor(s, 4, 64);
  if (item < total && sub == 0) {
    const int64_t bb = tok / sh.seq, i = tok % sh.seq;
    delta[(bb * sh.heads + a) * sh.seq + i] = s;
  }
}

// ============================ backward: dK, dV per key tile ======================================
// LDS stages of the dK/dV kernel's Q/dO ring. Two: 128-wide heads run one workgroup per CU whatever the LDS
// footprint (registers), so more stages would be free there, but three and four were measured equal to two
// (the 1300-2600 cycles a tile step spends outside its ~4100 cycles of compute are the wavefronts waiting
// for each other at the barrier, not for the next tile).
template <int D> constexpr int DKDV_STAGES = 2;

// OWN_DELTA: delta = rowsum(dO * O) of each query tile is computed here (see attn_bwd_both_kernel) instead of read.
template <int D, bool DROP, bool F16, bool OWN_DELTA, int G, bool SHORT>
__device__ __forceinline__ void attn_bwd_dkdv_block(const BlockId blk, const AttnShape& sh, const bf16_t* __restrict__ qkv,
                                                    const int32_t* __restrict__ seqlens, const bf16_t* __restrict__ out,
                                                    const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                    const float* __restrict__ delta, bf16_t* __restrict__ dqkv) {
  constexpr int NS = D / 16, NT = D / 32;
  constexpr int TE = Tile<D>::ELEMS;
  constexpr int TILE = 2 * TE + 256;    // bf16 units: Q tile, dO tile, 64 lse + 64 delta floats
  constexpr int STAGE = G * TILE, RB = 128 / G;
  constexpr int FB = 4;                 // k-steps of fragment prefetch (register budget: 8 FB registers)
  constexpr int NSTG = DKDV_STAGES<D>;
  constexpr bool ACC_A = (D == 128);    // dK/dV accumulators in AGPRs (see mfma16_agpr)
  constexpr bool PIPE = ACC_A && !DROP && !SHORT; // hand-pipelined sub-tiles for tiles without a mask boundary (see compute)
  static_assert(!PIPE || (NS == 8 && NT == 4), "the pipelined rounds are written for D = 128");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int S = sh.seq, H = sh.hidden;
  const int b = blk.b, a = blk.a, kv_base = blk.x * RB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kc = lane >> 5;
  const int row_wave = wave % (4 / G), grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / (4 / G));
  const int fr_base = rows_base<D>(lane), ft_base = tr_base<D>(lane);
  const int64_t rs = 3 * (int64_t)H;
  const bf16_t* base = qkv + (int64_t)b * S * rs + a * D;
  const bf16_t* dobase = dout + (int64_t)b * S * H + a * D;
  const float* lse_row = lse + ((int64_t)b * sh.heads + a) * S;
  const float* delta_row = delta + ((int64_t)b * sh.heads + a) * S;
  const int kv_len = visible_keys(sh, seqlens, b);
  const int my_kv = kv_base + 32 * row_wave + (lane & 31);
  const int kv_ld = my_kv < S ? my_kv : S - 1;
  const int wave_kv_min = kv_base + 32 * row_wave;
  const bool wave_kv_edge = wave_kv_min + 32 > kv_len;   // some of this wave's keys are hidden
  // DROP: block index of (query 0, key 0) of this head, and this wavefront's exchange area behind the stages
  const uint64_t head_blk = ((((uint64_t)b * sh.heads + a) * S) * (uint64_t)S) >> 3;
  uint32_t* xch = reinterpret_cast<uint32_t*>(smem + DKDV_STAGES<D> * STAGE) + wave * 512;
  const float scale = rsqrtf((float)D), sl2 = LOG2E * scale;

  bf16x8_t kf[NS], vf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    kf[s] = *reinterpret_cast<const bf16x8_t*>(base + H + kv_ld * rs + 16 * s + 8 * kc);
    vf[s] = *reinterpret_cast<const bf16x8_t*>(base + 2 * H + kv_ld * rs + 16 * s + 8 * kc);
  }
  f32x16_t dk[NT], dv[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[t][r] = dv[t][r] = 0.f;

  const int q_first = sh.causal ? (kv_base / 64) : 0;
  const int n_tiles = (kv_base < kv_len) ? (S + 63) / 64 - q_first : 0;  // nothing to do for fully hidden keys
  const int stat_row = tid & 63;
  // threads 0..63 carry lse, threads 64..127 delta, threads 128..255 duplicate them (same values to the same
  // slots, so no thread is special) or the second tile of a step; OWN_DELTA: every 64 threads lse, of the step's tiles in turn. The value is only
  // touched when it is stored to LDS after the step's compute, so the load stays in flight like the tile loads.
  const float* stat_src = OWN_DELTA || (tid & 127) < 64 ? lse_row : delta_row;
  const float stat_mul = OWN_DELTA || (tid & 127) < 64 ? LOG2E : 1.0f;
  const int stat_tile = OWN_DELTA ? (tid >> 6) % G : (tid >> 7) % G;
  auto load_stats = [&](int step) -> float {
    int q = (q_first + step * G + stat_tile) * 64 + stat_row;
    q = q < S ? q : S - 1;
    return stat_src[q];
  };
  // OWN_DELTA: four threads per query row, D / 4 elements of O and dO each, requested a tile ahead like the rest
  struct DeltaRows { bf16x8_t o[D / 32], d[D / 32]; };
  const bf16_t* obase = out + (int64_t)b * S * H + a * D;
  auto load_delta_rows = [&](int t, DeltaRows& r) {
    int q = (q_first + t) * 64 + (tid >> 2);
    q = q < S ? q : S - 1;
    const int64_t at = (int64_t)q * H + (tid & 3) * (D / 4);
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      r.o[k] = *reinterpret_cast<const bf16x8_t*>(obase + at + 8 * k);
      r.d[k] = *reinterpret_cast<const bf16x8_t*>(dobase + at + 8 * k);
    }
  };
  auto store_delta = [&](int stage, int g, const DeltaRows& r) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < D / 32; ++k) {
      const u32x4_t ow = __builtin_bit_cast(u32x4_t, r.o[k]), dw = __builtin_bit_cast(u32x4_t, r.d[k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v = fmaf(unpack_lo<F16>(ow[e]), unpack_lo<F16>(dw[e]), v);
        v = fmaf(unpack_hi<F16>(ow[e]), unpack_hi<F16>(dw[e]), v);
      }
    }
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    if ((tid & 3) == 0) reinterpret_cast<float*>(smem + stage * STAGE + g * TILE + 2 * TE)[64 + (tid >> 2)] = v;
  };
  // Q and dO tiles of 64 queries: direct loads into two LDS stages, tile t+1 on its way while tile t is computed
  TileDirect<D> tq, tdo;
  tq.init(lane, __builtin_amdgcn_readfirstlane(wave), (unsigned)(rs * 2));
  tdo.init(lane, __builtin_amdgcn_readfirstlane(wave), (unsigned)(H * 2));
  const unsigned qbytes = (unsigned)(((int64_t)sh.batch * S * rs - (base - qkv)) * 2);
  const unsigned dbytes = (unsigned)(((int64_t)sh.batch * S * H - (dobase - dout)) * 2);
  auto issue_step = [&](int stage, int step) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int t = step * G + g;
      if (t >= n_tiles) break;   // uniform
      const unsigned q0 = (unsigned)(q_first + t) * 64u;
      tq.issue(base, qbytes, smem + stage * STAGE + g * TILE, q0 * (unsigned)(rs * 2));
      tdo.issue(dobase, dbytes, smem + stage * STAGE + g * TILE + TE, q0 * (unsigned)(H * 2));
    }
  };
  auto store_stats = [&](int stage, float v) { reinterpret_cast<float*>(smem + stage * STAGE + stat_tile * TILE + 2 * TE)[OWN_DELTA ? tid & 63 : tid & 127] = v * stat_mul; };
  auto compute = [&](int stage, int step) {
    if (G > 1 && step * G + grp >= n_tiles) return;
    const int q0 = (q_first + step * G + grp) * 64;
    const bf16_t* qtile = smem + stage * STAGE + grp * TILE;
    const bf16_t* dtile = qtile + TE;
    const float* stats = reinterpret_cast<const float*>(qtile + 2 * TE);
    if constexpr (PIPE) {
      // One wavefront per SIMD (128-wide heads): nothing else runs while this wavefront does the softmax
      // arithmetic of a sub-tile, so for tiles without a mask boundary the two sub-tiles are software-
      // pipelined by hand: every MFMA is followed by the vector work of one score element of the OTHER
      // sub-tile, which issues while the matrix core is busy.
      //   scores(0);  scores(1) || softmax(0);  dV,dK(0) || softmax(1);  dV,dK(1)
      const bool interior = !wave_kv_edge && q0 + 64 <= S && !(sh.causal && q0 < wave_kv_min + 32);
      if (interior) {
        f32x16_t sc0, dp0, sc1, dp1;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc0[r] = dp0[r] = sc1[r] = dp1[r] = 0.f;
        // scores of sub-tile 0
#pragma unroll
        for (int s0 = 0; s0 < NS; s0 += FB) {
          bf16x8_t fq[FB], fd[FB];
#pragma unroll
          for (int s = 0; s < FB; ++s) {
            fq[s] = frag_rows<D>(qtile, fr_base, 0, s0 + s);
            fd[s] = frag_rows<D>(dtile, fr_base, 0, s0 + s);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int s = 0; s < FB; ++s) {
            sc0 = mfma16<F16>(fq[s], kf[s0 + s], sc0);
            dp0 = mfma16<F16>(fd[s], vf[s0 + s], dp0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        // The 16 score elements of a sub-tile go through three steps each - a = sc * scale - lse; p = exp2(a);
        // sc = p, dp = p * (dp - delta) - and run as a pipeline beside 16 MFMAs of the OTHER sub-tile: the slot of
        // MFMA s holds step 1 of element s + 1, step 2 of element s and step 3 of element s - 1, so no vector
        // instruction waits for the result of the one in front of it (one element's steps back to back are a
        // dependent chain whose latencies nothing hides with a single wavefront per SIMD). The row statistics of
        // four elements (one float4 each of lse and delta) are read from LDS three slots ahead of their first use.
        auto pick = [](const float4& v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
        auto soft_slots = [&](f32x16_t& sc, f32x16_t& dp, const float* srow, auto&& mfma_slot) {
          float4 l[2], d[2];
          l[0] = *reinterpret_cast<const float4*>(srow + 4 * kc);
          d[0] = *reinterpret_cast<const float4*>(srow + 64 + 4 * kc);
          float a_next = fmaf(sc[0], sl2, -l[0].x), p_prev = 0.f;
#pragma unroll
          for (int s = 0; s < 16; ++s) {
            const int g = s >> 2, e = s & 3;
            if (e == 1 && g + 1 < 4) {
              l[(g + 1) & 1] = *reinterpret_cast<const float4*>(srow + (g + 1) * 8 + 4 * kc);
              d[(g + 1) & 1] = *reinterpret_cast<const float4*>(srow + 64 + (g + 1) * 8 + 4 * kc);
            }
            mfma_slot(s);
            const float a_cur = a_next;
            if (s + 1 < 16) a_next = fmaf(sc[s + 1], sl2, -pick(l[((s + 1) >> 2) & 1], (s + 1) & 3));
            const float p_cur = __builtin_amdgcn_exp2f(a_cur);
            if (s > 0) {
              sc[s - 1] = p_prev;
              dp[s - 1] = p_prev * (dp[s - 1] - pick(d[((s - 1) >> 2) & 1], (s - 1) & 3));
            }
            p_prev = p_cur;
            __builtin_amdgcn_sched_barrier(0);
          }
          sc[15] = p_prev;
          dp[15] = p_prev * (dp[15] - d[1].w);
        };
        // scores of sub-tile 1 (two k-steps = four MFMAs per round) || softmax of sub-tile 0
        {
          bf16x8_t fq[2][2], fd[2][2];
#pragma unroll
          for (int k = 0; k < 2; ++k) { fq[0][k] = frag_rows<D>(qtile, fr_base, 32, k); fd[0][k] = frag_rows<D>(dtile, fr_base, 32, k); }
          soft_slots(sc0, dp0, stats, [&](int s) {
            const int g = s >> 2, e = s & 3, cur = g & 1;
            if (e == 0 && g + 1 < NS / 2) {
#pragma unroll
              for (int k = 0; k < 2; ++k) {
                fq[cur ^ 1][k] = frag_rows<D>(qtile, fr_base, 32, 2 * g + 2 + k);
                fd[cur ^ 1][k] = frag_rows<D>(dtile, fr_base, 32, 2 * g + 2 + k);
              }
            }
            // (a compiler-visible MFMA is a pure operation that the instruction selector may move past scheduling
            // barriers - all sixteen ended up behind the softmax; the empty statement pins its result to this slot)
            if (e == 0) { sc1 = mfma16<F16>(fq[cur][0], kf[2 * g], sc1); pin_here(sc1); }
            else if (e == 1) { dp1 = mfma16<F16>(fd[cur][0], vf[2 * g], dp1); pin_here(dp1); }
            else if (e == 2) { sc1 = mfma16<F16>(fq[cur][1], kf[2 * g + 1], sc1); pin_here(sc1); }
            else { dp1 = mfma16<F16>(fd[cur][1], vf[2 * g + 1], dp1); pin_here(dp1); }
          });
        }
        // dV, dK of sub-tile 0 (four MFMAs per round) || softmax of sub-tile 1
        {
          const bf16x8_t pf[2] = {pack8<F16>(sc0, 0), pack8<F16>(sc0, 1)}, dsf[2] = {pack8<F16>(dp0, 0), pack8<F16>(dp0, 1)};
          bf16x8_t td[2][2], tq[2][2];   // [round parity][column block of the round]
#pragma unroll
          for (int k = 0; k < 2; ++k) { td[0][k] = frag_tr<D>(dtile, ft_base, 0, k); tq[0][k] = frag_tr<D>(qtile, ft_base, 0, k); }
          soft_slots(sc1, dp1, stats + 32, [&](int s) {   // round g: half h = g / 2, column blocks t = 2 (g % 2), 2 (g % 2) + 1
            const int g = s >> 2, e = s & 3, cur = g & 1, h = g >> 1, t0 = 2 * (g & 1);
            if (e == 0 && g + 1 < 4) {
              const int hn = (g + 1) >> 1, tn = 2 * ((g + 1) & 1);
#pragma unroll
              for (int k = 0; k < 2; ++k) {
                td[cur ^ 1][k] = frag_tr<D>(dtile, ft_base, 16 * hn, tn + k);
                tq[cur ^ 1][k] = frag_tr<D>(qtile, ft_base, 16 * hn, tn + k);
              }
            }
            if (e == 0) mfma16_agpr<F16>(dv[t0], td[cur][0], pf[h]);
            else if (e == 1) mfma16_agpr<F16>(dk[t0], tq[cur][0], dsf[h]);
            else if (e == 2) mfma16_agpr<F16>(dv[t0 + 1], td[cur][1], pf[h]);
            else mfma16_agpr<F16>(dk[t0 + 1], tq[cur][1], dsf[h]);
          });
        }
        // dV, dK of sub-tile 1
        {
          const bf16x8_t pf[2] = {pack8<F16>(sc1, 0), pack8<F16>(sc1, 1)}, dsf[2] = {pack8<F16>(dp1, 0), pack8<F16>(dp1, 1)};
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            bf16x8_t td[NT], tq[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              td[t] = frag_tr<D>(dtile, ft_base, 32 + 16 * h, t);
              tq[t] = frag_tr<D>(qtile, ft_base, 32 + 16 * h, t);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NT; ++t) { mfma16_agpr<F16>(dv[t], td[t], pf[h]); mfma16_agpr<F16>(dk[t], tq[t], dsf[h]); }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        return;
      }
    }
#pragma unroll
    for (int i = 0; i < (SHORT ? 1 : 2); ++i) {   // (SHORT: the second 32 queries do not exist)
      const int qs = q0 + i * 32;
      if (sh.causal && qs + 31 < wave_kv_min) continue;  // every query of this sub-tile precedes my keys
      f32x16_t sc, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = dp[r] = 0.f;
      // Fragments are requested FB k-steps ahead of the MFMAs that use them and the order is pinned: left to
      // itself the scheduler reuses one register set for all fragments, and every MFMA then waits out the
      // full LDS latency of its own read.
#pragma unroll
      for (int s0 = 0; s0 < NS; s0 += FB) {
        bf16x8_t fq[FB], fd[FB];
#pragma unroll
        for (int s = 0; s < FB; ++s) {
          fq[s] = frag_rows<D>(qtile, fr_base, i * 32, s0 + s);
          fd[s] = frag_rows<D>(dtile, fr_base, i * 32, s0 + s);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < FB; ++s) {
          sc = mfma16<F16>(fq[s], kf[s0 + s], sc);
          dp = mfma16<F16>(fd[s], vf[s0 + s], dp);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // the first operands of the dV / dK products do not depend on the softmax: on their way during it
      bf16x8_t td0[NT], tq0[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        td0[t] = frag_tr<D>(dtile, ft_base, i * 32, t);
        tq0[t] = frag_tr<D>(qtile, ft_base, i * 32, t);
      }
      __builtin_amdgcn_sched_barrier(0);
      const bool edge = wave_kv_edge || (qs + 32 > S) || (sh.causal && qs < wave_kv_min + 32);
      uint32_t keep = 0xffffu;
      if (DROP) keep = keep16_key_lane(sh.drop, head_blk, S >> 3, qs, kv_ld, lane, xch);
      // two instances of the element loop, chosen by a wavefront-uniform branch: interior tiles carry no mask
      // code at all (as one loop the compiler turns the test into a compare and a select on every element)
      auto elements = [&](auto edge_tag) {
        constexpr bool EDGE = decltype(edge_tag)::value;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 l4 = *reinterpret_cast<const float4*>(stats + i * 32 + g * 8 + 4 * kc);
          const float4 d4 = *reinterpret_cast<const float4*>(stats + 64 + i * 32 + g * 8 + 4 * kc);
          const float ls[4] = {l4.x, l4.y, l4.z, l4.w}, ds[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = 4 * g + e;
            float p = __builtin_amdgcn_exp2f(fmaf(sc[r], sl2, -ls[e]));
            if (EDGE) {   // the per-lane part is a select, not a branch
              const int q = qs + g * 8 + 4 * kc + e;
              const bool hide = (my_kv >= kv_len) | (q >= S) | ((sh.causal != 0) & (my_kv > q));
              p = hide ? 0.f : p;
            }
            float dpr = dp[r];
            if (DROP) {
              const bool kept = (keep >> r) & 1u;
              dpr = kept ? dpr * sh.drop.scale : 0.f;          // dP = keep * (dO V^T) / (1 - p)
              sc[r] = kept ? p * sh.drop.scale : 0.f;          // what multiplied V in the forward pass
            } else {
              sc[r] = p;
            }
            dp[r] = p * (dpr - ds[e]);
          }
        }
      };
      if (edge) elements(std::true_type{});
      else elements(std::false_type{});
      {
        const bf16x8_t pf0 = pack8<F16>(sc, 0), dsf0 = pack8<F16>(dp, 0), pf1 = pack8<F16>(sc, 1), dsf1 = pack8<F16>(dp, 1);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8_t td1[NT], tq1[NT];   // second half's operands, requested in front of the first half's MFMAs
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          td1[t] = frag_tr<D>(dtile, ft_base, i * 32 + 16, t);
          tq1[t] = frag_tr<D>(qtile, ft_base, i * 32 + 16, t);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if constexpr (ACC_A) { mfma16_agpr<F16>(dv[t], td0[t], pf0); mfma16_agpr<F16>(dk[t], tq0[t], dsf0); }
          else { dv[t] = mfma16<F16>(td0[t], pf0, dv[t]); dk[t] = mfma16<F16>(tq0[t], dsf0, dk[t]); }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if constexpr (ACC_A) { mfma16_agpr<F16>(dv[t], td1[t], pf1); mfma16_agpr<F16>(dk[t], tq1[t], dsf1); }
          else { dv[t] = mfma16<F16>(td1[t], pf1, dv[t]); dk[t] = mfma16<F16>(tq1[t], dsf1, dk[t]); }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Ring of NSTG stages: step it + NSTG - 1 is requested while step it is computed; the statistics of step
  // it + 1 travel through registers and are requested BEFORE that step's tile loads, so that waiting for
  // them (loads complete in issue order) leaves the younger tile loads in flight. LPT = tile loads per step
  // that every wavefront issues.
  const int n_steps = (n_tiles + G - 1) / G;
  if constexpr (SHORT) {
    DeltaRows rows;
    if (OWN_DELTA && n_tiles > 0) load_delta_rows(0, rows);
    const float stat = load_stats(0);
    one_tile(n_tiles, [&](int, int) {
      issue_step(0, 0);
      store_stats(0, stat);
      if constexpr (OWN_DELTA) store_delta(0, 0, rows);
    }, compute);
  } else if (n_steps > 0) {
    constexpr int LPT = G * 2 * TileDirect<D>::MINE;
    static_assert(G == 1 || NSTG == 2, "partly filled steps are waited for as a whole");
    DeltaRows rows[G];
    const float stat0 = load_stats(0);
    if constexpr (OWN_DELTA) {
#pragma unroll
      for (int g = 0; g < G; ++g) load_delta_rows(g, rows[g]);
    }
#pragma unroll
    for (int t = 0; t < NSTG - 1; ++t)
      if (t < n_steps) issue_step(t, t);
    store_stats(0, stat0);
    if constexpr (OWN_DELTA) {
#pragma unroll
      for (int g = 0; g < G; ++g) store_delta(0, g, rows[g]);
    }
    if (n_steps >= NSTG - 1) wait_loads_and_lds<(NSTG - 2) * LPT>();
    else wait_loads_and_lds<0>();
    block_barrier();
    for (int it0 = 0; it0 < n_steps; it0 += NSTG) {
#pragma unroll
      for (int st = 0; st < NSTG; ++st) {   // (stages at compile time, as in tile_ring)
        const int it = it0 + st, next = (st + 1) % NSTG;
        if (it >= n_steps) break;           // uniform
        const bool more = it + 1 < n_steps, far = it + NSTG - 1 < n_steps;
        float next_stat = 0.f;
        if (more) {
          next_stat = load_stats(it + 1);
          if constexpr (OWN_DELTA) {
#pragma unroll
            for (int g = 0; g < G; ++g) load_delta_rows((it + 1) * G + g, rows[g]);
          }
        }
        if (far) issue_step((st + NSTG - 1) % NSTG, it + NSTG - 1);   // that stage was last read before the barrier that ended step it - 1
        compute(st, it);
        if (more) {
          store_stats(next, next_stat);
          if constexpr (OWN_DELTA) {
#pragma unroll
            for (int g = 0; g < G; ++g) store_delta(next, g, rows[g]);
          }
        }
        if (far) wait_loads_and_lds<(NSTG - 2) * LPT>();
        else wait_loads_and_lds<0>();
        block_barrier();
      }
    }
  }

  if (ACC_A) agpr_results_ready();
  if constexpr (G > 1) {   // (behind the last barrier: the stages are free)
    constexpr int REGS = 2 * NT * 16;
    if (grp > 0) {
      float* p = group_slot<G, REGS>(smem, grp, row_wave, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { p[(t * 16 + r) * 64] = dk[t][r]; p[((NT + t) * 16 + r) * 64] = dv[t][r]; }
    }
    __syncthreads();
    if (grp > 0) return;
    for (int g = 1; g < G; ++g) {
      const float* p = group_slot<G, REGS>(smem, g, row_wave, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dk[t][r] += p[(t * 16 + r) * 64]; dv[t][r] += p[((NT + t) * 16 + r) * 64]; }
    }
  }
  const RowsOut<D, F16, SHORT> rows(smem + row_wave * (G > 1 ? 2 * NT * 16 * 128 : RowsOut<D, F16, SHORT>::ELEMS), lane,
                                    SHORT ? wave_kv_min : __builtin_amdgcn_readfirstlane(wave_kv_min), S);
  if (rows.rows <= 0) return;
  bf16_t* krow = dqkv + ((int64_t)b * S + rows.first) * rs + H + a * D;
  rows.store([&](int t, int e) { return dk[t][e] * scale; }, krow, rs, sh.rope);
  rows.store([&](int t, int e) { return dv[t][e]; }, krow + H, rs);
}

// ============================ backward: dQ per query tile ========================================
template <int D, bool DROP, bool F16, int G, bool SHORT>
__device__ __forceinline__ void attn_bwd_dq_block(const BlockId blk, const AttnShape& sh, const bf16_t* __restrict__ qkv,
                                                  const int32_t* __restrict__ seqlens, const bf16_t* __restrict__ out,
                                                  const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                  float* __restrict__ delta, bf16_t* __restrict__ dqkv) {
  constexpr int NS = D / 16, NT = D / 32;
  constexpr int TE = Tile<D>::ELEMS;
  constexpr int RB = 128 / G;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];  // [2][G][K tile | V tile]
  const int S = sh.seq, H = sh.hidden;
  const int b = blk.b, a = blk.a, q_base = blk.x * RB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, kc = lane >> 5;
  const int row_wave = wave % (4 / G), grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / (4 / G));
  const int fr_base = rows_base<D>(lane), ft_base = tr_base<D>(lane);
  const int64_t rs = 3 * (int64_t)H;
  const bf16_t* base = qkv + (int64_t)b * S * rs + a * D;
  const int kv_len = visible_keys(sh, seqlens, b);
  int kv_end = kv_len;
  if (sh.causal && q_base + RB < kv_end) kv_end = q_base + RB;
  const int n_tiles = (kv_end + 63) / 64;
  const int my_q = q_base + 32 * row_wave + (lane & 31);
  const int q_ld = my_q < S ? my_q : S - 1;
  const int wave_q_min = q_base + 32 * row_wave, wave_q_max = wave_q_min + 31;
  const float scale = rsqrtf((float)D), sl2 = LOG2E * scale;

  bf16x8_t qf[NS], df[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    qf[s] = *reinterpret_cast<const bf16x8_t*>(base + q_ld * rs + 16 * s + 8 * kc);
    df[s] = *reinterpret_cast<const bf16x8_t*>(dout + ((int64_t)b * S + q_ld) * H + a * D + 16 * s + 8 * kc);
  }
  const float my_lse2 = lse[((int64_t)b * sh.heads + a) * S + q_ld] * LOG2E;
  const uint64_t row_blk = ((((uint64_t)b * sh.heads + a) * S + (uint64_t)q_ld) * (uint64_t)S) >> 3;   // DROP: block of key 0
  // delta = rowsum(dO * O) of this lane's query row: the lane holds half of the row's dO, lane^32 the other
  // half. It is also written out for the dK/dV kernel, which runs after this one.
  float my_delta = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const bf16x8_t of = *reinterpret_cast<const bf16x8_t*>(out + ((int64_t)b * S + q_ld) * H + a * D + 16 * s + 8 * kc);
    {
      const u32x4_t ow = __builtin_bit_cast(u32x4_t, of), dw = __builtin_bit_cast(u32x4_t, df[s]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        my_delta = fmaf(unpack_lo<F16>(ow[e]), unpack_lo<F16>(dw[e]), my_delta);
        my_delta = fmaf(unpack_hi<F16>(ow[e]), unpack_hi<F16>(dw[e]), my_delta);
      }
    }
  }
  my_delta += __shfl_xor(my_delta, 32, 64);
  if (delta != nullptr && kc == 0 && grp == 0 && my_q < S) delta[((int64_t)b * sh.heads + a) * S + my_q] = my_delta;
  f32x16_t dq[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[t][r] = 0.f;

  // K and V tiles of 64 keys: direct loads into two LDS stages, tile t+1 on its way while tile t is computed
  TileDirect<D> td;
  td.init(lane, __builtin_amdgcn_readfirstlane(wave), (unsigned)(rs * 2));
  const bf16_t* kbase = base + H;
  const bf16_t* vbase = base + 2 * H;
  const int64_t total_elems = (int64_t)sh.batch * S * rs;
  const unsigned kbytes = (unsigned)((total_elems - (kbase - qkv)) * 2), vbytes = (unsigned)((total_elems - (vbase - qkv)) * 2);
  auto issue_step = [&](int stage, int step) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int t = step * G + g;
      if (t >= n_tiles) break;   // uniform
      const unsigned row0_bytes = (unsigned)t * 64u * (unsigned)(rs * 2);
      td.issue(kbase, kbytes, smem + (stage * G + g) * 2 * TE, row0_bytes);
      td.issue(vbase, vbytes, smem + (stage * G + g) * 2 * TE + TE, row0_bytes);
    }
  };
  auto compute = [&](int stage, int step) {
    const int tile = step * G + grp, kv0 = tile * 64;
    if ((G > 1 && tile >= n_tiles) || (sh.causal && kv0 > wave_q_max)) return;
    const bf16_t* kt = smem + (stage * G + grp) * 2 * TE;
    const bf16_t* vt = kt + TE;
    const bool edge = (kv0 + 64 > kv_len) || (sh.causal && kv0 + 63 > wave_q_min);
#pragma unroll
    for (int i = 0; i < (SHORT ? 1 : 2); ++i) {
      f32x16_t sc, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = dp[r] = 0.f;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        sc = mfma16<F16>(frag_rows<D>(kt, fr_base, i * 32, s), qf[s], sc);
        dp = mfma16<F16>(frag_rows<D>(vt, fr_base, i * 32, s), df[s], dp);
      }
      uint32_t keep = 0xffffu;
      if (DROP) keep = keep16_query_lane(sh.drop, row_blk, kv0 + 32 * i, kc);
      auto elements = [&](auto edge_tag) {   // two instances: interior tiles carry no mask code
        constexpr bool EDGE = decltype(edge_tag)::value;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float p = __builtin_amdgcn_exp2f(fmaf(sc[r], sl2, -my_lse2));
          if (EDGE) {
            const int kv = kv0 + i * 32 + acc_row(r, lane);
            const bool hide = (kv >= kv_len) | ((sh.causal != 0) & (kv > my_q));
            p = hide ? 0.f : p;
          }
          if (DROP) dp[r] = ((keep >> r) & 1u) ? dp[r] * sh.drop.scale : 0.f;   // dP = keep * (dO V^T) / (1 - p)
          dp[r] = p * (dp[r] - my_delta);
        }
      };
      if (edge) elements(std::true_type{});
      else elements(std::false_type{});
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bf16x8_t dsf = pack8<F16>(dp, h);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          dq[t] = mfma16<F16>(frag_tr<D>(kt, ft_base, i * 32 + 16 * h, t), dsf, dq[t]);
      }
    }
  };
  if constexpr (SHORT) one_tile(n_tiles, issue_step, compute);
  else tile_ring<2, G * 2 * TileDirect<D>::MINE>((n_tiles + G - 1) / G, issue_step, compute);
  if constexpr (G > 1) {
    constexpr int REGS = NT * 16;
    if (grp > 0) {
      float* p = group_slot<G, REGS>(smem, grp, row_wave, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) p[(t * 16 + r) * 64] = dq[t][r];
    }
    __syncthreads();
    if (grp > 0) return;
    for (int g = 1; g < G; ++g) {
      const float* p = group_slot<G, REGS>(smem, g, row_wave, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[t][r] += p[(t * 16 + r) * 64];
    }
  }

  const RowsOut<D, F16, SHORT> rows(smem + row_wave * (G > 1 ? NT * 16 * 128 : RowsOut<D, F16, SHORT>::ELEMS), lane,
                                    SHORT ? wave_q_min : __builtin_amdgcn_readfirstlane(wave_q_min), S);
  if (rows.rows <= 0) return;
  rows.store([&](int t, int e) { return dq[t][e] * scale; }, dqkv + ((int64_t)b * S + rows.first) * rs + a * D, rs, sh.rope);
}

// ============================ backward: the launches =============================================
// OCC: wavefronts per SIMD at least. 128-wide heads with mask draws: two, in 230 registers; left to itself the kernel takes 257 and runs
// one (without mask draws it takes 248, and is 1 % slower in the 244 that a bound brings: 1 x 8192 tokens, 20 heads 1261 / 1272). dQ and dK/dV with mask draws, us, one / two: 64 x 64 tokens, 16 heads 72.2 / 64.5, 128 x 32, 8 62.5 / 54.6, 32 x 520, 5
// 254 / 225, causal 4 x 504, 26 86 / 80, 3 x 1000, 20 210 / 187, 2 x 2048, 20 310 / 278. One where that is faster: causal grids of 300 to 384 blocks,
// a round of the chip and a bit, whose last and shortest blocks then start behind the first that end instead of beside long ones: 2 x
// 1000, 20 (320 blocks) 108 / 114, 1 x 1800, 20 (300) 210 / 225, 2 x 1504, 16 (384) 153 / 161, 1 x 4096, 10 (320) 432 / 479, 10 x 504, 8 (320) 64.6
// / 67.0, but 3 x 896, 15 (315) 131 / 128. Not below (3 x 264, 32, 288 blocks 49.2 / 46.6; 2 x 1000, 18 162 / 157), above (18 x 384, 8, 432 74.7 /
// 69.2; 2 x 1000, 28, 448 131 / 127) or with short walks (7 x 384, 16, 336 63.4 / 60.7).
template <int D, bool DROP, bool F16, bool SHORT, int OCC>
__global__ __launch_bounds__(256, OCC) void attn_bwd_dq_bf16_kernel(AttnShape sh, const bf16_t* __restrict__ qkv,
                                                               const int32_t* __restrict__ seqlens, const bf16_t* __restrict__ out,
                                                               const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                               float* __restrict__ delta, bf16_t* __restrict__ dqkv) {
  attn_bwd_dq_block<D, DROP, F16, 1, SHORT>(xcd_local_block(sh.causal != 0, sh.lpt_heads), sh, qkv, seqlens, out, dout, lse, delta, dqkv);
}
template <int D, bool DROP, bool F16, bool SHORT>
__global__ __launch_bounds__(256) void attn_bwd_dkdv_bf16_kernel(AttnShape sh, const bf16_t* __restrict__ qkv,
                                                                 const int32_t* __restrict__ seqlens, const bf16_t* __restrict__ dout,
                                                                 const float* __restrict__ lse, const float* __restrict__ delta,
                                                                 bf16_t* __restrict__ dqkv) {
  attn_bwd_dkdv_block<D, DROP, F16, false, 1, SHORT>(xcd_local_block(false, sh.lpt_heads), sh, qkv, seqlens, nullptr, dout, lse, delta, dqkv);
}
// Both in one launch, for grids so small that the blocks of the two find room side by side: the dK/dV blocks first (they
// take longer), each with its own delta of every query tile (O is read once more, which a chip that is mostly idle does
// not notice), so that neither kind waits for the other. Two groups at 128-wide heads have no registers left for that:
// delta comes from a kernel in front.
template <int D, int G> constexpr bool OWN_DELTAS = D == 64 || G == 1;
template <int D, bool DROP, bool F16, int G, bool SHORT>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_both_kernel(AttnShape sh, int blocks_x, const bf16_t* __restrict__ qkv,
                                                            const int32_t* __restrict__ seqlens, const bf16_t* __restrict__ out,
                                                            const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                            float* delta, bf16_t* __restrict__ dqkv) {
  const int blocks = blocks_x * sh.heads * sh.batch, w = blockIdx.x;
  if (w < blocks)
    attn_bwd_dkdv_block<D, DROP, F16, OWN_DELTAS<D, G>, G, SHORT>(xcd_local_block(w, blocks_x, sh.heads, sh.batch, false, sh.lpt_heads), sh, qkv,
                                                           seqlens, out, dout, lse, delta, dqkv);
  else
    // (with deltas of the other kind's own, `delta` is left filled all the same, as by the other forms)
    attn_bwd_dq_block<D, DROP, F16, G, SHORT>(xcd_local_block(w - blocks, blocks_x, sh.heads, sh.batch, sh.causal != 0, sh.lpt_heads), sh, qkv,
                                       seqlens, out, dout, lse, OWN_DELTAS<D, G> ? delta : nullptr, dqkv);
}

// =================================== fp32, sequences that fit the LDS =============================
// A block owns 16 rows (queries, or keys for dK/dV) of one (sample, head) and keeps their scores against the whole
// sequence in LDS, [16][seq] floats (two such arrays for dK/dV), so nothing is rescaled. Products on
// v_mfma_f32_16x16x4_f32: inputs, products and sums are fp32, as in the plain loops below; operands go from memory to
// registers in the shape of its fragments. A lane's four elements per 16-deep chunk belong to k = 4 (lane / 16) + s in step
// s for either operand. First the four wavefronts share the score tiles of 16 x 16, then, behind a barrier, the 16-wide
// column tiles of the outputs; both are chains of load latencies, not of arithmetic.
// Small fp32 encoder layer (2 x 128 tokens, 4 heads of 64), against one wavefront per row with plain loops: forward 9.1 ->
// 6.8 us, backward 31 -> 10.8; 512 tokens, 6 heads of 64, causal 57 -> 16.6, 228 -> 26.
constexpr int F32_MAX_SEQ = 1024;   // 2 * 16 * 1028 floats of LDS
__host__ __device__ constexpr int f32_pitch(int seq) { return (seq + 15) / 16 * 16 + 4; }   // floats per row: 16 rows x 16 bytes meet every bank once

// 16 rows x D, this lane's share: row `row`, columns 16 c + 4 (lane / 16) ..
template <int D>
struct RowFrags {
  float4 v[D / 16];
  __device__ __forceinline__ void load(const float* __restrict__ x, int64_t row_offset, int g) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) v[c] = *reinterpret_cast<const float4*>(x + row_offset + 16 * c + 4 * g);
  }
};
// element r: row 4 (lane / 16) + r of a, row lane % 16 of b
template <int D>
__device__ __forceinline__ f32x4_t rows_times_rows(const RowFrags<D>& a, const RowFrags<D>& b) {
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < D / 16; ++c) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c].x, b.v[c].x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c].y, b.v[c].y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c].z, b.v[c].z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c].w, b.v[c].w, acc, 0, 0, 0);
  }
  return acc;
}
// sum over rows 16 t0 .. 16 t1 - 1 of w[lane % 16][row] * x[row][column of the lane]; element r: column 4 (lane / 16) + r of the
// 16 columns that start at x, for row lane % 16 of w. That row of w sees the rows first <= row < end of x (end <= rows); its
// weights elsewhere are 0. Rows at or beyond `rows` are read as the one in front.
// A chunk's rows are common to all 16 rows of w, and 0 times an infinity or a NaN is no zero. So a result that is not finite
// is taken again with such values left out of the products and added only to the rows of w that see them: nothing hidden
// reaches a result, and columns without such values keep their bits. (Tests per chunk instead of one at the end: 512 tokens,
// 6 heads of 64, causal forward 16.2 -> 17.7 us, backward 25.3 -> 27.3.)
__device__ __forceinline__ f32x4_t weighted_rows(const float* w, const float* __restrict__ x, int64_t stride, int t0, int t1, int rows,
                                                 int first, int end, int lane) {
  const int i = lane & 15, g = lane >> 4;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  struct Chunk { float4 w; float x[4]; };
  auto fetch = [&](int t) {
    Chunk c;
    c.w = *reinterpret_cast<const float4*>(w + 16 * t + 4 * g);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int row = 16 * t + 4 * g + s;
      c.x[s] = x[(int64_t)(row < rows ? row : rows - 1) * stride + i];
    }
    return c;
  };
  auto add = [&](const Chunk& c) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x[0], c.w.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x[1], c.w.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x[2], c.w.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c.x[3], c.w.w, acc, 0, 0, 0);
  };
  constexpr int U = 4;   // chunks in flight
  for (int t = t0; t < t1; t += U) {
    Chunk c[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + u < t1) c[u] = fetch(t + u);   // (uniform)
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + u < t1) add(c[u]);
  }
  auto finite = [](float v) { return fabsf(v) < INFINITY; };
  if (__any(!(finite(acc[0]) && finite(acc[1]) && finite(acc[2]) && finite(acc[3])))) {
    acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
      Chunk c = fetch(t);
#pragma unroll
      for (int s = 0; s < 4; ++s) c.x[s] = finite(c.x[s]) ? c.x[s] : 0.f;
      add(c);
    }
    const int from = first > 16 * t0 ? first : 16 * t0, to = end < 16 * t1 ? end : 16 * t1;
#pragma unroll 1
    for (int row = from; row < to; ++row) {
      const float4 v = *reinterpret_cast<const float4*>(x + (int64_t)row * stride + 4 * g);
      const float wr = w[row];
      if (!finite(v.x)) acc[0] = fmaf(v.x, wr, acc[0]);
      if (!finite(v.y)) acc[1] = fmaf(v.y, wr, acc[1]);
      if (!finite(v.z)) acc[2] = fmaf(v.z, wr, acc[2]);
      if (!finite(v.w)) acc[3] = fmaf(v.w, wr, acc[3]);
    }
  }
  return acc;
}
__device__ __forceinline__ int clamp_row(int r, int rows) { return r < rows ? r : rows - 1; }

template <int D>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(AttnShape sh, const float* __restrict__ qkv, const int32_t* __restrict__ seqlens,
                                                           float* __restrict__ out, float* __restrict__ lse) {
  extern __shared__ __attribute__((aligned(16))) float f32sm[];   // scores [16][pitch], 1 / row sum [16]
  const int S = sh.seq, H = sh.hidden, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int b = blockIdx.z, a = blockIdx.y, q0 = blockIdx.x * 16, q = q0 + i, pitch = f32_pitch(S);
  const int64_t rs = 3 * (int64_t)H;
  const float* base = qkv + (int64_t)b * S * rs + a * D;
  int kv_end = visible_keys(sh, seqlens, b);
  if (sh.causal && q0 + 16 < kv_end) kv_end = q0 + 16;
  const int tiles = (kv_end + 15) / 16;
  const float scale = rsqrtf((float)D);
  RowFrags<D> qf;
  qf.load(base, clamp_row(q, S) * rs, g);
  for (int t = wave; t < tiles; t += 4) {
    RowFrags<D> kf;
    kf.load(base + H, clamp_row(16 * t + i, S) * rs, g);
    f32x4_t sc = rows_times_rows<D>(kf, qf);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = 16 * t + 4 * g + r;
      const bool hide = (key >= kv_end) | ((sh.causal != 0) & (key > q));
      sc[r] = hide ? -INFINITY : sc[r] * scale;
    }
    *reinterpret_cast<f32x4_t*>(f32sm + i * pitch + 16 * t + 4 * g) = sc;
  }
  __syncthreads();
  // softmax: 16 threads per row
  float* inv_sum = f32sm + 16 * pitch;
  {
    const int row = threadIdx.x >> 4, c = threadIdx.x & 15, n = tiles * 16;
    float* p = f32sm + row * pitch;
    auto over16 = [](float v, auto op) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 16));
      return v;
    };
    float mx = -INFINITY;
    for (int j = c; j < n; j += 16) mx = fmaxf(mx, p[j]);
    mx = over16(mx, [](float x, float y) { return fmaxf(x, y); });
    const uint64_t e_row = (((uint64_t)b * sh.heads + a) * S + clamp_row(q0 + row, S)) * S;   // element index of probability (row, 0)
    float sum = 0.f;
    for (int j = c; j < n; j += 16) {
      const float e = __expf(p[j] - mx);
      sum += e;                                                        // the softmax is normalised before dropout
      p[j] = (sh.drop.thr != 0 && !dropout_keep1(sh.drop, e_row + j)) ? 0.f : e;
    }
    sum = over16(sum, [](float x, float y) { return x + y; });
    if (c == 0) {
      inv_sum[row] = sum > 0.f ? sh.drop.scale / sum : 0.f;
      if (q0 + row < S) lse[((int64_t)b * sh.heads + a) * S + q0 + row] = sum > 0.f ? mx + __logf(sum) : -INFINITY;
    }
  }
  __syncthreads();
  const float inv = inv_sum[i];
  const int seen = sh.causal && q + 1 < kv_end ? q + 1 : kv_end;   // keys in front of this one are visible to query q
  for (int ct = wave; ct < D / 16; ct += 4) {
    const f32x4_t o = weighted_rows(f32sm + i * pitch, base + 2 * H + ct * 16, rs, 0, tiles, kv_end, 0, seen, lane);
    if (q < S) *reinterpret_cast<float4*>(out + ((int64_t)b * S + q) * H + a * D + ct * 16 + 4 * g) = make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
  }
}

// dQ and dK/dV blocks in one launch, dK/dV (which take longer) first; delta = rowsum(dO * O) comes from a kernel in front.
// Grid: (blocks of 16 rows of all heads, samples, kind); in one dimension, the work items of a batch of many short samples
// would not fit 32 bits.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_f32_kernel(AttnShape sh, int blocks_x, const float* __restrict__ qkv,
                                                           const int32_t* __restrict__ seqlens, const float* __restrict__ dout,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           float* __restrict__ dqkv) {
  extern __shared__ __attribute__((aligned(16))) float f32sm[];   // dS [16][pitch]; dK/dV: P behind it
  const int S = sh.seq, H = sh.hidden, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4, pitch = f32_pitch(S);
  const bool keys = blockIdx.z == 0;
  const int row0 = ((int)blockIdx.x % blocks_x) * 16, a = (int)blockIdx.x / blocks_x, b = blockIdx.y, head = b * sh.heads + a, row = row0 + i;
  const int64_t rs = 3 * (int64_t)H;
  const float* base = qkv + (int64_t)b * S * rs + a * D;
  const float* dobase = dout + (int64_t)b * S * H + a * D;
  float* dbase = dqkv + (int64_t)b * S * rs + a * D;
  const float* lse_row = lse + (int64_t)head * S;       // (head counts the heads of all samples)
  const float* delta_row = delta + (int64_t)head * S;
  const int kv_len = visible_keys(sh, seqlens, b);
  const float scale = rsqrtf((float)D), keep_scale = sh.drop.thr != 0 ? sh.drop.scale : 1.f;
  const uint64_t e_head = (uint64_t)head * S * S;       // element index of probability (0, 0)
  float *ds_rows = f32sm + i * pitch, *p_rows = f32sm + (16 + i) * pitch;
  if (keys) {
    const int first = sh.causal ? row0 / 16 : 0, end = row0 < kv_len ? (S + 15) / 16 : first;   // hidden keys: no query sees them
    RowFrags<D> kf, vf;
    kf.load(base + H, clamp_row(row, S) * rs, g);
    vf.load(base + 2 * H, clamp_row(row, S) * rs, g);
    for (int t = first + wave; t < end; t += 4) {
      RowFrags<D> qf, df;
      qf.load(base, clamp_row(16 * t + i, S) * rs, g);
      df.load(dobase, clamp_row(16 * t + i, S) * (int64_t)H, g);
      float ls[4], de[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) { const int q = clamp_row(16 * t + 4 * g + r, S); ls[r] = lse_row[q]; de[r] = delta_row[q]; }
      const f32x4_t sc = rows_times_rows<D>(qf, kf), dp = rows_times_rows<D>(df, vf);
      f32x4_t pv, ds;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = 16 * t + 4 * g + r;
        const bool hide = (row >= kv_len) | (q >= S) | ((sh.causal != 0) & (row > q));
        const float p = hide ? 0.f : __expf(sc[r] * scale - ls[r]);
        bool keep = true;
        if (sh.drop.thr != 0) keep = dropout_keep1(sh.drop, e_head + (uint64_t)clamp_row(q, S) * S + clamp_row(row, S));
        pv[r] = keep ? p * keep_scale : 0.f;            // what multiplied V in the forward pass
        ds[r] = hide ? 0.f : p * ((keep ? dp[r] * keep_scale : 0.f) - de[r]);
      }
      *reinterpret_cast<f32x4_t*>(p_rows + 16 * t + 4 * g) = pv;
      *reinterpret_cast<f32x4_t*>(ds_rows + 16 * t + 4 * g) = ds;
    }
    __syncthreads();
    const int seen_from = sh.causal ? row : 0, seen_to = row < kv_len ? S : 0;   // queries that see key `row`
    for (int ct = wave; ct < D / 16; ct += 4) {
      const f32x4_t dk = weighted_rows(ds_rows, base + ct * 16, rs, first, end, S, seen_from, seen_to, lane);
      const f32x4_t dv = weighted_rows(p_rows, dobase + ct * 16, H, first, end, S, seen_from, seen_to, lane);
      if (row < S) {
        float* o = dbase + row * rs + H + ct * 16 + 4 * g;
        float v[4] = {dk[0] * scale, dk[1] * scale, dk[2] * scale, dk[3] * scale};
        if (sh.rope) rope_back(v, sh.rope, row, D, ct * 16 + 4 * g);
        *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(o + H) = make_float4(dv[0], dv[1], dv[2], dv[3]);
      }
    }
  } else {
    int kv_end = kv_len;
    if (sh.causal && row0 + 16 < kv_end) kv_end = row0 + 16;
    const int tiles = (kv_end + 15) / 16, q = clamp_row(row, S);
    RowFrags<D> qf, df;
    qf.load(base, q * rs, g);
    df.load(dobase, q * (int64_t)H, g);
    const float my_lse = lse_row[q], my_delta = delta_row[q];
    for (int t = wave; t < tiles; t += 4) {
      RowFrags<D> kf, vf;
      kf.load(base + H, clamp_row(16 * t + i, S) * rs, g);
      vf.load(base + 2 * H, clamp_row(16 * t + i, S) * rs, g);
      const f32x4_t sc = rows_times_rows<D>(kf, qf), dp = rows_times_rows<D>(vf, df);
      f32x4_t ds;
      uint32_t keep = 0xfu;
      if (sh.drop.thr != 0)   // (seq % 8 == 0: four consecutive keys lie in one block of eight; beyond the last key all are hidden)
        keep = dropout_keep8(sh.drop, (e_head + (uint64_t)q * S + 16 * t + 4 * g) >> 3) >> (4 * (g & 1));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = 16 * t + 4 * g + r;
        const bool hide = (key >= kv_end) | ((sh.causal != 0) & (key > q));
        ds[r] = hide ? 0.f : __expf(sc[r] * scale - my_lse) * (((keep >> r) & 1u ? dp[r] * keep_scale : 0.f) - my_delta);
      }
      *reinterpret_cast<f32x4_t*>(ds_rows + 16 * t + 4 * g) = ds;
    }
    __syncthreads();
    const int seen = sh.causal && row + 1 < kv_end ? row + 1 : kv_end;
    for (int ct = wave; ct < D / 16; ct += 4) {
      const f32x4_t dq = weighted_rows(ds_rows, base + H + ct * 16, rs, 0, tiles, kv_end, 0, seen, lane);
      if (row < S) {
        float v[4] = {dq[0] * scale, dq[1] * scale, dq[2] * scale, dq[3] * scale};
        if (sh.rope) rope_back(v, sh.rope, row, D, ct * 16 + 4 * g);
        *reinterpret_cast<float4*>(dbase + row * rs + ct * 16 + 4 * g) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

// =================================== fp32, longer sequences =======================================
// One wavefront per query row; lane <-> key for the scores, lane <-> head-dim column for the output. Both loops are
// chains of load latencies: the row of a key is read 16 bytes at a time, and the rows behind an output column eight at a
// time (added in row order). Small fp32 encoder layer (2 x 128 tokens, 4 heads of 64), against one float at a time:
// forward 18.1 -> 12.7 us, dQ 15.1 -> 14.0, dK/dV 24.4 -> 18.0, the same bits.
__host__ __device__ constexpr int padded4(int n) { return (n + 3) / 4 * 4; }   // LDS rows start at 16 bytes
template <int D>
__device__ __forceinline__ float row_dot(const float* a, const float* __restrict__ b, float s) {   // s + a . b, in order
#pragma unroll 8
  for (int d = 0; d < D; d += 4) {
    const float4 x = *reinterpret_cast<const float4*>(a + d), y = *reinterpret_cast<const float4*>(b + d);
    s = fmaf(x.x, y.x, s); s = fmaf(x.y, y.y, s); s = fmaf(x.z, y.z, s); s = fmaf(x.w, y.w, s);
  }
  return s;
}
// acc + sum over rows first <= j < end of w[j] * x[j * stride], in order
__device__ __forceinline__ float rows_sum(const float* w, const float* __restrict__ x, int64_t stride, int first, int end, float acc) {
  int j = first;
  for (; j + 8 <= end; j += 8) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = x[(j + e) * stride];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(w[j + e], v[e], acc);
  }
  for (; j < end; ++j) acc = fmaf(w[j], x[j * stride], acc);
  return acc;
}
// rope_back for a lane that holds one column, the other one of its pair in the neighbouring lane
__device__ __forceinline__ float rope_back1(float v, const float* __restrict__ table, int pos, int d, int col) {
  const float other = __shfl_xor(v, 1, 64), cs = table[(int64_t)pos * d + (col & ~1)], sn = table[(int64_t)pos * d + (col | 1)];
  float a = col & 1 ? other : v, b = col & 1 ? v : other;
  turn_pair(a, b, cs, -sn);
  return col & 1 ? b : a;
}
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_fwd_simple_kernel(AttnShape sh, const T* __restrict__ qkv,
                                                              const int32_t* __restrict__ seqlens,
                                                              T* __restrict__ out, float* __restrict__ lse) {
  extern __shared__ float fsm[];  // per wave: q[D], p[S]
  const int S = sh.seq, H = sh.hidden, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.z, a = blockIdx.y, i = blockIdx.x * 4 + wave;
  float* qs = fsm + wave * (D + padded4(S));
  float* ps = qs + D;
  if (i >= S) return;  // no block-wide barrier below
  const int64_t rs = 3 * (int64_t)H;
  const T* base = qkv + (int64_t)b * S * rs + a * D;
  int kv_end = visible_keys(sh, seqlens, b);
  if (sh.causal && i + 1 < kv_end) kv_end = i + 1;
  const float scale = rsqrtf((float)D);
  for (int dd = lane; dd < D; dd += 64) qs[dd] = to_f32(base[i * rs + dd]);
  __builtin_amdgcn_wave_barrier();
  float mx = -INFINITY;
  for (int j = lane; j < kv_end; j += 64) {
    const float s = row_dot<D>(qs, base + H + j * rs, 0.f) * scale;
    ps[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  const bool drop = sh.drop.thr != 0;
  const uint64_t e_row = (((uint64_t)b * sh.heads + a) * S + i) * S;   // element index of probability (i, 0)
  for (int j = lane; j < kv_end; j += 64) {
    const float p = __expf(ps[j] - mx);
    sum += p;                                                         // the softmax is normalised before dropout
    ps[j] = (drop && !dropout_keep1(sh.drop, e_row + j)) ? 0.f : p;
  }
  sum = wave_sum(sum);
  __builtin_amdgcn_wave_barrier();
  const float inv = sum > 0.f ? sh.drop.scale / sum : 0.f;
  for (int dd = lane; dd < D; dd += 64) {
    const float acc = rows_sum(ps, base + 2 * H + dd, rs, 0, kv_end, 0.f);
    from_f32(out[((int64_t)b * S + i) * H + a * D + dd], acc * inv);
  }
  if (lane == 0) lse[((int64_t)b * sh.heads + a) * S + i] = sum > 0.f ? mx + __logf(sum) : -INFINITY;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_bwd_dq_simple_kernel(AttnShape sh, const T* __restrict__ qkv,
                                                                 const int32_t* __restrict__ seqlens,
                                                                 const T* __restrict__ dout,
                                                                 const float* __restrict__ lse,
                                                                 const float* __restrict__ delta,
                                                                 T* __restrict__ dqkv) {
  extern __shared__ float fsm[];  // per wave: q[D], do[D], ds[S]
  const int S = sh.seq, H = sh.hidden, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.z, a = blockIdx.y, i = blockIdx.x * 4 + wave;
  float* qs = fsm + wave * (2 * D + padded4(S));
  float* dos = qs + D;
  float* ds = dos + D;
  if (i >= S) return;
  const int64_t rs = 3 * (int64_t)H;
  const T* base = qkv + (int64_t)b * S * rs + a * D;
  int kv_end = visible_keys(sh, seqlens, b);
  if (sh.causal && i + 1 < kv_end) kv_end = i + 1;
  const float scale = rsqrtf((float)D);
  const float my_lse = lse[((int64_t)b * sh.heads + a) * S + i], my_delta = delta[((int64_t)b * sh.heads + a) * S + i];
  const uint64_t e_row = (((uint64_t)b * sh.heads + a) * S + i) * S;
  for (int dd = lane; dd < D; dd += 64) {
    qs[dd] = to_f32(base[i * rs + dd]);
    dos[dd] = to_f32(dout[((int64_t)b * S + i) * H + a * D + dd]);
  }
  __builtin_amdgcn_wave_barrier();
  for (int j = lane; j < kv_end; j += 64) {
    const float s = row_dot<D>(qs, base + H + j * rs, 0.f);
    float dp = row_dot<D>(dos, base + 2 * H + j * rs, 0.f);
    const float p = __expf(s * scale - my_lse);
    if (sh.drop.thr != 0) dp = dropout_keep1(sh.drop, e_row + j) ? dp * sh.drop.scale : 0.f;
    ds[j] = p * (dp - my_delta);
  }
  __builtin_amdgcn_wave_barrier();
  for (int dd = lane; dd < D; dd += 64) {
    float v = rows_sum(ds, base + H + dd, rs, 0, kv_end, 0.f) * scale;
    if (sh.rope) v = rope_back1(v, sh.rope, i, D, dd);
    from_f32(dqkv[((int64_t)b * S + i) * rs + a * D + dd], v);
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_bwd_dkdv_simple_kernel(AttnShape sh, const T* __restrict__ qkv,
                                                                   const int32_t* __restrict__ seqlens,
                                                                   const T* __restrict__ dout,
                                                                   const float* __restrict__ lse,
                                                                   const float* __restrict__ delta,
                                                                   T* __restrict__ dqkv) {
  extern __shared__ float fsm[];  // per wave: k[D], v[D], p[S], ds[S]
  const int S = sh.seq, H = sh.hidden, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.z, a = blockIdx.y, j = blockIdx.x * 4 + wave;
  float* ks = fsm + wave * (2 * D + 2 * padded4(S));
  float* vs = ks + D;
  float* ps = vs + D;
  float* ds = ps + padded4(S);
  if (j >= S) return;
  const int64_t rs = 3 * (int64_t)H;
  const T* base = qkv + (int64_t)b * S * rs + a * D;
  const int kv_len = visible_keys(sh, seqlens, b);
  const float scale = rsqrtf((float)D);
  const int i_first = (j >= kv_len) ? S : (sh.causal ? j : 0);  // hidden key: no query sees it
  for (int dd = lane; dd < D; dd += 64) { ks[dd] = to_f32(base[H + j * rs + dd]); vs[dd] = to_f32(base[2 * H + j * rs + dd]); }
  __builtin_amdgcn_wave_barrier();
  for (int i = i_first + lane; i < S; i += 64) {
    const float s = row_dot<D>(ks, base + i * rs, 0.f);
    float dp = row_dot<D>(vs, dout + ((int64_t)b * S + i) * H + a * D, 0.f);
    const float p = __expf(s * scale - lse[((int64_t)b * sh.heads + a) * S + i]);
    float pv = p;   // what multiplies V in the forward pass
    if (sh.drop.thr != 0) {
      const bool keep = dropout_keep1(sh.drop, ((((uint64_t)b * sh.heads + a) * S + i) * S) + j);
      pv = keep ? p * sh.drop.scale : 0.f;
      dp = keep ? dp * sh.drop.scale : 0.f;
    }
    ps[i] = pv;
    ds[i] = p * (dp - delta[((int64_t)b * sh.heads + a) * S + i]);
  }
  __builtin_amdgcn_wave_barrier();
  for (int dd = lane; dd < D; dd += 64) {
    float dk = rows_sum(ds, base + dd, rs, i_first, S, 0.f) * scale;
    if (sh.rope) dk = rope_back1(dk, sh.rope, j, D, dd);
    const float dv = rows_sum(ps, dout + (int64_t)b * S * H + a * D + dd, H, i_first, S, 0.f);
    from_f32(dqkv[((int64_t)b * S + j) * rs + H + a * D + dd], dk);
    from_f32(dqkv[((int64_t)b * S + j) * rs + 2 * H + a * D + dd], dv);
  }
}

// =================================== launchers ===================================================
// Blocks of 128 rows that the chip runs at a time where they fit a CU twice (64-wide heads) or once.
template <int D> constexpr int64_t ONE_ROUND = D == 64 ? 512 : 256;
constexpr int SHORT_SEQ = 32;   // (RowsOut; not where gradients are turned)
static int64_t attn_blocks(const AttnShape& s) { return (int64_t)((s.seq + 127) / 128) * s.heads * s.batch; }

template <int D, bool F16, int G, bool SHORT = false>
static void fwd_bf16_groups(const AttnShape& s, const void* qkv, const int32_t* seqlens, void* out, float* lse, hipStream_t st) {
  constexpr size_t tiles = (size_t)FWD_STAGES<D> * G * 2 * Tile<D>::ELEMS * sizeof(bf16_t) + (G > 1 ? 128 * sizeof(float) : 0);
  constexpr size_t meet = (size_t)(G - 1) * (4 / G) * (D / 2 + 2) * 64 * sizeof(float), lds = tiles > meet ? tiles : meet;
  auto kern = s.drop.thr ? attn_fwd_bf16_kernel<D, true, F16, G, SHORT> : attn_fwd_bf16_kernel<D, false, F16, G, SHORT>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  constexpr int rows = 128 / G;
  hipLaunchKernelGGL(kern, dim3((s.seq + rows - 1) / rows, s.heads, s.batch), dim3(256), lds, st, s, (const bf16_t*)qkv,
                     seqlens, (bf16_t*)out, lse);
}
// Two groups per block, by the number of 64-row blocks that this makes and of those that run at a time (ONE_ROUND):
// - at most one per CU, whatever the sequence: 1.0-1.6 times as fast as blocks of 128 rows from 65 tokens on.
// - two per CU (64-wide heads): causal blocks, whose lengths differ, gain 0.97-1.4. Others gain 1.02-1.19 where the
//   sequence has an even number of 64-row blocks or is long, and lose 3-10 % where a short one has an odd number (136 or 520
//   tokens: half of a 128-row block's wavefronts have no rows and cost it nothing) or is one block of 128.
// - up to two rounds of 128-wide causal blocks that start longest-first (lpt_heads_for: heads x samples in eights): the more
//   the longer the sequence, and a few more where mask draws lengthen the blocks. In another order fewer (the second round
//   starts late: 7 x 104 tokens, 20 heads 10.8 -> 14.9 us), the fewest with an odd number of 64-row blocks.
// Blocks of 128 rows / two groups, us (heads of all samples x tokens). 64-wide: 16 x 128 5.8 / 5.2; 64 x 512 11.9 / 10.8; 72 x 384
// 9.8 / 9.2; 96 x 136 7.1 / 7.6; causal 16 x 1024 20.0 / 14.1. 128-wide: 14 x 1032 28.4 / 22.4, 17 x 1032 28.5 / 39; causal 16 x
// 1032 27.1 / 18.8, 48 x 384 14.7 / 13.4, 64 x 384 14.9 / 15.4, 48 x 512 17.4 / 16.7, 64 x 512 17.7 / 18.4, 32 x 1024 27.7 / 24.7, 8
// x 4096 88 / 64; not in eights 30 x 640 20.0 / 22.7, 20 x 776 22.3 / 18.0, 22 x 776 22.4 / 23.8, 20 x 1024 27.3 / 26.0, 22 x 1024
// 27.6 / 29.3, 12 x 2048 47.9 / 40.0, 9 x 2056 47.7 / 55.
// (Telling each other the maxima costs up to 1 us of these; without it the probabilities are rounded against other maxima
// and the output differs by 1-2e-3 in bf16 from that of one group, with it by 2-4e-5, like any other order of sums.)
template <int D>
static bool fwd_two_groups(const AttnShape& s) {
  const int64_t per_head = (s.seq + 63) / 64, heads = (int64_t)s.heads * s.batch, blocks = per_head * heads;
  if (s.seq <= 64) return false;
  if (blocks <= 256) return true;
  if (blocks <= ONE_ROUND<D>) return s.causal || (per_head % 2 == 0 && s.seq > 192) || s.seq >= 768;
  if (D == 64 || !s.causal) return false;
  if (heads % 8 != 0) return s.seq >= 640 && blocks <= (per_head % 2 ? 280 : s.seq < 1640 ? 220 + s.seq / 10 : 384);
  return blocks <= 512 && blocks <= (s.drop.thr && s.seq >= 384 ? 192 : 128) + s.seq / 2;
}
template <int D, bool F16>
static void fwd_bf16(const AttnShape& s, const void* qkv, const int32_t* seqlens, void* out, float* lse, hipStream_t st) {
  if (s.seq <= SHORT_SEQ) fwd_bf16_groups<D, F16, 1, true>(s, qkv, seqlens, out, lse, st);
  else if (fwd_two_groups<D>(s)) fwd_bf16_groups<D, F16, 2>(s, qkv, seqlens, out, lse, st);
  else fwd_bf16_groups<D, F16, 1>(s, qkv, seqlens, out, lse, st);
}
template <int D>
static void fwd_f32(const AttnShape& s, const void* qkv, const int32_t* seqlens, void* out, float* lse, hipStream_t st) {
  if (s.seq <= F32_MAX_SEQ) {
    const size_t lds = (size_t)(16 * f32_pitch(s.seq) + 16) * sizeof(float);
    auto kern = attn_fwd_f32_kernel<D>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3((s.seq + 15) / 16, s.heads, s.batch), dim3(256), lds, st, s, (const float*)qkv, seqlens, (float*)out, lse);
    return;
  }
  const size_t lds = (size_t)4 * (D + padded4(s.seq)) * sizeof(float);
  auto kern = attn_fwd_simple_kernel<float, D>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3((s.seq + 3) / 4, s.heads, s.batch), dim3(256), lds, st, s, (const float*)qkv, seqlens,
                     (float*)out, lse);
}

// Causal shapes: every XCD walks the blocks of ALL its heads longest-first (one group). Measured alone against the
// head-by-head order: OPT-1.3B-shaped layer forward 80 -> 63 us, backward 239 -> 217; 2.7B-shaped 147 -> 123 and
// 450 -> 404; LLaMA-7B-shaped 75 -> 61 and 240 -> 203. Groups of 8 or 16 heads are within a few per cent of that
// for some shapes and kernels (LLaMA-7B-shaped: 55 and 191 with groups of 8) and worse for others (a remainder
// group starts its long blocks late), so the one rule is kept.
static int lpt_heads_for(const AttnShape& s) { return s.causal ? s.batch * s.heads : 0; }

void launch_attn_fwd(int dtype, const AttnShape& s0, const void* qkv, const int32_t* seqlens, void* out,
                     float* lse, hipStream_t st) {
  AttnShape s = s0;
  s.lpt_heads = lpt_heads_for(s);
  const int D = s.hidden / s.heads;
  if (dtype == DT_FP32) { if (D == 64) fwd_f32<64>(s, qkv, seqlens, out, lse, st); else fwd_f32<128>(s, qkv, seqlens, out, lse, st); }
  else if (dtype == DT_FP16) { if (D == 64) fwd_bf16<64, true>(s, qkv, seqlens, out, lse, st); else fwd_bf16<128, true>(s, qkv, seqlens, out, lse, st); }
  else { if (D == 64) fwd_bf16<64, false>(s, qkv, seqlens, out, lse, st); else fwd_bf16<128, false>(s, qkv, seqlens, out, lse, st); }
}

template <int D, bool F16, int G, bool SHORT = false>
static void bwd_both(const AttnShape& s, const void* qkv, const int32_t* seqlens, const void* out, const void* dout,
                     const float* lse, float* delta, void* dqkv, hipStream_t st) {
  constexpr size_t tiles = (size_t)DKDV_STAGES<D> * G * (2 * Tile<D>::ELEMS + 256) * sizeof(bf16_t);
  constexpr size_t meet = (size_t)(G - 1) * (4 / G) * D * 64 * sizeof(float);
  const size_t main = tiles + (s.drop.thr ? 4 * 2048 : 0), lds = main > meet ? main : meet;
  auto kern = s.drop.thr ? attn_bwd_both_kernel<D, true, F16, G, SHORT> : attn_bwd_both_kernel<D, false, F16, G, SHORT>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (!OWN_DELTAS<D, G>) {
    using T = std::conditional_t<F16, f16_t, bf16_t>;
    const int64_t items = (int64_t)s.batch * s.seq * s.heads * 8;
    hipLaunchKernelGGL((attn_delta_kernel<T, D>), dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, s, (const T*)out, (const T*)dout, delta);
  }
  constexpr int rows = 128 / G;
  const int blocks_x = (s.seq + rows - 1) / rows;
  hipLaunchKernelGGL(kern, dim3(2 * blocks_x * s.heads * s.batch), dim3(256), lds, st, s, blocks_x, (const bf16_t*)qkv, seqlens,
                     (const bf16_t*)out, (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv);
}
// dQ first: it also produces delta = rowsum(dO * O), which the dK/dV kernel reads
template <int D, bool F16, bool SHORT>
static void bwd_two_launches(const AttnShape& s, const void* qkv, const int32_t* seqlens, const void* out, const void* dout,
                             const float* lse, float* delta, void* dqkv, hipStream_t st) {
  const dim3 grid((s.seq + 127) / 128, s.heads, s.batch);
  const int64_t blocks = attn_blocks(s);
  {
    const size_t lds = (size_t)4 * Tile<D>::ELEMS * sizeof(bf16_t);
    constexpr int OCC = D == 128 ? 2 : 1;
    const bool alone = !SHORT && D == 128 && s.causal && s.seq >= 504 && blocks >= 300 && blocks <= 384;
    auto kern = !s.drop.thr ? attn_bwd_dq_bf16_kernel<D, false, F16, SHORT, 1>
                : alone     ? attn_bwd_dq_bf16_kernel<D, true, F16, SHORT, SHORT ? OCC : 1>
                            : attn_bwd_dq_bf16_kernel<D, true, F16, SHORT, OCC>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, s, (const bf16_t*)qkv, seqlens, (const bf16_t*)out,
                       (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv);
  }
  {
    // with dropout: 2 KB per wavefront behind the stages for the exchange of mask draws
    const size_t lds = (size_t)DKDV_STAGES<D> * (2 * Tile<D>::ELEMS + 256) * sizeof(bf16_t) + (s.drop.thr ? 4 * 2048 : 0);
    auto kern = s.drop.thr ? attn_bwd_dkdv_bf16_kernel<D, true, F16, SHORT> : attn_bwd_dkdv_bf16_kernel<D, false, F16, SHORT>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, s, (const bf16_t*)qkv, seqlens, (const bf16_t*)dout, lse,
                       (const float*)delta, (bf16_t*)dqkv);
  }
}
template <int D, bool F16>
static void bwd_bf16(const AttnShape& s, const void* qkv, const int32_t* seqlens, const void* out, const void* dout,
                     const float* lse, float* delta, void* dqkv, hipStream_t st) {
  // One launch while either kind's blocks alone fit one round (128-wide blocks that do not differ in length: while they
  // leave an eighth of the chip free, with mask draws three eighths); two groups per block while the four times as many
  // blocks do.
  // Two launches / one / one with two groups, us: 64-wide 16 blocks (one sample of 128) 14.6 / 8.7 / 7.0, 128 (1024 tokens,
  // causal) 48.7 / 32.8 / 24.1, 192 (4 x 512, 12 heads) 31 / 22.5 / 26.2, 256 (2048, causal) 90 / 62 / 47, 512 (8 x 512, padded)
  // 48.5 / 45.3 / 54, 1536 (6 x 1024, causal) 132 / 141; 128-wide 64 (2 x 1024, causal) 68 / 44.5 / 29, 128 (2 x 512) 44 / 29 / 34.5,
  // 192 (3 x 1024, causal) 73 / 46 / 57, 256 (4 x 1024, causal) 74 / 56 / 68, 384 80 / 85; not causal 216 (24 x 1032) 84 / 77,
  // 255 (15 x 2056) 159 / 166. With mask draws, 64-wide 16 blocks 18.7 / - / 9.2, 128 (1024, causal) 85 / - / 43, 256 (4 x 512) 48.5 /
  // 34.8, 512 (8 x 512) 70.5 / 65.3; 128-wide causal 256 116 / 85, not causal 144 (16 x 1032) 123 / 99, 160
  // (4 x 512) 61 / 54, 176 (4 x 512) 61 / 64, 256 (4 x 512) 62.6 / 66.9.
  // Beside weight gradients in K ranges (s.beside) two launches again from 129 to 256 blocks of 64-wide heads: one at a time
  // they leave the half of every CU's LDS that a workgroup of those needs. Steps at hidden 256, two launches / one: 52 x 128 tokens
  // 215 / 217 us, 10 x 670 234 / 246, 16 x 512 245 / 255, 7 x 1024 229 / 253, 8 x 1024 262 / 271; up to 6143 tokens, without K
  // ranges, the other way round (7 x 670 218 / 206).
  const int64_t blocks = attn_blocks(s), room = D == 64 || s.causal ? ONE_ROUND<D> : s.drop.thr ? 160 : 224;
  if (blocks <= ONE_ROUND<D> / (s.causal ? 2 : 4) && s.seq > 64) return bwd_both<D, F16, 2>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  const bool make_way = D == 64 && s.beside && blocks > 128 && blocks <= 256;
  const bool is_short = s.seq <= SHORT_SEQ && !s.rope;
  if (blocks <= room && !make_way) {
    if (is_short) bwd_both<D, F16, 1, true>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
    else bwd_both<D, F16, 1>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  } else {
    if (is_short) bwd_two_launches<D, F16, true>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
    else bwd_two_launches<D, F16, false>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  }
}
template <int D>
static void bwd_f32(const AttnShape& s, const void* qkv, const int32_t* seqlens, const void* out, const void* dout,
                    const float* lse, float* delta, void* dqkv, hipStream_t st) {
  const int64_t items = (int64_t)s.batch * s.seq * s.heads * 8;
  hipLaunchKernelGGL((attn_delta_kernel<float, D>), dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, s,
                     (const float*)out, (const float*)dout, delta);
  if (s.seq <= F32_MAX_SEQ) {
    const size_t lds = (size_t)2 * 16 * f32_pitch(s.seq) * sizeof(float);
    auto kern = attn_bwd_f32_kernel<D>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    const int blocks_x = (s.seq + 15) / 16;
    hipLaunchKernelGGL(kern, dim3(blocks_x * s.heads, s.batch, 2), dim3(256), lds, st, s, blocks_x, (const float*)qkv, seqlens,
                       (const float*)dout, lse, (const float*)delta, (float*)dqkv);
    return;
  }
  dim3 grid((s.seq + 3) / 4, s.heads, s.batch);
  {
    const size_t lds = (size_t)4 * (2 * D + padded4(s.seq)) * sizeof(float);
    auto kern = attn_bwd_dq_simple_kernel<float, D>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, s, (const float*)qkv, seqlens, (const float*)dout, lse,
                       (const float*)delta, (float*)dqkv);
  }
  {
    const size_t lds = (size_t)4 * (2 * D + 2 * padded4(s.seq)) * sizeof(float);
    auto kern = attn_bwd_dkdv_simple_kernel<float, D>;
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, s, (const float*)qkv, seqlens, (const float*)dout, lse,
                       (const float*)delta, (float*)dqkv);
  }
}

void launch_attn_bwd(int dtype, const AttnShape& s0, const void* qkv, const int32_t* seqlens, const void* out,
                     const void* dout, const float* lse, float* delta, void* dqkv, hipStream_t st) {
  AttnShape s = s0;
  s.lpt_heads = lpt_heads_for(s);
  const int D = s.hidden / s.heads;
  if (dtype == DT_FP32) {
    if (D == 64) bwd_f32<64>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
    else bwd_f32<128>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  } else if (dtype == DT_FP16) {
    if (D == 64) bwd_bf16<64, true>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
    else bwd_bf16<128, true>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  } else {
    if (D == 64) bwd_bf16<64, false>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
    else bwd_bf16<128, false>(s, qkv, seqlens, out, dout, lse, delta, dqkv, st);
  }
}

}  // namespace slapo
