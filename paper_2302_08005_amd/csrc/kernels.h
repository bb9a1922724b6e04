// Host-side launch interface between the C ABI (api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "common.h"

namespace slapo {

// true if `name` is listed in the SLAPO_DEBUG environment variable (comma-separated debugging / A-B switches)
bool debug_flag(const char* name);

enum { GEMM_NT = 0, GEMM_NN = 1, GEMM_TN = 2 };
// EPI_GATE: the product's columns are (gate, up) pairs; C [M,N/2] = silu(gate) * up, aux_out [M,N] = the pair
//   (up * silu'(gate), silu(gate)), the two factors backward multiplies the gradient of C with.
// EPI_DACT: C = acc * act'(aux_in); aux_out (16-bit storage; NULL: none) = column sums of every DACT_SUM_ROWS rows of C, as
//   floats [M / DACT_SUM_ROWS rounded up][N], for launch_colreduce_partials.
// EPI_DGATE: the product is that gradient [M,N]; C [M,2N] = (acc * aux_in[m,2n], acc * aux_in[m,2n+1]).
// EPI_SPLITK (internal to the weight-gradient path): the workgroup covers one of `act` K ranges of its tile and
//   writes the fp32 accumulators to aux_out (a float workspace [splits][M][N]); splitk_reduce sums them.
// EPI_ROPE (internal to the gated layer's QKV projection): the first two thirds of the columns are heads whose adjacent
//   pairs are turned by the angles of the row's position; bias = the (cos, sin) table (launch_rope_table), act = rope_act(...).
enum { EPI_NONE = 0, EPI_BIAS = 1, EPI_BIAS_ACT = 2, EPI_DACT = 3, EPI_ADD = 4, EPI_GATE = 5, EPI_DGATE = 6, EPI_SPLITK = 7, EPI_ROPE = 8 };
constexpr int DACT_SUM_ROWS = 32;
inline int rope_act(int seq, int head_dim) { return 2 * seq + (head_dim == 128 ? 1 : 0); }

// solo: nothing else runs beside this GEMM (it may then pick tiles by round count, see launch_bf16)
// ws / ws_bytes: optional fp32 workspace (gemm_ws_bytes says how much a shape can use; 0: none). With it, a grid
//   that would end in a thin last round computes its last tiles in several K ranges instead.
void launch_gemm(int dtype, int layout, int epi, int act, int M, int N, int K, const void* A, const void* B,
                 void* C, const void* bias, const void* aux_in, void* aux_out, hipStream_t st, bool solo = false,
                 float* ws = nullptr, size_t ws_bytes = 0);
size_t gemm_ws_bytes(int dtype, int layout, int epi, int M, int N, int K);
// tiles that make the product exactly one round, which is faster than K ranges: launch_gemm without a workspace takes them
bool gemm_in_one_round(int dtype, int layout, int M, int N, int K);
// Products whose reader adds up K ranges itself (the row kernels, launch_add_ranges): product_in_ranges says whether a product of
// this shape is worth computing so (N then is a width of rows that the row kernels have such forms for), launch_gemm_ranges
// leaves the ranges as fp32 arrays [K_RANGES][M][N].
constexpr int K_RANGES = 4, RANGES_MIN_N = 512, RANGES_MAX_N = 4096;
bool product_in_ranges(int dtype, int M, int N, int K);
void launch_gemm_ranges(int dtype, int layout, int M, int N, int K, const void* A, const void* B, float* parts, hipStream_t st);
// out [mn] = sum of the ranges, in order, + addend (NULL: nothing); 16-bit storage
void launch_add_ranges(int dtype, int64_t mn, int ranges, const float* parts, const void* addend, void* out, hipStream_t st);
// the smallest workspace that a caller who passes one may pass: 256x256 grids whose K is a multiple of 128 have always
// asked for all that they can use; other K and grids of smaller tiles do without one that is too small for them
size_t gemm_ws_least_bytes(int dtype, int layout, int epi, int M, int N, int K);
void describe_gemm(int dtype, int layout, int epi, int M, int N, int K, bool solo, bool weight_grad, bool with_ws,
                   char* buf, size_t len);
// Weight gradient C[M,N] (+)= A[K,M]^T B[K,N] (accumulate: add to C). Outputs with too few tiles to fill the
// chip are computed in several K ranges at once (fp32 partial tiles in `ws`, summed in range order by a second
// kernel: deterministic), outputs whose tile grid ends in a thin round have their last tiles cut into K ranges
// (launch_gemm); weight_grad_ws_bytes says how much workspace a shape wants (0: none, plain GEMM).
size_t weight_grad_ws_bytes(int dtype, int M, int N, int K);
// what a caller has to bring: the same where K is a multiple of 256 (K ranges of few tiles) or 128 (thin last rounds), as
// ever; other K run as one plain GEMM without a workspace
size_t weight_grad_ws_least_bytes(int dtype, int M, int N, int K);
void launch_weight_grad(int dtype, int accumulate, int M, int N, int K, const void* A, const void* B, void* C,
                        float* ws, hipStream_t st, bool solo = false);

// Independent products in one launch of 256x256 tiles, 16-bit storage (products.hip): C [M,N] = A B (layout GEMM_NN) or A^T B
// (GEMM_TN), + aux (NULL: nothing; it may be C).
constexpr int MAX_PRODUCTS = 5, TILE_SLABS = 6;   // TILE_SLABS: what a tile takes besides its 64-deep slabs, in such slabs
struct Product { int layout, M, N, K; const void *A, *B; void* C; const void* aux; };
void launch_products(int dtype, int n, const Product* products, hipStream_t st);
// how long the launch takes, in 64-deep slabs of one tile (sizes only, no pointers)
int products_slabs(int n, const Product* products);
// the same for a product (NN, 16-bit) that has a launch of its own and the chip to itself
int gemm_slabs(int layout, int M, int N, int K);
// and for one that another stream's tiles run beside (backward with a launch for each product)
double gemm_slabs_beside(int layout, int M, int N, int K);

// What backward computes from one gradient array, in one launch: the gradient that goes on (layout NN, C [M,N] = A [M,K]
// B [K,N], epilogue EPI_DACT, EPI_DGATE or EPI_ADD; the latter adds nothing if aux is NULL), the weight gradient
// dW [wM,wN] (+)= wA [wK,wM]^T wB [wK,wN] (NULL: none), the column sums of wA (a bias gradient; NULL: none) and the sums over the partial
// rows [nblk][3][H] that an earlier row kernel left (outputs as in launch_colreduce3; partials NULL: none).
struct GradPair {
  int epi, act, M, N, K;
  const void *A, *B;
  void* C;
  const void* aux;
  int wM, wN, wK;
  const void *wA, *wB;
  void* dW;
  void* colsum;
  const float* partials;
  int nblk, H;
  void* sums[3];
  int accumulate;
  // the data gradient in K ranges (product_in_ranges), left as fp32 arrays [K_RANGES][M][N] in place of C; NULL: C
  float* parts;
};
void launch_grad_pair(int dtype, const GradPair& p, hipStream_t st);

struct AttnShape {
  int batch, seq, hidden, heads, causal;
  int lpt_heads = 0;   // causal block order: heads per longest-first group (set by the launchers; 0 = head by head)
  // dropout on the attention probabilities (site 2; element ((b*heads + a)*seq + i)*seq + j); thr == 0: none
  DropoutParams drop = {0u, 0u, 2u, 0u, 0u, 1.0f};
  // backward: (cos, sin) table of the rotation that queries and keys went through (NULL: none); dQ and dK are turned back
  const float* rope = nullptr;
  bool beside = false;   // backward: another stream computes weight gradients in K ranges meanwhile
};
void launch_attn_fwd(int dtype, const AttnShape& s, const void* qkv, const int32_t* seqlens, void* out,
                     float* lse, hipStream_t st);
void launch_attn_bwd(int dtype, const AttnShape& s, const void* qkv, const int32_t* seqlens, const void* out,
                     const void* dout, const float* lse, float* delta, void* dqkv, hipStream_t st);

// rms: the normalisation is RMSNorm (no mean subtraction, no offset; beta, mu unused). bias may be null.
// r_in_ranges: r is fp32 arrays [K_RANGES][rows][H], which add up to the branch's output (launch_gemm_ranges).
void launch_bdrln_fwd(int dtype, int64_t rows, int H, const void* r, const void* bias, const void* res,
                      const void* gamma, const void* beta, void* z_out, void* out, float* mu, float* rstd,
                      const DropoutParams& dp, float eps, int rms, hipStream_t st, bool r_in_ranges = false);
// dout_in_ranges: dout is fp32 arrays [K_RANGES][rows][H], which add up, with dout_add (NULL: nothing), to the gradient.
int bdrln_bwd_blocks(int64_t rows);
void launch_bdrln_bwd(int dtype, int64_t rows, int H, const void* dout, const void* z, const float* mu,
                      const float* rstd, const void* gamma, const void* dres_in, void* dz_out, void* dr_out,
                      float* partials, const DropoutParams& dp, int rms, hipStream_t st, int dr_from_stored = 0, int blocks = 0,
                      bool dout_in_ranges = false, const void* dout_add = nullptr);
// Blocks (and partial rows) for launch_bdrln_bwd inside a layer (blocks = 0: bdrln_bwd_blocks, which the exported kernel has):
// few rows go to more blocks of fewer, because a launch that short is its latency chain, of which the column sums across a
// block's groups are a part: 16 blocks of 8 rows -> 64 of 2 at 128 rows of 1024, 7.2 -> 5.4 us; steps of 128 tokens at hidden 1024
// 112.6 -> 108.3, of 512 158.7 -> 154.6, equal from 2048 tokens on.
int bdrln_bwd_blocks_wide(int64_t rows, int H);
// Rotary embedding on the Q and K parts of a packed [rows, 3H] array, in place: inside every head of width d
// the adjacent pair (2j, 2j+1) of row t is turned by the angle of table entry (t % seq, j) (negated when
// `inverse`). table: [seq, d/2] (cos, sin) pairs in fp32, written by launch_rope_table (angle m * base^(-2j/d),
// evaluated in double precision).
void launch_rope_table(int seq, int d, float base, float* table, hipStream_t st);
void launch_rope(int dtype, int64_t rows, int seq, int H, int d, const float* table, void* qkv, int inverse,
                 hipStream_t st);
int colsum_blocks(int64_t rows);
void launch_colsum_partials(int dtype, int64_t rows, int64_t N, const void* a, float* partials,
                            hipStream_t st);
void launch_colreduce_partials(int dtype, int64_t nblk, int64_t stride, int64_t N, const float* partials,
                               void* out, int accumulate, hipStream_t st);
// out_k[n] (+)= sum_i partials[(i*3 + k)*H + n] for k = 0..2 in one launch; null outputs are skipped
void launch_colreduce3(int dtype, int64_t nblk, int H, const float* partials, void* out0, void* out1, void* out2,
                       int accumulate, hipStream_t st);
void launch_dropout_mask(int64_t n_elements, uint8_t* mask, const DropoutParams& dp, hipStream_t st);

}  // namespace slapo
