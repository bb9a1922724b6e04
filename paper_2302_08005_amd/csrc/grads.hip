// Backward launches that hold several products. What backward computes from one gradient array - the gradient that goes
// on down the layer (layout NN) and the gradient of the weights (layout TN) - does not depend on each other, and neither do
// the column sums behind the bias gradients: one launch takes a workgroup per tile of either product and a few more for
// the sums. A call of a few hundred tokens is bound by the number of its launches, each of which fills the chip for a few
// microseconds at best; here the tiles of the second product run where the first leaves CUs idle. Backward of a post-LN
// layer takes 7 launches instead of 18 on one stream (two row kernels, four of these, attention), of a pre-LN layer 9; a step
// of 128 tokens at hidden 1024 155 -> 123 us when they came, of 1024 tokens at hidden 512 174 -> 129. Which calls take them:
// gradients_paired (api.hip).
#include <type_traits>

#include "common.h"
#include "gemm_tile.h"
#include "kernels.h"

namespace slapo {

namespace {

struct PairArgs {
  GradPair p;
  int red_blocks, cs_blocks, nn_blocks, tn_blocks, nn_first;
};

// out[n] (+)= sum of column n of a [rows, N]: a workgroup owns 128 columns, 16 threads of 8 columns side by side; the
// other threads share the rows, eight rows' loads in flight each, and meet in LDS (added in thread order).
template <typename T, int THREADS>
__device__ __forceinline__ void column_sums(int block, int rows, int N, const T* __restrict__ a, T* out, int accumulate, float* lds) {
  constexpr int RY = THREADS / 16;
  const int cx = threadIdx.x & 15, ry = threadIdx.x >> 4;
  const int64_t c = (int64_t)block * 128 + cx * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (c < N) {
    const T* p = a + c;
    int r = ry;
    for (; r + 7 * RY < rows; r += 8 * RY) {
      Raw8<T> raw[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) raw[u].load(p + (int64_t)(r + u * RY) * N);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        float v[8];
        raw[u].get(v);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += v[e];
      }
    }
    for (; r < rows; r += RY) {
      float v[8];
      load8(p + (int64_t)r * N, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  }
  store8(lds + ry * 128 + cx * 8, acc);
  __syncthreads();
  const int64_t n = (int64_t)block * 128 + threadIdx.x;
  if (threadIdx.x < 128 && n < N) {
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < RY; ++k) s += lds[k * 128 + threadIdx.x];
    if (accumulate) s += to_f32(out[n]);
    from_f32(out[n], s);
  }
}

// out_k[n] (+)= sum_i partials[(i * 3 + k) * H + n], k = block / (column blocks): a workgroup owns 64 columns of one k, four
// of its wavefronts contiguous shares of the rows, eight loads in flight; the shares are added in wavefront order, so the
// bits are those of colreduce3_kernel (rowwise.hip), which a layer without a next launch uses.
template <typename T>
__device__ __forceinline__ void partial_row_sums(int block, int nblk, int H, const float* __restrict__ partials, T* out0, T* out1,
                                                 T* out2, int accumulate, float* lds) {
  constexpr int WAVES = 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col_blocks = (H + 63) / 64;
  const int which = block / col_blocks, n = (block - which * col_blocks) * 64 + lane;
  T* out = which == 0 ? out0 : which == 1 ? out1 : out2;
  if (out == nullptr) return;   // uniform for the block
  const int per = (nblk + WAVES - 1) / WAVES, i0 = wave * per, i1 = i0 + per < nblk ? i0 + per : nblk;
  const float* src = partials + (int64_t)which * H + n;
  const int64_t stride = 3 * (int64_t)H;
  float s = 0.f;
  if (n < H && wave < WAVES) {
    int i = i0;
    for (; i + 8 <= i1; i += 8) {
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = src[(i + k) * stride];
#pragma unroll
      for (int k = 0; k < 8; ++k) s += v[k];
    }
    for (; i < i1; ++i) s += src[i * stride];
  }
  if (wave < WAVES) lds[wave * 64 + lane] = s;
  __syncthreads();
  if (wave == 0 && n < H) {
    float t = lds[lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) t += lds[w * 64 + lane];
    if (accumulate) t += to_f32(out[n]);
    from_f32(out[n], t);
  }
}

// The workgroups with sums to add come first: they are chains of loads, which pass beside the products. Returns false for
// a workgroup that belongs to a product.
template <typename T, int THREADS>
__device__ __forceinline__ bool sums(const PairArgs& a, int& block, float* lds) {
  const GradPair& p = a.p;
  if (block < a.red_blocks) {
    partial_row_sums<T>(block, p.nblk, p.H, p.partials, (T*)p.sums[0], (T*)p.sums[1], (T*)p.sums[2], p.accumulate, lds);
    return true;
  }
  block -= a.red_blocks;
  if (block < a.cs_blocks) {
    column_sums<T, THREADS>(block, p.wK, p.wM, (const T*)p.wA, (T*)p.colsum, p.accumulate, lds);
    return true;
  }
  block -= a.cs_blocks;
  return false;
}

// Tiles of either product: 512 threads, four computing wavefronts in a 2x2 grid and four loader wavefronts (gemm_tile.h),
// with as many LDS stages as let two workgroups share a CU.
template <int BM_, int BN_, int NS_>
struct PairTile {
  static constexpr int BM = BM_, BN = BN_, NS = NS_;
  static constexpr size_t LDS = gemm_lds_bytes<BM, BN, 64, 2, 2, 1, NS>();
  static int count(int M, int N) { return ((M + BM - 1) / BM) * ((N + BN - 1) / BN); }
};
constexpr int PAIR_LOADERS = 4, PAIR_THREADS = (2 * 2 + PAIR_LOADERS) * 64;
constexpr size_t max_lds(size_t a, size_t b) { return a > b ? a : b; }

// X: tiles of the data gradient (layout NN), W: of the weight gradient (TN).
template <class X, class W, bool KTAIL, int EPI, bool F16>
__global__ __launch_bounds__(PAIR_THREADS, 4) void grad_pair_kernel(PairArgs a) {
  using T = std::conditional_t<F16, f16_t, bf16_t>;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  int block = blockIdx.x;
  if (sums<T, PAIR_THREADS>(a, block, reinterpret_cast<float*>(smem))) return;
  const GradPair& p = a.p;
  const bool nn = a.nn_first ? block < a.nn_blocks : block >= a.tn_blocks;
  if (nn) {
    gemm_bf16_tile<GEMM_NN, X::BM, X::BN, 64, 2, 2, 1, X::NS, PAIR_LOADERS, KTAIL, EPI, F16, false, EPI == EPI_ADD>(
        a.nn_first ? block : block - a.tn_blocks, p.M, p.N, p.K, (const bf16_t*)p.A, (const bf16_t*)p.B, (bf16_t*)p.C, nullptr,
        (const bf16_t*)p.aux, reinterpret_cast<bf16_t*>(p.parts), EPI == EPI_SPLITK ? K_RANGES : p.act, 0, 1, nullptr);
  } else {
    gemm_bf16_tile<GEMM_TN, W::BM, W::BN, 64, 2, 2, 1, W::NS, PAIR_LOADERS, false, EPI_ADD, F16, false, true>(
        a.nn_first ? block - a.nn_blocks : block, p.wM, p.wN, p.wK, (const bf16_t*)p.wA, (const bf16_t*)p.wB, (bf16_t*)p.dW, nullptr,
        p.accumulate ? (const bf16_t*)p.dW : nullptr, nullptr, 0, 0, 1, nullptr);
  }
}

template <int W>
__global__ __launch_bounds__(F32_WAVES * 64) void grad_pair_f32_kernel(PairArgs a) {
  constexpr int SUM_FLOATS = F32_WAVES * 64 * 8;   // (column_sums: eight per thread)
  __shared__ __attribute__((aligned(16))) float lds[f32_lds_floats(W) > SUM_FLOATS ? f32_lds_floats(W) : SUM_FLOATS];
  int block = blockIdx.x;
  if (sums<float, F32_WAVES * 64>(a, block, lds)) return;
  const GradPair& p = a.p;
  if (a.nn_first ? block < a.nn_blocks : block >= a.tn_blocks) {
    gemm_f32_tile<GEMM_NN, W>(a.nn_first ? block : block - a.tn_blocks, lds, p.M, p.N, p.K, (const float*)p.A, (const float*)p.B,
                              (float*)p.C, nullptr, (const float*)p.aux, nullptr, p.epi == EPI_ADD && !p.aux ? EPI_NONE : p.epi, p.act);
  } else {
    gemm_f32_tile<GEMM_TN, W>(a.nn_first ? block - a.nn_blocks : block, lds, p.wM, p.wN, p.wK, (const float*)p.wA, (const float*)p.wB,
                              (float*)p.dW, nullptr, (const float*)p.dW, nullptr, p.accumulate ? EPI_ADD : EPI_NONE, 0);
  }
}

template <class X, class W, bool F16>
void launch_pair_tiles(PairArgs a, hipStream_t st) {
  a.nn_blocks = X::count(a.p.M, a.p.N) * (a.p.parts ? K_RANGES : 1);
  a.tn_blocks = a.p.dW ? W::count(a.p.wM, a.p.wN) : 0;
  constexpr size_t lds = max_lds(max_lds(X::LDS, W::LDS), PAIR_THREADS * 8 * sizeof(float));
  const dim3 grid(a.red_blocks + a.cs_blocks + a.nn_blocks + a.tn_blocks);
#define SLAPO_PAIR(E)                                                                                                     \
  do {                                                                                                                    \
    auto kern = a.p.K % 64 == 0 ? grad_pair_kernel<X, W, false, E, F16> : grad_pair_kernel<X, W, true, E, F16>;           \
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                  \
    hipLaunchKernelGGL(kern, grid, dim3(PAIR_THREADS), lds, st, a);                                                       \
  } while (0)
  if constexpr (X::BM == 64) {
    if (a.p.parts) { SLAPO_PAIR(EPI_SPLITK); return; }
  }
  if (a.p.epi == EPI_DACT) SLAPO_PAIR(EPI_DACT);
  else if (a.p.epi == EPI_DGATE) SLAPO_PAIR(EPI_DGATE);
  else SLAPO_PAIR(EPI_ADD);
#undef SLAPO_PAIR
}

// Tiles by how many there are. Steps (forward and backward) of an encoder layer, us, same card, tiles of the data gradient /
// the weight gradient:
//                                64x64/64x64   64x64/128x64   64x64/128x128   128x64/128x64   128x64/128x128
//   hidden 256,  1024 tokens         106            113            134             112             133
//   hidden 512,  1024                129            128            145             133             144
//   hidden 1024, 128                 126            125            125             137             139
//   hidden 1024, 1024                210            204            207             196             202
//   hidden 2048, 128                 195            188            185             209             205
//   768, 2286 (half)                 250            241            269             236             255
// The data gradient takes 64x64 tiles while its 128x64 ones would leave half of the 256 CUs idle (thresholds of 64 to 256
// tiles: within 2 % of each other); the weight gradient 64x64 while both products together then are at most two tiles per
// CU, 128x128 where its 128x64 ones are more than two per CU.
template <bool F16>
void launch_pair_16(const PairArgs& a, hipStream_t st) {
  using Small = PairTile<64, 64, 4>;
  using Medium = PairTile<128, 64, 3>;
  using Large = PairTile<128, 128, 2>;
  const GradPair& p = a.p;
  const int nn = Medium::count(p.M, p.N), tn = p.dW ? Medium::count(p.wM, p.wN) : 0;
  if (p.parts) {   // (K ranges of 64x64 tiles, at most one workgroup per CU)
    if (tn <= 128) launch_pair_tiles<Small, Small, F16>(a, st);
    else if (tn <= 512) launch_pair_tiles<Small, Medium, F16>(a, st);
    else launch_pair_tiles<Small, Large, F16>(a, st);
  } else if (nn <= 128) {
    if (tn + 2 * nn <= 512) launch_pair_tiles<Small, Small, F16>(a, st);
    else if (tn <= 512) launch_pair_tiles<Small, Medium, F16>(a, st);
    else launch_pair_tiles<Small, Large, F16>(a, st);
  } else {
    if (tn <= 512) launch_pair_tiles<Medium, Medium, F16>(a, st);
    else launch_pair_tiles<Medium, Large, F16>(a, st);
  }
}

}  // namespace

void launch_grad_pair(int dtype, const GradPair& p, hipStream_t st) {
  PairArgs a = {};
  a.p = p;
  a.red_blocks = p.partials ? 3 * ((p.H + 63) / 64) : 0;
  a.cs_blocks = p.dW && p.colsum ? (p.wM + 127) / 128 : 0;
  a.nn_first = p.K / (p.parts ? K_RANGES : 1) >= p.wK;   // the longer tiles start first
  if (dtype == DT_FP32) {
    auto count = [](int M, int N, int t) { return ((M + t - 1) / t) * ((N + t - 1) / t); };
    // (as for one product: 16x16 tiles where the larger ones would leave half of the CUs idle)
    const int t = count(p.M, p.N, 32) + (p.dW ? count(p.wM, p.wN, 32) : 0) > 128 ? 32 : 16;
    a.nn_blocks = count(p.M, p.N, t);
    a.tn_blocks = p.dW ? count(p.wM, p.wN, t) : 0;
    const dim3 grid(a.red_blocks + a.cs_blocks + a.nn_blocks + a.tn_blocks);
    if (t == 32) hipLaunchKernelGGL(grad_pair_f32_kernel<2>, grid, dim3(F32_WAVES * 64), 0, st, a);
    else hipLaunchKernelGGL(grad_pair_f32_kernel<1>, grid, dim3(F32_WAVES * 64), 0, st, a);
    return;
  }
  if (dtype == DT_FP16) launch_pair_16<true>(a, st);
  else launch_pair_16<false>(a, st);
}

}  // namespace slapo
