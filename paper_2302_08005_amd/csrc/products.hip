// Several independent products of backward in one launch of 256x256 tiles: data gradients (layout NN) and weight gradients (TN).
// Each product alone ends in a round that is partly empty, or has too few such tiles for the 256 CUs and is then cut into 128x128
// ones, which read twice the bytes from LDS per multiply. Together they fill rounds of the large tiles. Which calls: products_together
// (api.hip). What bounds it: the matrix cores under the chip's power limit (1.3 us per 64-deep slab with all CUs busy, 1.0 with a
// quarter of them) and 8-10 us per tile of first loads and last stores.
// us, alone / together (the same operands again and again, so that the last-level cache holds those of the smaller ones):
//   T = 4096, hidden 1024, FFN 4096: dX (NN, K = 3072) and the four weight gradients, 256 tiles 139 / 95 (in the step, with operands from
//   memory and a pass over dQKV beside it, the launch takes 113-130); T = 16384 of it, 448 tiles 435 / 390 (375-385 in the step); T = 2048,
//   hidden 4096, attention 512, FFN 1376, 528 tiles: 158 / 105-109 (122 in the step); T = 8192, hidden 2560, FFN 10240, 1520 tiles 1210 / 1170;
//   whole rounds by themselves gain nothing (8192, hidden 2048, FFN 8192: 707 / 733; the tiles of several rounds drift apart).
#include <algorithm>

#include "common.h"
#include "gemm_tile.h"
#include "kernels.h"

namespace slapo {

namespace {

constexpr int CUS = 256;
int tiles_of(const Product& p) { return ((p.M + 255) / 256) * ((p.N + 255) / 256); }
int slabs_of(const Product& p) { return (p.K + 63) / 64; }

struct ProductArgs {
  // longest K first. `group`: products of this K from here on (0: belongs to the group in front), `group_tiles` of theirs.
  struct { int layout, M, N, K, tiles, group, group_tiles; const bf16_t *A, *B; bf16_t* C; const bf16_t* aux; } p[MAX_PRODUCTS];
  int whole, total;   // tiles from `whole` on come in quarters
};

// Tiles start in the order of their length, the longest first. Workgroups are handed to the XCDs round-robin; each XCD gets a run of
// consecutive tiles (operand panels shared through its L2) of every group of equal length, so that all XCDs have the same work in
// every length: a run of the whole list would hand one XCD all of the long tiles (2000 tokens, hidden 2560, 80 tiles of K = 7680 in
// front of 400 of 2000: 198 us, by group 153). A group of at most one round is one list, which makes compacter blocks of
// tiles (192 tiles of three products: 367 / 350); longer ones go by product (1200 tiles, K = 8192: 990 / 957).
//
// The tiles that would end alone come in quarters, 128x128 tiles of the same eight wavefronts on 128-deep slabs, which take a third of
// a tile's time (gemm.hip has them for single products): 528 tiles of 2048 tokens, hidden 4096, attention 512, FFN 1376, end on 16 that
// start when the others are through their second; 126 -> 105 us, 138 -> 148 with all operands from memory, backward 290 -> 275. Over 45
// layers that cut 1 to 32 tiles backward takes 0.90 to 1.01 of what it takes with whole ones. The quarters of a tile go to one XCD.
template <int LAYOUT, bool KTAIL, bool F16>
__device__ __forceinline__ void product_tile(bool quarter, int m0, int n0, int M, int N, int K, const bf16_t* A, const bf16_t* B, bf16_t* C,
                                             const bf16_t* aux) {
  if (!quarter)
    gemm_bf16_tile<LAYOUT, 256, 256, 64, 2, 4, 1, 2, 0, KTAIL, EPI_ADD, F16, false, true>(0, M, N, K, A, B, C, nullptr, aux, nullptr, 0, 0, 1,
                                                                                          nullptr, m0, n0);
  else if (m0 < M && n0 < N)
    gemm_bf16_tile<LAYOUT, 128, 128, 128, 2, 4, 1, 2, 0, KTAIL, EPI_ADD, F16, false, true>(0, M, N, K, A, B, C, nullptr, aux, nullptr, 0, 0, 1,
                                                                                           nullptr, m0, n0);
}

template <bool KTAIL, bool F16>
__global__ __launch_bounds__(512, 1) void gemm_bf16_products_kernel(ProductArgs a) {
  int g = blockIdx.x, i = 0, at = 0;
  const bool quarter = g >= a.whole;
  if (quarter) {
    const int u = g - a.whole;
    g = a.whole + (u >> 5) * 8 + (u & 7);
    at = (u >> 3) & 3;
    if (g >= a.total) return;
  }
  while (g >= a.p[i].group_tiles) { g -= a.p[i].group_tiles; i += a.p[i].group; }   // (uniform; fewer than `total`)
  const bool one_list = a.p[i].group_tiles <= CUS;
  if (one_list) {
    const int per_xcd = a.p[i].group_tiles >> 3;
    if (g < per_xcd * 8) g = (g & 7) * per_xcd + (g >> 3);
  }
  while (g >= a.p[i].tiles) g -= a.p[i++].tiles;
  const int M = a.p[i].M, N = a.p[i].N, K = a.p[i].K, tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
  const TilePos pos = one_list ? tile_in_order(g, tiles_m, tiles_n) : tile_position(g, tiles_m, tiles_n, 1);
  const int m0 = pos.tile_m * 256 + (at >> 1) * 128, n0 = pos.tile_n * 256 + (at & 1) * 128;
  if (a.p[i].layout == GEMM_TN) product_tile<GEMM_TN, false, F16>(quarter, m0, n0, M, N, K, a.p[i].A, a.p[i].B, a.p[i].C, a.p[i].aux);
  else product_tile<GEMM_NN, KTAIL, F16>(quarter, m0, n0, M, N, K, a.p[i].A, a.p[i].B, a.p[i].C, a.p[i].aux);
}

void longest_first(int n, Product* p) {
  std::stable_sort(p, p + n, [](const Product& x, const Product& y) { return x.K > y.K; });
}

// A tile costs its slabs and about six more for first loads and last stores. CUs take tiles in the order of the launch, each the
// next one when it is done: a multiset of the times at which CUs are free, all tiles of a length that start together at once.
// `quarters`: that many of the last tiles (of the last product at most) in quarters. *last: how many tiles end with the launch.
int slabs_of_launch(int n, const Product* p, int quarters, int* last) {
  struct { int at, cus; } free_at[CUS] = {{0, CUS}};
  int times = 1, end = 0;
  for (int i = 0; i <= n; ++i) {
    const Product& q = p[i < n ? i : n - 1];
    const int len = (i < n ? slabs_of(q) : slabs_of(q) * 3 / 10) + TILE_SLABS;
    for (int left = i < n ? tiles_of(q) - (i == n - 1 ? quarters : 0) : 4 * quarters; left > 0;) {
      int first = 0;
      for (int k = 1; k < times; ++k) first = free_at[k].at < free_at[first].at ? k : first;
      const int at = free_at[first].at + len, take = std::min(left, free_at[first].cus);
      left -= take;
      if (!(free_at[first].cus -= take)) free_at[first] = free_at[--times];
      int same = 0;
      while (same < times && free_at[same].at != at) ++same;
      if (same == times) free_at[times++] = {at, 0};   // (at most one entry per CU)
      free_at[same].cus += take;
      if (at > end) *last = 0;
      end = std::max(end, at);
      if (at == end) *last += take;
    }
  }
  return end;
}

// Quarters for the tiles that end with the launch if it then ends earlier, and they are at most an eighth of a round: more of
// them run at a higher clock as they are (400 tiles of 8192 tokens, hidden 2560, whole / the last 144 in quarters: 340 / 379 us; a
// decoder of 3696 tokens, hidden 3712, apart / a launch per block with the last 53 in quarters: 2845 / 2918).
struct ProductPlan { int quarters, slabs; };
ProductPlan plan_of(int n, const Product* p) {
  int last = 0, ignored = 0;
  const int whole = slabs_of_launch(n, p, 0, &last);
  last = std::min(last, tiles_of(p[n - 1]));
  if (last > CUS / 8) return {0, whole};
  const int cut = slabs_of_launch(n, p, last, &ignored);
  return cut < whole ? ProductPlan{last, cut} : ProductPlan{0, whole};
}

}  // namespace

int products_slabs(int n, const Product* products) {
  Product p[MAX_PRODUCTS];
  std::copy(products, products + n, p);
  longest_first(n, p);
  return plan_of(n, p).slabs;
}

void launch_products(int dtype, int n, const Product* products, hipStream_t st) {
  Product p[MAX_PRODUCTS];
  std::copy(products, products + n, p);
  longest_first(n, p);
  ProductArgs a = {};
  bool ktail = false;
  for (int i = 0, head = 0; i < n; ++i) {
    a.p[i] = {p[i].layout, p[i].M, p[i].N, p[i].K, tiles_of(p[i]), 0, 0, (const bf16_t*)p[i].A, (const bf16_t*)p[i].B, (bf16_t*)p[i].C, (const bf16_t*)p[i].aux};
    if (p[i].K != p[head].K) head = i;
    ++a.p[head].group;
    a.p[head].group_tiles += a.p[i].tiles;
    a.total += a.p[i].tiles;
    ktail = ktail || (p[i].layout == GEMM_NN && p[i].K % 128 != 0);
  }
  const int quarters = plan_of(n, p).quarters;
  a.whole = a.total - quarters;
  constexpr size_t l0 = gemm_lds_bytes<256, 256, 64, 2, 4, 1, 2>(), l1 = gemm_lds_bytes<128, 128, 128, 2, 4, 1, 2>(), lds = l0 > l1 ? l0 : l1;
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(a.whole + (quarters + 7) / 8 * 32), dim3(512), lds, st, a);
  };
  if (dtype == DT_FP16) { if (ktail) go(gemm_bf16_products_kernel<true, true>); else go(gemm_bf16_products_kernel<false, true>); }
  else { if (ktail) go(gemm_bf16_products_kernel<true, false>); else go(gemm_bf16_products_kernel<false, false>); }
}

}  // namespace slapo
