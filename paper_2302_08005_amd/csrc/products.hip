// Several independent products of backward in one launch of 256x256 tiles: data gradients (layout NN) and weight gradients (TN).
// Each product alone ends in a round that is partly empty, or has too few such tiles for the 256 CUs and is then cut into 128x128
// ones, which read twice the bytes from LDS per multiply. Together they fill rounds of the large tiles. Which calls: products_together
// (api.hip). What bounds it: the matrix cores under the chip's power limit (1.3 us per 64-deep slab with all CUs busy, 1.0 with a
// quarter of them) and 8-10 us per tile of first loads and last stores.
// us, alone / together (operands in the last-level cache):
//   T = 4096, hidden 1024, FFN 4096: dX (NN, K = 3072) and the four weight gradients, 256 tiles 139 / 95; T = 16384 of it, 448 tiles
//   435 / 390; T = 2048, hidden 4096, attention 512, FFN 1376: 158 / 119; T = 8192, hidden 2560, FFN 10240, 1520 tiles 1210 / 1170;
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
};

// Tiles start in the order of their length, the longest first. Workgroups are handed to the XCDs round-robin; each XCD gets a run of
// consecutive tiles (operand panels shared through its L2) of every group of equal length, so that all XCDs have the same work in
// every length: a run of the whole list would hand one XCD all of the long tiles (2000 tokens, hidden 2560, 80 tiles of K = 7680 in
// front of 400 of 2000: 198 us, by group 153). A group of at most one round is one list, which makes compacter blocks of
// tiles (192 tiles of three products: 367 / 350); longer ones go by product (1200 tiles, K = 8192: 990 / 957).
template <bool KTAIL, bool F16>
__global__ __launch_bounds__(512, 1) void gemm_bf16_products_kernel(ProductArgs a) {
  int g = blockIdx.x, i = 0;
  while (g >= a.p[i].group_tiles) { g -= a.p[i].group_tiles; i += a.p[i].group; }   // (uniform; the grid holds no more tiles)
  const bool one_list = a.p[i].group_tiles <= CUS;
  if (one_list) {
    const int per_xcd = a.p[i].group_tiles >> 3;
    if (g < per_xcd * 8) g = (g & 7) * per_xcd + (g >> 3);
  }
  while (g >= a.p[i].tiles) g -= a.p[i++].tiles;
  const int M = a.p[i].M, N = a.p[i].N, K = a.p[i].K, tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
  const TilePos pos = one_list ? tile_in_order(g, tiles_m, tiles_n) : tile_position(g, tiles_m, tiles_n, 1);
  if (a.p[i].layout == GEMM_TN)
    gemm_bf16_tile<GEMM_TN, 256, 256, 64, 2, 4, 1, 2, 0, false, EPI_ADD, F16, false, true>(
        0, M, N, K, a.p[i].A, a.p[i].B, a.p[i].C, nullptr, a.p[i].aux, nullptr, 0, 0, 1, nullptr, pos.tile_m * 256, pos.tile_n * 256);
  else
    gemm_bf16_tile<GEMM_NN, 256, 256, 64, 2, 4, 1, 2, 0, KTAIL, EPI_ADD, F16, false, true>(
        0, M, N, K, a.p[i].A, a.p[i].B, a.p[i].C, nullptr, a.p[i].aux, nullptr, 0, 0, 1, nullptr, pos.tile_m * 256, pos.tile_n * 256);
}

void longest_first(int n, Product* p) {
  std::stable_sort(p, p + n, [](const Product& x, const Product& y) { return x.K > y.K; });
}

}  // namespace

// A tile costs its slabs and about six more for first loads and last stores. CUs take tiles in the order of the launch, each the
// next one when it is done: a multiset of the times at which CUs are free, all tiles of a length that start together at once.
int products_slabs(int n, const Product* products, int64_t* work) {
  Product p[MAX_PRODUCTS];
  std::copy(products, products + n, p);
  longest_first(n, p);
  struct { int at, cus; } free_at[CUS] = {{0, CUS}};
  int times = 1, end = 0;
  for (int i = 0; i < n; ++i) {
    const int len = slabs_of(p[i]) + TILE_SLABS;
    *work += (int64_t)tiles_of(p[i]) * len;
    for (int left = tiles_of(p[i]); left > 0;) {
      int first = 0;
      for (int k = 1; k < times; ++k) first = free_at[k].at < free_at[first].at ? k : first;
      const int at = free_at[first].at + len, take = std::min(left, free_at[first].cus);
      left -= take;
      if (!(free_at[first].cus -= take)) free_at[first] = free_at[--times];
      int same = 0;
      while (same < times && free_at[same].at != at) ++same;
      if (same == times) free_at[times++] = {at, 0};   // (at most one entry per CU)
      free_at[same].cus += take;
      end = std::max(end, at);
    }
  }
  return end;
}

void launch_products(int dtype, int n, const Product* products, hipStream_t st) {
  Product p[MAX_PRODUCTS];
  std::copy(products, products + n, p);
  longest_first(n, p);
  ProductArgs a = {};
  int total = 0;
  bool ktail = false;
  for (int i = 0, head = 0; i < n; ++i) {
    a.p[i] = {p[i].layout, p[i].M, p[i].N, p[i].K, tiles_of(p[i]), 0, 0, (const bf16_t*)p[i].A, (const bf16_t*)p[i].B, (bf16_t*)p[i].C, (const bf16_t*)p[i].aux};
    if (p[i].K != p[head].K) head = i;
    ++a.p[head].group;
    a.p[head].group_tiles += a.p[i].tiles;
    total += a.p[i].tiles;
    ktail = ktail || (p[i].layout == GEMM_NN && p[i].K % 64 != 0);
  }
  constexpr size_t lds = gemm_lds_bytes<256, 256, 64, 2, 4, 1, 2>();
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(total), dim3(512), lds, st, a);
  };
  if (dtype == DT_FP16) { if (ktail) go(gemm_bf16_products_kernel<true, true>); else go(gemm_bf16_products_kernel<false, true>); }
  else { if (ktail) go(gemm_bf16_products_kernel<true, false>); else go(gemm_bf16_products_kernel<false, false>); }
}

}  // namespace slapo
