// C ABI of the library: argument validation, layout of the `saved` / `scratch` buffers and the
// sequence of kernel launches that makes up one layer forward / backward. Host code only.
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "../../include/slapo.h"
#include "kernels.h"

using namespace slapo;

namespace {

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
inline bool overlap(const void* a, const void* b, size_t bytes) {   // arrays of `bytes` each
  const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
  return p < q + bytes && q < p + bytes;
}
inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// width of each of Q, K, V (heads * head dim): the hidden size unless the descriptor says otherwise
inline int attn_width(const slapo_layer_desc* d) { return d->attn_dim > 0 ? d->attn_dim : d->hidden; }

int check_desc(const slapo_layer_desc* d) {
  if (!d) return SLAPO_ERR_NULL;
  if (d->batch <= 0 || d->seq <= 0 || d->hidden <= 0 || d->heads <= 0 || d->ffn <= 0 || d->attn_dim < 0) return SLAPO_ERR_SHAPE;
  if (attn_width(d) % d->heads != 0) return SLAPO_ERR_SHAPE;
  if (!(d->dropout_p >= 0.f && d->dropout_p < 1.f)) return SLAPO_ERR_SHAPE;
  if (!(d->ln_eps > 0.f)) return SLAPO_ERR_SHAPE;
  if (d->hidden % 8 != 0 || d->ffn % 8 != 0) return SLAPO_ERR_ALIGN;
  const int hd = attn_width(d) / d->heads;
  if (hd != 64 && hd != 128) return SLAPO_ERR_UNSUPPORTED;
  if (d->hidden > 8192) return SLAPO_ERR_UNSUPPORTED;   // the row kernels hold a row per wavefront / per block
  // fp32 (correctness mode): beyond 1024 tokens dK/dV keeps two score rows per wavefront in LDS, 16 (2 d + 2 seq) bytes per block
  if (d->dtype == SLAPO_FP32 && (int64_t)16 * (2 * hd + 2 * (int64_t)d->seq) > 160 * 1024) return SLAPO_ERR_UNSUPPORTED;
  if (d->dtype != SLAPO_BF16 && d->dtype != SLAPO_FP32 && d->dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (d->act != SLAPO_GELU_ERF && d->act != SLAPO_RELU) return SLAPO_ERR_UNSUPPORTED;
  if ((d->causal != 0 && d->causal != 1) || (d->pre_ln != 0 && d->pre_ln != 1)) return SLAPO_ERR_UNSUPPORTED;
  if (d->checkpoint != 0 && d->checkpoint != 1) return SLAPO_ERR_UNSUPPORTED;
  if (!(d->attn_dropout_p >= 0.f && d->attn_dropout_p < 1.f)) return SLAPO_ERR_SHAPE;
  if (d->attn_dropout_p > 0.f && d->seq % 8 != 0) return SLAPO_ERR_ALIGN;   // a mask block of 8 keys stays inside one query row
  if ((int64_t)d->batch * d->seq * 3 * d->hidden >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if ((int64_t)d->batch * d->seq * 3 * attn_width(d) >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if ((int64_t)d->batch * d->seq * d->ffn >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if (d->arch != SLAPO_ARCH_CLASSIC && d->arch != SLAPO_ARCH_LLAMA) return SLAPO_ERR_UNSUPPORTED;
  if (d->arch == SLAPO_ARCH_LLAMA) {
    if (!d->pre_ln) return SLAPO_ERR_UNSUPPORTED;                    // the family is pre-norm by definition
    if (!(d->rope_base > 1.f)) return SLAPO_ERR_SHAPE;
    if ((int64_t)d->batch * d->seq * 2 * d->ffn >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  }
  return SLAPO_OK;
}

inline bool is_llama(const slapo_layer_desc* d) { return d->arch == SLAPO_ARCH_LLAMA; }
inline bool keeps_dact(const slapo_layer_desc* d) { return is_llama(d) || d->act != SLAPO_RELU; }
// The pointer tables list weight, bias (or gain, offset) alternately; the LLaMA-style layer has the six
// weights and gains only, i.e. the even entries.
inline bool param_needed(const slapo_layer_desc* d, int index) { return !is_llama(d) || index % 2 == 0; }
int check_tables(const slapo_layer_desc* d, const void* const (&ps)[12]) {
  for (int i = 0; i < 12; ++i) {
    if (!param_needed(d, i)) continue;
    if (!ps[i]) return SLAPO_ERR_NULL;
    if (misaligned(ps[i])) return SLAPO_ERR_ALIGN;
  }
  return SLAPO_OK;
}

}  // namespace

namespace slapo {
// SLAPO_DEBUG in the environment: a comma-separated list of switches for debugging and A/B timing, read once.
//   single-stream  backward keeps all of its work on the caller's stream (no helper stream)
//   no-splitk      weight gradients always run as one plain GEMM (no K ranges; also shrinks the workspace sizes
//                  the *_workspace calls report, so set it before the first call, not between size query and use)
bool debug_flag(const char* name) {
  const char* env = getenv("SLAPO_DEBUG");
  if (!env) return false;
  const size_t n = strlen(name);
  for (const char* p = env; *p;) {
    const char* e = strchr(p, ',');
    const size_t len = e ? (size_t)(e - p) : strlen(p);
    if (len == n && !strncmp(p, name, n)) return true;
    p += len + (e ? 1 : 0);
  }
  return false;
}
}  // namespace slapo

namespace {

DropoutParams make_dropout(const slapo_layer_desc* d, int site) {
  DropoutParams dp;
  dp.key0 = (uint32_t)(d->seed & 0xffffffffu);
  dp.key1 = (uint32_t)(d->seed >> 32);
  dp.site = (uint32_t)site;
  dp.layer = (uint32_t)d->layer_id;
  dp.thr = (uint32_t)llround((double)d->dropout_p * 65536.0);
  dp.scale = 1.0f / (1.0f - d->dropout_p);
  return dp;
}

// No element is dropped and none is scaled (a rate below half a draw's step still scales).
bool dropout_keeps_all(const DropoutParams& dp) { return dp.thr == 0 && dp.scale == 1.0f; }

AttnShape make_attn_shape(const slapo_layer_desc* d) {
  AttnShape as = {d->batch, d->seq, attn_width(d), d->heads, d->causal};
  as.drop.key0 = (uint32_t)(d->seed & 0xffffffffu);
  as.drop.key1 = (uint32_t)(d->seed >> 32);
  as.drop.site = 2u;
  as.drop.layer = (uint32_t)d->layer_id;
  as.drop.thr = (uint32_t)llround((double)d->attn_dropout_p * 65536.0);
  as.drop.scale = 1.0f / (1.0f - d->attn_dropout_p);
  return as;
}

// A launch that failed leaves its error in the runtime's per-thread "last error". Every entry point samples that
// slot before its first launch (entry_error) and again after its last one (finish): an error that was already
// there belongs to somebody else and is neither reported as ours nor cleared; one that appeared in between is
// ours, is reported as SLAPO_ERR_HIP and cleared.
thread_local hipError_t g_error_at_entry = hipSuccess;
void entry_error() { g_error_at_entry = hipPeekAtLastError(); }
int finish() {
  if (g_error_at_entry != hipSuccess) return SLAPO_OK;   // cannot tell ours from the stale one: leave it to its owner
  return hipGetLastError() == hipSuccess ? SLAPO_OK : SLAPO_ERR_HIP;
}

// The weight-gradient GEMMs of the backward pass do not feed the data-gradient chain, and most kernels of
// the chain leave half of each CU's LDS and wave slots free (one 128x128 tile per CU). Where they do not share
// launches with each other and the data gradients (products_together, grad pairs) they are therefore
// issued on a helper stream that forks from and joins back into the caller's stream with events, so the
// two kinds of GEMM share the CUs. One helper stream and a few events per device are created on first use
// and kept for the life of the process (the only state the library holds). Host threads that call into the
// library on the same device share them: every event record and the stream wait that consumes it are issued
// under the device's mutex, so a wait always captures the record of its own call (a wait refers to the
// record that precedes it at the time it is issued), and the calls' helper-stream work simply queues up
// behind each other. "single-stream" in SLAPO_DEBUG turns the helper stream off; small
// calls do without it (backward_on_one_stream).
struct SideStream {
  hipStream_t stream = nullptr;
  hipEvent_t fork[4] = {nullptr, nullptr, nullptr, nullptr};
  hipEvent_t join = nullptr;
  int state = 0;   // 0 untried, 1 ready, -1 unavailable
  std::mutex pair_mu;   // held across each (record, wait) pair
  // everything issued on `from` so far happens before what is issued on `to` from now on
  void order(hipEvent_t ev, hipStream_t from, hipStream_t to) {
    std::lock_guard<std::mutex> lock(pair_mu);
    (void)hipEventRecord(ev, from);
    (void)hipStreamWaitEvent(to, ev, 0);
  }
};
SideStream* side_stream() {
  static SideStream table[16];
  static std::mutex mu;
  static const bool disabled = debug_flag("single-stream");
  if (disabled) return nullptr;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  SideStream& s = table[dev];
  if (s.state == 0) {
    bool ok = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) == hipSuccess;
    // the events order work of two streams of ONE device: no timing, and no system-scope fence at the record
    // (the host and other devices never look at what they guard; the fence cost ~7 us of idle stream per fork)
    const unsigned flags = hipEventDisableTiming | hipEventDisableSystemFence;
    for (int i = 0; ok && i < 4; ++i) ok = hipEventCreateWithFlags(&s.fork[i], flags) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&s.join, flags) == hipSuccess;
    s.state = ok ? 1 : -1;
    if (!ok) (void)hipGetLastError();
  }
  return s.state == 1 ? &s : nullptr;
}

// Small calls keep all of backward on the caller's stream. The forks and the join of two streams cost the host about as
// much as the launches of a layer that has one per product (a step's calls take 150-210 us instead of 85-130, by machine and
// moment), so two streams pay where the step keeps the GPU busy for about that long and the weight gradients, whose few workgroups walk all tokens,
// leave the chip to the data gradients beside them. The rule estimates the GPU's time for a step on one stream, in us:
// launches; multiply-adds of the projections, with 300 tokens' worth for the weights that each call reads and writes
// whatever its size (fp32 products take eight times as long); row work and the weight gradients' walk, per token, at a third
// more than their time because two streams win that back; attention's walk over the keys, which lengthens with the head
// width. Steps per call of classic layers (feed-forward 4 x hidden, 64-wide heads), one stream / two, on machines of
// either speed, with the estimate (two machines where the answer differs):
//   hidden 256   1024 tokens in sequences of 128: 135 / 169 us (151), of 1024: 184 / 173, 185 / 197 (191); 1536 of 128:
//                147 / 170 (168); 2048 of 128: 158 / 161, 160 / 197 (185), of 512: 178 / 214 (202), of 2048: 263 / 241
//                (271); 2560 of 128: 174 / 163 (202); 4096 of 2048: 312 / 272 (339); 8192 of 512: 289 / 255 (407)
//   hidden 384   1024 of 128: 145 / 195 (156); 1536 of 128: 163 / 148 (175); 2048 of 128: 174 / 152, 174 / 200 (195)
//   hidden 512   1024 of 128: 156 / 161 (164); 1536 of 128: 177 / 159 (186); 2048 of 128: 194 / 165, 193 / 206 (208)
//   hidden 768   512 of 128: 174 / 191 (155); 1024 of 128: 193 / 180 (186), of 1024: 242 / 227 (226)
//   hidden 1024  128: 157 / 200 (142); 512 of 128: 185 / 201 (174); 1024 of 128: 230 / 218 (216)
// These figures, and the constants made from them, are of one product per launch. With paired launches (gradients_paired) a
// step on one stream has 15 to 17 launches, and one stream is the faster form beyond the line too (hidden 1024, 600 tokens: 162 /
// 176 us; 512, 2048 159 / 170); the line is kept where it was, and beyond it paired calls fork once.
bool backward_on_one_stream(const slapo_layer_desc* d) {
  const double T = (double)d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  const double weights = 4.0 * H * A + (is_llama(d) ? 3.0 : 2.0) * H * F;
  const double products = 4.2e-9 * weights * (T * (d->dtype == SLAPO_FP32 ? 8.0 : 1.0) + 300.0);
  return 110.0 + products + 0.03 * T + 7e-4 * (A / d->heads) * d->seq < 184.0;
}

// Whether backward puts each weight gradient into the launch of the data gradient beside it (GradPair): always on one
// stream, whose calls are bound by the number of their launches; on two streams where the products are small enough that
// the smaller tiles of those launches cost less than three of the four forks (only the gradient of the output projection
// still goes to the helper stream, beside the attention kernels). Few tokens do not make the products small: with weights
// beyond 64 million elements reading them and writing their gradients is most of the step, and plain launches on two
// streams do that faster (fp32 products, which are bound by arithmetic, gain at every size). Not for the gated layer on
// two streams: its wider products lose more to the smaller tiles than the forks cost, but for the narrowest layers.
// Steps in us, every weight gradient forked / paired:
//   classic  hidden 512, 2048 tokens 186 / 170; 768, 2286 261 / 246; 1024, 600 201 / 176, 2000 296 / 282, 4096 470 / 495;
//            1536, 640 269 / 255, 3000 648 / 676; 2048, 384 280 / 272, 1500 477 / 493; 256, 4096 364 / 351, 8192 253 / 264
//   few tokens, two machines: 2048 (50 M), 46 tokens 244 / 193, 189 / 193, 256 258 / 233, 240 / 238; 2304 (64 M), 128 227 / 233;
//            2432 (71 M), 46 215 / 226; 2560 (79 M), 46 253 / 273, 128 260 / 305; 4096 (201 M), 128 486 / 568
//   fp32     2560, 128 1271 / 1232; 4096, 16 1187 / 1125
//   gated    hidden 512, 2048 tokens 194 / 180, 4000 257 / 272; 1024, 600 203 / 182, 1000 199 / 221, 2000 308 / 334; 2048, 384 268
//            / 294, 600 354 / 361; 4096 (an eighth of the heads and columns), 2048 492 / 527
bool gradients_paired(const slapo_layer_desc* d) {
  if (backward_on_one_stream(d)) return true;
  const double T = (double)d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  const double weights = 4.0 * H * A + 2.0 * H * F;
  return !is_llama(d) && T <= 4096.0 && weights * T <= 3.2e10 && (weights <= 6.4e7 || d->dtype == SLAPO_FP32);
}

}  // namespace

namespace slapo {

// Whether the weight gradients of backward share launches of 256x256 tiles with each other and with data gradients (launch_products),
// all on the caller's stream, and which: the gradient of the layer's input and all four behind the attention kernels (BEHIND), or those
// of each block with the gradient of the block's input (BLOCKS; the better form at equal slabs, fewer tiles drift apart). Decided
// by what either form takes in slabs of such a tile. Shared, the launches as they fill rounds (products_slabs) and the two products
// that then have the chip to themselves; apart, the tiles of all products spread over the chip, because two streams fill each other's
// thin rounds. Where the gradient of the second feed-forward weight alone has tiles for three quarters of the chip, the two streams run
// the same large tiles and hide more behind each other: 7 % and 12 slabs between the estimates (12 % where only the gradient of the gated
// layer's first feed-forward weight, twice as wide, is as large). Elsewhere they run 128x128 tiles and pay for forks and launches: 12 % and 22
// slabs the other way; the gated layer has no sums that would leave the chain: 10 % and 8 slabs, but where sharing takes at most
// 76 slabs, the calls for two streams cost the host more than that (140 us; from hidden 512 on, where it was measured). Its calls on one
// stream pair gradients, which is faster there (77 / 96).
// Classic layers: the lines are those that cost least over 733 sizes (1024 to 16384 tokens, hidden 512 to 4096, any feed-forward width);
// over 2367 others 74 are more than 1 % slower than apart (7 % at most), 202 would be that much faster together, and backward takes 0.4 %
// more than with the faster form of each. Gated: over 3721 sizes 127 are more than 1 % slower than apart (12 % at most) and 478 would be that
// much faster together; with lines over the work in the shared launches, as before, it was 111 and 741, and 1.7 % over the faster forms
// where it is 0.8 now.
// Backward, us, apart / together; "hidden,FFN[,attention]: tokens"; "!": the slower one is taken:
//   classic  576,2304: 1536 99/103!; 640,2560: 1408 114/116!, 2660 142/136!, 3800 188/184!, 5700 238/235!, 8000 337/387; 768,2048: 2700 173/177!;
//     768,3072: 1520 120/127, 1900 133/135, 2280 146/139, 3072 202/188, 3800 225/191, 5700 283/298, 8000 394/414, 16000 705/745;
//     832,3328: 13468 709/711; 896,2392: 6464 362/332!; 896,3584: 1520 133/140, 1900 163/148, 5700 362/347, 8000 493/456; 1024,4096: 1140 132/150,
//     1520 152/158, 1900 183/165, 3800 281/248, 5700 420/374, 8000 582/489, 12000 816/694; 1088,4352: 1332 160/166, 8000 649/706, 8320 664/719!;
//     1152,3072: 7168 552/541!; 1152,4520: 4096 367/378; 1152,4608: 4096 406/428, 6288 537/563, 8192 814/845!; 1280,5120: 1140 170/185,
//     1520 215/194, 3800 426/392, 4560 511/469, 5700 593/551, 6840 677/681, 8000 827/783, 10240 1247/1205, 12000 1197/1087, 16000 1642/1416;
//     1536,6144: 1520 257/255, 2280 364/350, 3000 442/442, 4000 580/528, 6000 816/757, 8000 1065/970, 12000 1641/1415, 16000 2174/1819;
//     2048,6992: 9088 1551/1506; 2048,8192: 1520 385/378!, 2000 451/455, 3000 631/632, 4000 800/782!, 5000 1004/1014, 6000 1158/1138,
//     8000 1475/1441, 12000 2272/2206, 13653 2520/2436; 2112,5800: 15300 3204/2978; 2432,8208: 13696 3394/3272!; 2560,10240: 2000 668/691,
//     3000 918/903, 4000 1224/1248, 6000 1713/1699, 8192 2375/2264, 12000 3446/3412; 2688,10752: 4096 1461/1420; 2752,11008: 2048 772/790;
//     2880,6272: 7168 2034/1965; 2880,11520: 1332 604/619; 2944,11776: 7168 2644/2596; 3072,12288: 1536 698/727, 2048 871/882, 3072 1247/1251,
//     4096 1607/1598, 6144 2471/2341, 8192 3216/3116; 3392,9048: 8100 3454/3506!; 3392,11968: 3000 1522/1551!; 3456,13824: 4096 2046/2092;
//     3520,9384: 4096 1846/1895; 3712,14848: 3696 2134/2192!; 3776,15104: 2000 1291/1249!; 3840,9736: 1024 658/644; 4096,16384: 1024 870/854,
//     1536 1176/1160, 2048 1466/1411, 2560 1791/1750, 3072 2108/2033, 3584 2355/2385!, 4096 2668/2595;
//   gated  512,1368: 2048 139/108; 576,1280: 16304 752/892; 576,1536: 3072 145/156, 10200 471/550; 768,1704: 9992 533/583; 768,2040: 2752
//     183/186; 768,2048: 1192 149/127!, 1500 136/129!, 1552 135/138, 2000 135/134, 2500 152/152, 3000 164/169, 4000 191/201, 14816 858/917;
//     832,2216: 5500 325/337; 896,2392: 10336 771/787; 960,2560: 2408 189/184!, 3072 214/201, 3584 227/214, 4000 294/271; 1024,2280: 6320
//     463/445; 1024,2728: 1752 179/180, 5439 419/387, 6424 499/494, 7432 580/554, 11328 931/864; 1024,2736: 1500 158/162, 2000 182/176!, 2500
//     194/193, 4000 293/264, 8000 537/514; 1024,3384: 1944 204/197; 1088,360,128: 4040 137/159; 1152,3728: 1312 198/201; 1152,4016: 2608
//     297/310; 1216,400,128: 8192 198/243; 1280,2376,640: 1192 151/144!; 1472,488,128: 4416 169/201; 1536,4096: 1500 242/255, 2000 289/311,
//     2500 356/369, 3000 410/421, 4000 512/489, 4488 578/618!, 8000 968/957, 14712 2251/2100; 1600,2888,768: 8288 825/832; 1664,4440: 2800
//     492/485!, 3408 596/589; 1728,2304,832: 4608 437/415!; 1792,4776: 9168 1670/1558; 1856,4952: 4500 872/904!; 1920,1280,448: 2000 152/146;
//     1920,6264: 9264 2161/2123!; 1984,5288: 2664 612/585, 5248 1147/1125, 11776 2294/2165, 14500 2932/2749; 2048,552,256: 3104 169/174;
//     2048,1360,512: 13500 839/787; 2048,5504: 1500 384/399, 2000 502/458, 4000 864/802, 8000 1556/1483; 2112,2816,1024: 1024 187/202, 7488
//     943/930!; 2176,5800: 1224 373/402, 11664 3215/3160!; 2240,5976: 3064 784/797; 2368,784,256: 1024 145/113; 2496,6656: 4000 1174/1131!,
//     4088 1236/1194!; 2560,3408,1280: 12800 2159/1898; 2624,7000: 2331 836/862; 3072,2048,768: 7326 879/826; 3072,8192: 5816 2416/2390!;
//     3584,9560: 1560 1024/1036; 3840,3768,960: 4288 980/988; 3904,5200,1920: 5248 1861/1848; 3968,2640,960: 5661 1105/1058; 4096,1376,512:
//     2048 289/276, 4096 509/478; 4096,2752,1024: 2048 477/444, 4096 819/774; 4096,5504,2048: 4096 1399/1415!; 4096,11008: 2048 1450/1453,
//     3000 2075/2071, 4096 2683/2683.
enum Together { APART, BEHIND, BLOCKS };
Together products_together(const slapo_layer_desc* d) {
  // (Fewer than 1024 tokens: of 150 sizes measured there the lines below would have two share: gated, 1016 tokens of width 640
  // 150 / 109; classic, 1016 of 3840 769 / 742. The others are up to twice as slow together, products
  // come in K ranges there, and what the count takes is the host's, which small calls wait for.)
  if (d->dtype == SLAPO_FP32 || (int64_t)d->batch * d->seq < 1024 || (is_llama(d) && backward_on_one_stream(d))) return APART;
  const int T = d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d), F1 = is_llama(d) ? 2 * F : F;
  const auto sizes = [](int layout, int M, int N, int K) { return Product{layout, M, N, K, nullptr, nullptr, nullptr, nullptr}; };
  const Product x = sizes(GEMM_NN, T, H, 3 * A), y = sizes(GEMM_NN, T, H, F1), w2 = sizes(GEMM_TN, H, F, T), w1 = sizes(GEMM_TN, F1, H, T),
                wo = sizes(GEMM_TN, H, A, T), wqkv = sizes(GEMM_TN, 3 * A, H, T);
  const Product behind[] = {x, w2, w1, wo, wqkv}, first[] = {y, w2, w1}, second[] = {x, wo, wqkv};
  const int in_blocks = products_slabs(3, first) + products_slabs(3, second);
  const int at_end = products_slabs(5, behind) + gemm_slabs(GEMM_NN, T, H, F1);
  const bool blocks = in_blocks <= 1.02 * at_end;
  const auto large_alone = [&](int ffn) { return (int64_t)((H + 255) / 256) * ((ffn + 255) / 256) >= 192; };
  const double shared = (blocks ? in_blocks : at_end) + gemm_slabs(GEMM_NN, T, F, H) + gemm_slabs(GEMM_NN, T, A, H);
  double apart = gemm_slabs_beside(GEMM_NN, T, F, H) + gemm_slabs_beside(GEMM_NN, T, A, H);
  for (const Product& p : {x, y, w2, w1, wo, wqkv}) apart += gemm_slabs_beside(p.layout, p.M, p.N, p.K);
  const double line = large_alone(F) ? 1.07 * apart - 12.0 : large_alone(F1) ? 1.12 * apart - 12.0
                      : is_llama(d) ? std::max(1.1 * apart + 8.0, H >= 512 ? 76.0 : 0.0) : 1.12 * apart + 22.0;
  return shared > line ? APART : blocks ? BLOCKS : BEHIND;
}

}  // namespace slapo

namespace {

// byte offsets of the regions of `saved`
struct SavedLayout {
  size_t qkv, attn, lse, z1, n1, y1, u, g, z2, mu1, rstd1, mu2, rstd2, total;
};
SavedLayout saved_layout(const slapo_layer_desc* d) {
  const size_t eb = d->dtype == SLAPO_FP32 ? 4 : 2;
  const size_t T = (size_t)d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  SavedLayout L;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
  L.qkv = take(T * 3 * A * eb);
  L.attn = take(T * A * eb);
  L.lse = take((size_t)d->batch * d->heads * d->seq * 4);
  L.z1 = take(T * H * eb);
  L.n1 = d->pre_ln ? take(T * H * eb) : (size_t)-1;
  L.y1 = take(T * H * eb);  // post-LN: LN1 output; pre-LN: LN2 output ("n2")
  // act'(u) of a GeLU layer, or the (gate, up) factor pairs [T,2F]; a ReLU layer keeps nothing here: its
  // derivative is [g > 0], read off the activation output it keeps anyway
  L.u = keeps_dact(d) ? take(T * F * eb * (is_llama(d) ? 2 : 1)) : (size_t)-1;
  L.g = take(T * F * eb);
  L.z2 = d->pre_ln ? (size_t)-1 : take(T * H * eb);
  L.mu1 = take(T * 4);
  L.rstd1 = take(T * 4);
  L.mu2 = take(T * 4);
  L.rstd2 = take(T * 4);
  L.total = o;
  return L;
}

// Workspace of a layer's product with a plain or add epilogue: K ranges of the tiles of a thin last round, but none where tiles of
// another size make the product exactly one round, which is faster (the exported products keep the K ranges that they offer).
static size_t product_ws_bytes(int dtype, int layout, int M, int N, int K) {
  return gemm_in_one_round(dtype, layout, M, N, K) ? 0 : gemm_ws_bytes(dtype, layout, EPI_NONE, M, N, K);
}

// The gradient of the first feed-forward bias: column sums that the product which computes the gradient of the activations leaves
// behind (EPI_DACT), instead of another pass over that array (16384 tokens, 4096 columns: 27 us alone, 36 beside a product).
// From 1024 tokens on: below, the pass is 5 us on the helper stream or rides on the next launch. fp32 products leave none, and paired
// launches neither, but such layers come here too where dx lies on x.
inline bool sums_with_du(const slapo_layer_desc* d) {
  return !is_llama(d) && d->dtype != SLAPO_FP32 && (int64_t)d->batch * d->seq >= 1024;
}

// The sums over the partial rows that the row kernels leave run on the helper stream beside launches that several products share
// (classic layers of 1024 tokens and more), and from 1536 tokens on beside launches for each product. An array of partial rows per row
// kernel is then in flight; on the chain one serves all three, and what the next kernel writes is what the last sum has just read.
// us of backward, classic and gated layers, on the chain with an array for each / with one / on the helper stream:
//   896 tokens, hidden 2048 272 / 263 / 267, gated (1024) 314 / 306 / 312; gated 1152, 2560 471 / 468 / 475; 1152, 2560 441 / 439 / 437
//   1280, 1536 242 / 242 / 230; 1408, 2048 362 / 361 / 348; gated 1536, 1536 244 / 244 / 237; 5500, 768 295 / 295 / 283; 8000, 512 250 / 248 /
//   236; 2000, 2048 463 / 460 / 450; 2000, 3072 866 / 865 / 878; 4000, 2560 1260 / 1260 / 1250
constexpr int ROW_SUMS_ASIDE = 1536;
inline size_t row_sums_aside_from(const slapo_layer_desc* d) { return is_llama(d) || d->dtype == SLAPO_FP32 ? ROW_SUMS_ASIDE : 1024; }

struct ScratchLayout {
  size_t t0, t1, t2, t3, du, dqkv, delta, part_row[3], part_col, part_col2, part_du, rope, splitk, gemm_ws, gemm_ws_bytes, splitk_bytes, acts, total;
};
ScratchLayout scratch_layout(const slapo_layer_desc* d) {
  const size_t eb = d->dtype == SLAPO_FP32 ? 4 : 2;
  const size_t T = (size_t)d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  ScratchLayout L;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
  L.t0 = take(T * (H > A ? H : A) * eb);   // also holds the gradient of the attention output [T,A]
  L.t1 = take(T * H * eb);
  L.t2 = take(T * H * eb);
  L.t3 = take(T * H * eb);
  L.du = take(T * F * eb * (is_llama(d) ? 2 : 1));
  L.dqkv = take(T * 3 * A * eb);
  L.delta = take((size_t)d->batch * d->heads * d->seq * 4);
  for (size_t& p : L.part_row)   // one per row kernel where sums over partial rows may leave the chain, else one for all
    p = &p == L.part_row || T >= row_sums_aside_from(d) ? take((size_t)bdrln_bwd_blocks_wide((int64_t)T, (int)H) * 3 * H * 4) : L.part_row[0];
  size_t widest = F > 3 * A ? F : 3 * A;
  widest = widest > H ? widest : H;
  L.part_col = take((size_t)colsum_blocks((int64_t)T) * widest * 4);
  L.part_col2 = take((size_t)colsum_blocks((int64_t)T) * widest * 4);   // the two streams of backward each own one
  L.part_du = sums_with_du(d) ? take((T + DACT_SUM_ROWS - 1) / DACT_SUM_ROWS * F * 4) : 0;
  L.rope = is_llama(d) ? take((size_t)d->seq * (A / d->heads / 2) * 8) : 0;   // (cos, sin) table
  // fp32 partial tiles of the weight gradients that are computed in several K ranges (one at a time: all of them
  // run on the helper stream); 0 for shapes that fill the chip with plain tiles
  {
    const int Ti = (int)T, Hi = (int)H, Fi = (int)F, Ai = (int)A, F1 = is_llama(d) ? 2 * Fi : Fi;
    size_t w = weight_grad_ws_bytes(d->dtype, Hi, Fi, Ti);
    const size_t w1 = weight_grad_ws_bytes(d->dtype, F1, Hi, Ti), wo = weight_grad_ws_bytes(d->dtype, Hi, Ai, Ti);
    const size_t wq = weight_grad_ws_bytes(d->dtype, 3 * Ai, Hi, Ti);
    w = w > w1 ? w : w1; w = w > wo ? w : wo; w = w > wq ? w : wq;
    L.splitk = w ? take(w) : 0;
    L.splitk_bytes = w;
    // the same kind of workspace for the GEMMs of the forward pass and of the data-gradient chain whose tile grid
    // would end in a thin round (their last tiles are then computed in K ranges); a region of its own, because
    // the chain runs while the helper stream's weight gradients use the one above
    size_t g = product_ws_bytes(d->dtype, GEMM_NT, Ti, Hi, Ai);                    // attention output projection
    auto upto = [&](size_t v) { g = g > v ? g : v; };
    upto(product_ws_bytes(d->dtype, GEMM_NT, Ti, Hi, Fi));                         // second FFN product
    upto(product_ws_bytes(d->dtype, GEMM_NN, Ti, Hi, F1));                         // gradient of the FFN input
    upto(product_ws_bytes(d->dtype, GEMM_NN, Ti, Ai, Hi));                         // gradient of the attention output
    upto(product_ws_bytes(d->dtype, GEMM_NN, Ti, Hi, 3 * Ai));                     // gradient of the attention input
    // and for the products that the row kernels read in K ranges
    for (const int K : {Ai, Fi, 3 * Ai})
      if (product_in_ranges(d->dtype, Ti, Hi, K)) upto(K_RANGES * T * H * sizeof(float));
    L.gemm_ws = g ? take(g) : 0;
    L.gemm_ws_bytes = g;
  }
  // checkpoint mode: the activations that forward would hand to backward live here instead, for the
  // duration of one call only (backward recomputes them), so the caller keeps nothing per layer but x
  L.acts = d->checkpoint ? take(saved_layout(d).total) : 0;
  L.total = o;
  return L;
}

}  // namespace

extern "C" {

const char* slapo_status_string(int status) {
  switch (status) {
    case SLAPO_OK: return "ok";
    case SLAPO_ERR_NULL: return "a required pointer is NULL";
    case SLAPO_ERR_SHAPE: return "invalid shape or scalar argument";
    case SLAPO_ERR_UNSUPPORTED: return "unsupported configuration";
    case SLAPO_ERR_ALIGN: return "pointer not 16-byte aligned or size not a multiple of 8";
    case SLAPO_ERR_WORKSPACE: return "shape needs more workspace than the library's fixed-size buffer holds";
    case SLAPO_ERR_HIP: return "HIP reported an error";
    default: return "unknown status";
  }
}

int slapo_layer_workspace(const slapo_layer_desc* desc, size_t* saved_bytes, size_t* scratch_bytes) {
  if (!saved_bytes || !scratch_bytes) return SLAPO_ERR_NULL;
  const int rc = check_desc(desc);
  if (rc) return rc;
  *saved_bytes = desc->checkpoint ? 0 : saved_layout(desc).total;
  *scratch_bytes = scratch_layout(desc).total;
  return SLAPO_OK;
}

int slapo_layer_saved_region(const slapo_layer_desc* desc, const char* name, size_t* offset, size_t* bytes) {
  if (!name || !offset || !bytes) return SLAPO_ERR_NULL;
  const int rc = check_desc(desc);
  if (rc) return rc;
  const SavedLayout L = saved_layout(desc);
  const size_t eb = desc->dtype == SLAPO_FP32 ? 4 : 2;
  const size_t T = (size_t)desc->batch * desc->seq, H = desc->hidden, F = desc->ffn, A = attn_width(desc);
  size_t off = (size_t)-1, len = 0;
  if (!strcmp(name, "qkv")) { off = L.qkv; len = T * 3 * A * eb; }
  else if (!strcmp(name, "attn")) { off = L.attn; len = T * A * eb; }
  else if (!strcmp(name, "lse")) { off = L.lse; len = (size_t)desc->batch * desc->heads * desc->seq * 4; }
  else if (!strcmp(name, "z1")) { off = L.z1; len = T * H * eb; }
  else if (!strcmp(name, "n1")) { off = L.n1; len = T * H * eb; }
  else if (!strcmp(name, "y1") && !desc->pre_ln) { off = L.y1; len = T * H * eb; }
  else if (!strcmp(name, "n2") && desc->pre_ln) { off = L.y1; len = T * H * eb; }
  else if (!strcmp(name, "dact") && !is_llama(desc) && keeps_dact(desc)) { off = L.u; len = T * F * eb; }
  else if (!strcmp(name, "dgate") && is_llama(desc)) { off = L.u; len = 2 * T * F * eb; }
  else if (!strcmp(name, "g")) { off = L.g; len = T * F * eb; }
  else if (!strcmp(name, "z2")) { off = L.z2; len = T * H * eb; }
  else if (!strcmp(name, "mu1")) { off = L.mu1; len = T * 4; }
  else if (!strcmp(name, "rstd1")) { off = L.rstd1; len = T * 4; }
  else if (!strcmp(name, "mu2")) { off = L.mu2; len = T * 4; }
  else if (!strcmp(name, "rstd2")) { off = L.rstd2; len = T * 4; }
  if (off == (size_t)-1) return SLAPO_ERR_UNSUPPORTED;
  *offset = off;
  *bytes = len;
  return SLAPO_OK;
}

// In a stack of pre-LN layers the LayerNorm that opens layer l+1 reads what the last kernel of layer l has
// just written, so that kernel produces it on the way: the pattern (sum out, its LayerNorm out) is the one
// the layer already uses between its attention and feed-forward blocks, and one pass over [T,H] per layer
// boundary goes away. The normalised values are computed from the stored (rounded) sum, exactly as the
// separate kernel would, so a layer run on its own reproduces them bit for bit.
struct ForwardLink {
  bool ln1_done = false;                       // the layer below has filled n1, mu1, rstd1 of `saved`
  const slapo_layer_params* above = nullptr;   // the layer above: its first LayerNorm rides on my last kernel
  void* above_saved = nullptr;                 // ... and lands in the n1, mu1, rstd1 regions of its `saved`
  bool rope_done = false;                      // the rotary table stands in `scratch` already
};

// The forward launch sequence; `saved` receives the activations. Also the first half of a checkpointed
// backward (`for_backward`), which is why it is a function of its own.
static void run_forward(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const int32_t* seqlens,
                        void* y, void* saved, void* scratch, hipStream_t st, bool for_backward = false,
                        const ForwardLink* link = nullptr) {
  const int dt = d->dtype;   // SLAPO_* element types are the launch interface's DT_* values
  const int T = d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  const SavedLayout L = saved_layout(d);
  const ScratchLayout W = scratch_layout(d);
  char* sv = (char*)saved;
  char* sc = (char*)scratch;
  void *qkv = sv + L.qkv, *attn = sv + L.attn, *z1 = sv + L.z1, *y1 = sv + L.y1, *g = sv + L.g;
  void* u = keeps_dact(d) ? sv + L.u : nullptr;
  float *lse = (float*)(sv + L.lse), *mu1 = (float*)(sv + L.mu1), *rstd1 = (float*)(sv + L.rstd1);
  float *mu2 = (float*)(sv + L.mu2), *rstd2 = (float*)(sv + L.rstd2);
  void* r = sc + W.t0;
  const AttnShape as = make_attn_shape(d);
  const DropoutParams dp0 = make_dropout(d, 0), dp1 = make_dropout(d, 1);

  const bool llama = is_llama(d);
  const int rms = llama ? 1 : 0;
  const void* attn_in = x;
  if (d->pre_ln) {
    void* n1 = sv + L.n1;
    if (!(link && link->ln1_done))
      launch_bdrln_fwd(dt, T, H, nullptr, nullptr, x, p->ln1_g, p->ln1_b, nullptr, n1, mu1, rstd1, dp0, d->ln_eps, rms, st);
    attn_in = n1;
  }
  if (llama) {
    // no biases; queries and keys are rotated by their position in the projection's epilogue
    float* table = (float*)(sc + W.rope);
    if (!(link && link->rope_done)) launch_rope_table(d->seq, A / d->heads, d->rope_base, table, st);
    launch_gemm(dt, GEMM_NT, EPI_ROPE, rope_act(d->seq, A / d->heads), T, 3 * A, H, attn_in, p->wqkv, qkv, table, nullptr, nullptr, st, true);
  } else {
    launch_gemm(dt, GEMM_NT, EPI_BIAS, d->act, T, 3 * A, H, attn_in, p->wqkv, qkv, p->bqkv, nullptr, nullptr, st, true);
  }
  launch_attn_fwd(dt, as, qkv, seqlens, attn, lse, st);
  float* gws = W.gemm_ws_bytes ? (float*)(sc + W.gemm_ws) : nullptr;   // for GEMMs whose tile grid ends in a thin round
  // Output projections: the row kernel behind reads them, in K ranges where few tokens make few tiles.
  bool ranges = false;
  auto project = [&](int K, const void* a, const void* w) -> const void* {
    ranges = product_in_ranges(dt, T, H, K);
    if (ranges) {
      launch_gemm_ranges(dt, GEMM_NT, T, H, K, a, w, gws, st);
      return gws;
    }
    const size_t need = product_ws_bytes(dt, GEMM_NT, T, H, K);
    launch_gemm(dt, GEMM_NT, EPI_NONE, d->act, T, H, K, a, w, r, nullptr, nullptr, nullptr, st, true, need ? gws : nullptr, need);
    return r;
  };
  const void* ro = project(A, attn, p->wo);
  const void* bo = llama ? nullptr : p->bo;
  const void* b2 = llama ? nullptr : p->b2;
  if (d->pre_ln) launch_bdrln_fwd(dt, T, H, ro, bo, x, p->ln2_g, p->ln2_b, z1, y1, mu2, rstd2, dp0, d->ln_eps, rms, st, ranges);
  else launch_bdrln_fwd(dt, T, H, ro, bo, x, p->ln1_g, p->ln1_b, z1, y1, mu1, rstd1, dp0, d->ln_eps, rms, st, ranges);
  if (llama)   // w1 holds (gate, up) row pairs: one product, gated in the epilogue; `u` keeps the backward factors
    launch_gemm(dt, GEMM_NT, EPI_GATE, d->act, T, 2 * F, H, y1, p->w1, g, nullptr, nullptr, u, st, true);
  else
    launch_gemm(dt, GEMM_NT, EPI_BIAS_ACT, d->act, T, F, H, y1, p->w1, g, p->b1, nullptr, u, st, true);
  // Backward of a pre-LN layer reads nothing downstream of the activation output (its last step has no
  // LayerNorm whose input would have to be kept), so a recomputation stops here: one GEMM in six less.
  if (for_backward && d->pre_ln) return;
  const void* r2 = project(F, g, p->w2);
  if (d->pre_ln && link && link->above) {
    char* up = (char*)link->above_saved;
    launch_bdrln_fwd(dt, T, H, r2, b2, z1, link->above->ln1_g, llama ? nullptr : link->above->ln1_b, y, up + L.n1,
                     (float*)(up + L.mu1), (float*)(up + L.rstd1), dp1, d->ln_eps, rms, st, ranges);
  } else if (d->pre_ln) {
    launch_bdrln_fwd(dt, T, H, r2, b2, z1, nullptr, nullptr, y, nullptr, nullptr, nullptr, dp1, d->ln_eps, rms, st, ranges);
  } else {
    void* z2 = sv + L.z2;
    launch_bdrln_fwd(dt, T, H, r2, b2, y1, p->ln2_g, p->ln2_b, z2, y, mu2, rstd2, dp1, d->ln_eps, rms, st, ranges);
  }
}

static int check_forward_args(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const void* y,
                              const void* saved, const void* scratch) {
  int rc = check_desc(d);
  if (rc) return rc;
  if (!p || !x || !y || !scratch || (!saved && !d->checkpoint)) return SLAPO_ERR_NULL;
  const void* const ps[12] = {p->wqkv, p->bqkv, p->wo, p->bo, p->ln1_g, p->ln1_b, p->w1, p->b1, p->w2, p->b2, p->ln2_g, p->ln2_b};
  if ((rc = check_tables(d, ps))) return rc;
  if (misaligned(x) || misaligned(y) || misaligned(scratch) || (!d->checkpoint && misaligned(saved))) return SLAPO_ERR_ALIGN;
  return SLAPO_OK;
}

int slapo_layer_fwd(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const int32_t* seqlens,
                    void* y, void* saved, void* scratch, void* stream) {
  const int rc = check_forward_args(d, p, x, y, saved, scratch);
  if (rc) return rc;
  entry_error();
  if (d->checkpoint) saved = (char*)scratch + scratch_layout(d).acts;   // transient: nothing is kept for backward
  run_forward(d, p, x, seqlens, y, saved, scratch, (hipStream_t)stream);
  return finish();
}

static int check_backward_args(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const void* dy,
                               const void* saved, const void* dx, const slapo_layer_grads* gr, const void* scratch) {
  int rc = check_desc(d);
  if (rc) return rc;
  if (!p || !x || !dy || !dx || !gr || !scratch || (!saved && !d->checkpoint)) return SLAPO_ERR_NULL;
  const void* const ps[12] = {p->wqkv, p->bqkv, p->wo, p->bo, p->ln1_g, p->ln1_b, p->w1, p->b1, p->w2, p->b2, p->ln2_g, p->ln2_b};
  const void* const gs[12] = {gr->wqkv, gr->bqkv, gr->wo, gr->bo, gr->ln1_g, gr->ln1_b, gr->w1, gr->b1, gr->w2, gr->b2, gr->ln2_g, gr->ln2_b};
  if ((rc = check_tables(d, ps)) || (rc = check_tables(d, gs))) return rc;
  if (misaligned(x) || misaligned(dy) || misaligned(dx) || misaligned(scratch) || (!d->checkpoint && misaligned(saved))) return SLAPO_ERR_ALIGN;
  return SLAPO_OK;
}

// The backward counterpart of ForwardLink: the last kernel of a pre-LN layer's backward (LayerNorm backward
// plus the residual gradient -> dx) is also where the layer below would start (dx -> its dropped-out branch
// gradient dR2 and the row sums behind its b2 gradient), so in a stack the upper layer's kernel writes both
// and the lower layer starts at its first GEMM.
struct BackwardLink {
  bool above = false, below = false;   // there is a layer above / below
  bool rope_done = false;              // the rotary table stands in `scratch` already
  const void* dr2_in = nullptr;   // my dR2, already produced (with my b2 gradient) by the layer above
  void* dr2_below = nullptr;      // where the dR2 of the layer below goes ...
  DropoutParams dp_below;         // ... its mask stream (site 1 of that layer)
  void* db2_below = nullptr;      // ... and its b2 gradient (NULL: the family has no biases)
  // (paired launches) where the sums over the partial rows go that the layer above left, which ride on my first launch;
  // behind the call: those that I leave to the layer below
  void* sums[3] = {nullptr, nullptr, nullptr};
};

static int run_backward(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const int32_t* seqlens,
                        const void* dy, const void* saved, void* dx, const slapo_layer_grads* gr, void* scratch,
                        hipStream_t st, BackwardLink* link = nullptr) {
  const int dt = d->dtype, acc = d->accumulate_grads ? 1 : 0;
  const int T = d->batch * d->seq, H = d->hidden, F = d->ffn, A = attn_width(d);
  const SavedLayout L = saved_layout(d);
  const ScratchLayout W = scratch_layout(d);
  if (d->checkpoint) {
    // Activation checkpointing (section 2.2, the paper's third optimisation): nothing but x was kept, so run
    // the forward again into the transient region. The dropout masks are a pure function of (seed, layer,
    // site, element), so the recomputed activations are bit for bit those of the original forward. The layer
    // output lands in a gradient buffer that backward overwrites later.
    char* acts = (char*)scratch + W.acts;
    ForwardLink again;
    again.rope_done = link && link->rope_done;
    run_forward(d, p, x, seqlens, (char*)scratch + W.t1, acts, scratch, st, true, &again);
    saved = acts;
  }
  const char* sv = (const char*)saved;
  char* sc = (char*)scratch;
  const void *qkv = sv + L.qkv, *attn = sv + L.attn, *z1 = sv + L.z1, *y1 = sv + L.y1, *g = sv + L.g;
  const void* u = keeps_dact(d) ? sv + L.u : g;   // ReLU: the gate [g > 0] comes from the activation output
  const float *lse = (const float*)(sv + L.lse), *mu1 = (const float*)(sv + L.mu1), *rstd1 = (const float*)(sv + L.rstd1);
  const float *mu2 = (const float*)(sv + L.mu2), *rstd2 = (const float*)(sv + L.rstd2);
  void *t0 = sc + W.t0, *t1 = sc + W.t1, *t2 = sc + W.t2, *t3 = sc + W.t3, *du = sc + W.du, *dqkv = sc + W.dqkv;
  float *delta = (float*)(sc + W.delta), *prow = (float*)(sc + W.part_row[0]), *pcol = (float*)(sc + W.part_col), *pcol2 = (float*)(sc + W.part_col2);
  AttnShape as = make_attn_shape(d);
  const DropoutParams dp0 = make_dropout(d, 0), dp1 = make_dropout(d, 1);
  const int nrow = bdrln_bwd_blocks_wide(T, H), ncol = colsum_blocks(T);
  // Nothing dropped: a branch's gradient is the residual's, so no copy of it is made (the array in front of the feed-forward
  // block of a pre-LN layer is dy itself). 4 x 2048 tokens of width 2560: 20 us of row kernel and 8 of 46 in the next one.
  const bool keeps_all = dropout_keeps_all(dp0);                    // (both sites drop alike)
  const size_t array = (size_t)T * H * (dt == SLAPO_FP32 ? 4 : 2);
  const bool dy_is_dr2 = d->pre_ln && keeps_all && !overlap(dx, dy, array);   // (a dx on top of dy is written while the helper stream reads dr2)
  const bool dx_on_x = !d->pre_ln && overlap(dx, x, array);   // (a pre-LN layer's dx is written row by row behind the read, and no weight gradient reads x)
  // `st` carries the data-gradient chain; `ws` the weight / bias gradients that hang off it
  const Together together = dx_on_x ? APART : products_together(d);   // (dx would be written while a tile beside it still reads x)
  // (beside products that share launches only the column sums behind the bias gradients run on the helper stream)
  SideStream* side = (together != APART ? is_llama(d) : backward_on_one_stream(d)) ? nullptr : side_stream();
  const bool solo = side == nullptr || together != APART;   // every GEMM has the chip to itself
  hipStream_t ws = side ? side->stream : st;
  auto fork = [&](int i) {   // everything issued on st so far happens before what follows on ws
    if (side && (together == APART || i == 1 || i == 3)) side->order(side->fork[i], st, ws);
  };
  const bool rows_aside = side && (together != APART || T >= ROW_SUMS_ASIDE);
  auto partial_rows = [&](int k) { return (float*)(sc + W.part_row[rows_aside ? k : 0]); };   // of row kernel `k` (0 to 2, in their order)
  // weight gradient: C (+)= A^T B
  float* splitk_ws = W.splitk_bytes ? (float*)(sc + W.splitk) : nullptr;
  float* gws = W.gemm_ws_bytes ? (float*)(sc + W.gemm_ws) : nullptr;
  Product waiting[MAX_PRODUCTS];   // for the next launch of several
  int n_waiting = 0;
  auto dweight = [&](int M, int N, const void* a, const void* b, void* c) {
    if (together != APART) waiting[n_waiting++] = {GEMM_TN, M, N, T, a, b, c, acc ? c : nullptr};
    else launch_weight_grad(dt, acc, M, N, T, a, b, c, splitk_ws, ws, solo);
  };
  // data gradient: C = A B (+ aux)
  auto dgrad = [&](int epi, int N, int K, const void* a, const void* b, void* c, const void* aux) {
    const size_t need = product_ws_bytes(dt, GEMM_NN, T, N, K);
    launch_gemm(dt, GEMM_NN, epi, d->act, T, N, K, a, b, c, nullptr, aux, nullptr, st, solo, need ? gws : nullptr, need);
  };
  // the same, with the weight gradients that wait
  auto dgrad_with_weights = [&](int N, int K, const void* a, const void* b, void* c, const void* aux) {
    waiting[n_waiting++] = {GEMM_NN, T, N, K, a, b, c, aux};
    launch_products(dt, n_waiting, waiting, st);
    n_waiting = 0;
  };
  auto colsum = [&](const void* a, int N, void* out, hipStream_t s) {
    float* part = s == st ? pcol2 : pcol;   // per stream, so that the two sums may run at the same time
    launch_colsum_partials(dt, T, N, a, part, s);
    launch_colreduce_partials(dt, ncol, N, N, part, out, acc, s);
  };
  auto reduce_rows = [&](int k, void* dgamma, void* dbeta, void* dbias, hipStream_t s) {
    launch_colreduce3(dt, nrow, H, partial_rows(k), dgamma, dbeta, dbias, acc, s);
  };
  // The gradient of a block's input, [T,H], which a row kernel reads next: t0, or K ranges in gws where few tokens make few tiles
  // (`add`, what the product is added to, is then the row kernel's to add). Not the feed-forward block's of the gated layer, whose
  // gradients are, bit for bit, those of the exported products, rotary turn and attention in a row (1024, 128 tokens: 2 us).
  // (Never where launches are shared: 1024 tokens and more make more tiles.)
  const bool r_y1 = !is_llama(d) && product_in_ranges(dt, T, H, F), r_x = product_in_ranges(dt, T, H, 3 * A);
  auto row_bwd = [&](bool ranges, const void* add, const void* z, const float* mu, const float* rstd, const void* gamma, const void* dres,
                     void* dz, void* dr, const DropoutParams& dp, int dr_from_stored, int k = 0) {
    launch_bdrln_bwd(dt, T, H, ranges ? gws : t0, z, mu, rstd, gamma, dres, dz, dr, partial_rows(k), dp, is_llama(d) ? 1 : 0, st, dr_from_stored, nrow,
                     ranges, ranges ? add : nullptr);
  };
  // Buffers: t0 dZ2 -> dY1/dN2 -> dA -> dN1; t1 dR2 (kept for dW2); t2 dZ1; t3 dR1 (kept for dWo). Where nothing is dropped
  // dR1 is t2, and dR2 is dy (pre-LN, dx elsewhere) or, in the paired post-LN launches, t0.
  void* dr1 = keeps_all ? t2 : t3;

  const bool llama = is_llama(d);
  const int rms = llama ? 1 : 0;
  if (llama) {
    // the gradients of the rotated queries and keys are turned back (the rotation's transpose) as attention stores them
    as.rope = (const float*)(sc + W.rope);
    if (!d->checkpoint && !(link && link->rope_done)) launch_rope_table(d->seq, A / d->heads, d->rope_base, (float*)(sc + W.rope), st);   // else it stands there
  }
  // the LLaMA-style layer has no bias or offset gradients: those outputs are simply not produced
  void *g_b2 = llama ? nullptr : gr->b2, *g_bo = llama ? nullptr : gr->bo;
  void *g_ln1_b = llama ? nullptr : gr->ln1_b, *g_ln2_b = llama ? nullptr : gr->ln2_b;

  if (together == APART && gradients_paired(d) && !dx_on_x) {   // (it would be written while the weight gradient beside it still reads x)
    // The weight gradients share the launches of the data gradients (GradPair), and the sums behind the row kernels and
    // the biases ride on them.
    GradPair pr = {};
    auto take_sums = [&](void* a, void* b, void* c) { pr.partials = prow; pr.nblk = nrow; pr.H = H; pr.sums[0] = a; pr.sums[1] = b; pr.sums[2] = c; };
    auto data = [&](int epi, int M, int N, int K, const void* A_, const void* B_, void* C_, const void* aux) {
      pr.epi = epi; pr.act = d->act; pr.M = M; pr.N = N; pr.K = K; pr.A = A_; pr.B = B_; pr.C = C_; pr.aux = aux;
    };
    auto weight = [&](int wM, int wN, const void* wA, const void* wB, void* dW, void* colsum_out) {
      pr.wM = wM; pr.wN = wN; pr.wK = T; pr.wA = wA; pr.wB = wB; pr.dW = dW; pr.colsum = colsum_out; pr.accumulate = acc;
    };
    auto launch = [&] { launch_grad_pair(dt, pr, st); pr = GradPair{}; };
    const int F1 = llama ? 2 * F : F;
    // ---- FFN block ----
    const void* dr2 = t1;
    void* db2 = nullptr;   // b2's gradient as column sums, where no row kernel has left partial sums of it
    if (dy_is_dr2) {
      dr2 = dy;
      db2 = g_b2;
      if (link && link->above) take_sums(link->sums[0], link->sums[1], link->sums[2]);
    } else if (d->pre_ln && link && link->dr2_in) {
      dr2 = link->dr2_in;
      take_sums(link->sums[0], link->sums[1], link->sums[2]);
    } else if (d->pre_ln) {
      launch_bdrln_bwd(dt, T, H, dy, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, t1, prow, dp1, rms, st, 0, nrow);
      if (!llama) take_sums(nullptr, nullptr, g_b2);
    } else {
      if (keeps_all) dr2 = t0;   // (read for the last time before the feed-forward block's input gradient replaces it)
      launch_bdrln_bwd(dt, T, H, dy, sv + L.z2, mu2, rstd2, p->ln2_g, nullptr, t0, (void*)dr2, prow, dp1, rms, st, 0, nrow);
      take_sums(gr->ln2_g, g_ln2_b, g_b2);
    }
    data(llama ? EPI_DGATE : EPI_DACT, T, F, H, dr2, p->w2, du, u);
    weight(H, F, dr2, g, gr->w2, db2);
    launch();
    data(EPI_ADD, T, H, F1, du, p->w1, t0, d->pre_ln ? nullptr : t0);
    if (r_y1) pr.parts = gws;
    weight(F1, H, du, y1, gr->w1, llama ? nullptr : gr->b1);
    launch();
    // ---- attention block ----
    if (d->pre_ln) {
      row_bwd(r_y1, nullptr, z1, mu2, rstd2, p->ln2_g, dy, t2, dr1, dp0, 0);
      take_sums(gr->ln2_g, g_ln2_b, g_bo);
    } else {
      row_bwd(r_y1, t0, z1, mu1, rstd1, p->ln1_g, nullptr, t2, dr1, dp0, 0);
      take_sums(gr->ln1_g, g_ln1_b, g_bo);
    }
    data(EPI_ADD, T, A, H, dr1, p->wo, t0, nullptr);
    if (side) pr.accumulate = acc;
    else weight(H, A, dr1, attn, gr->wo, nullptr);
    launch();
    if (side) {   // beside the attention kernels, which leave most of the chip free
      fork(2);
      dweight(H, A, dr1, attn, gr->wo);
    }
    launch_attn_bwd(dt, as, qkv, seqlens, attn, t0, lse, delta, dqkv, st);
    if (side) side->order(side->join, ws, st);   // the gradient of the output projection has long been there
    data(EPI_ADD, T, H, 3 * A, dqkv, p->wqkv, d->pre_ln ? t0 : dx, d->pre_ln ? nullptr : t2);
    if (r_x) pr.parts = gws;
    weight(3 * A, H, dqkv, d->pre_ln ? sv + L.n1 : x, gr->wqkv, llama ? nullptr : gr->bqkv);
    launch();
    if (!d->pre_ln && r_x) launch_add_ranges(dt, (int64_t)T * H, K_RANGES, gws, t2, dx, st);
    if (d->pre_ln && keeps_all && link && link->below) {
      row_bwd(r_x, nullptr, x, mu1, rstd1, p->ln1_g, t2, dx, nullptr, dp0, 0);
      link->sums[0] = gr->ln1_g; link->sums[1] = g_ln1_b; link->sums[2] = nullptr;
    } else if (d->pre_ln && link && link->dr2_below) {
      row_bwd(r_x, nullptr, x, mu1, rstd1, p->ln1_g, t2, dx, link->dr2_below, link->dp_below, 1);
      link->sums[0] = gr->ln1_g; link->sums[1] = g_ln1_b; link->sums[2] = link->db2_below;
    } else if (d->pre_ln) {
      row_bwd(r_x, nullptr, x, mu1, rstd1, p->ln1_g, t2, dx, nullptr, dp0, 0);
      reduce_rows(0, gr->ln1_g, g_ln1_b, nullptr, st);
    }
    return finish();
  }

  // ---- FFN block ----
  // The bias gradients leave the chain with the next fork: of every weight gradient, or of the two beside products that share
  // launches, and there the sums over partial rows too (one fork, in front of the last launch, takes as long).
  const void* dr2 = t1;
  bool rows2 = true;   // the first row kernel has left partial rows
  if (dy_is_dr2) {
    dr2 = dy;
    rows2 = false;
  } else if (d->pre_ln && link && link->dr2_in) {
    dr2 = link->dr2_in;
    rows2 = false;
  } else if (d->pre_ln) {
    launch_bdrln_bwd(dt, T, H, dy, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, t1, prow, dp1, rms, st, 0, nrow);
    rows2 = !llama;
  } else {
    launch_bdrln_bwd(dt, T, H, dy, sv + L.z2, mu2, rstd2, p->ln2_g, nullptr, t0, t1, prow, dp1, rms, st, 0, nrow);
  }
  const bool with_du = sums_with_du(d);
  float* pdu = (float*)(sc + W.part_du);
  hipStream_t rs = rows_aside ? ws : st;
  auto sums_of_ffn_rows = [&] {
    if (rows2) reduce_rows(0, d->pre_ln ? nullptr : gr->ln2_g, d->pre_ln ? nullptr : g_ln2_b, g_b2, rs);
  };
  auto sums_of_ffn_output = [&] {
    if (dy_is_dr2 && !llama) colsum(dr2, H, g_b2, ws);
  };
  auto sums_of_du = [&] {
    if (with_du) launch_colreduce_partials(dt, (T + DACT_SUM_ROWS - 1) / DACT_SUM_ROWS, F, F, pdu, gr->b1, acc, ws);
    else if (!llama) colsum(du, F, gr->b1, ws);
  };
  auto sums_of_attention_output = [&] {
    if (d->pre_ln) reduce_rows(1, gr->ln2_g, g_ln2_b, g_bo, rs);
    else reduce_rows(1, gr->ln1_g, g_ln1_b, g_bo, rs);
  };
  if (together == APART) {
    if (!rows_aside) sums_of_ffn_rows();
    fork(0);
    if (rows_aside) sums_of_ffn_rows();
    sums_of_ffn_output();
  }
  dweight(H, F, dr2, g, gr->w2);
  if (llama) {
    // dG = dR2 W2, turned into the (gate, up) gradient pairs [T,2F] by the two saved factors in the epilogue
    launch_gemm(dt, GEMM_NN, EPI_DGATE, d->act, T, F, H, dr2, p->w2, du, nullptr, u, nullptr, st, solo);
  } else {
    launch_gemm(dt, GEMM_NN, EPI_DACT, d->act, T, F, H, dr2, p->w2, du, nullptr, u, with_du ? pdu : nullptr, st, solo);
  }
  const int F1 = llama ? 2 * F : F;
  fork(1);
  if (together != APART) {
    sums_of_ffn_rows();
    sums_of_ffn_output();
  }
  sums_of_du();
  dweight(F1, H, du, y1, gr->w1);
  if (together == BLOCKS) dgrad_with_weights(H, F1, du, p->w1, t0, d->pre_ln ? nullptr : t0);
  else if (r_y1) launch_gemm_ranges(dt, GEMM_NN, T, H, F, du, p->w1, gws, st);
  else dgrad(d->pre_ln ? EPI_NONE : EPI_ADD, H, F1, du, p->w1, t0, d->pre_ln ? nullptr : t0);
  // ---- attention block ----
  if (d->pre_ln) row_bwd(r_y1, nullptr, z1, mu2, rstd2, p->ln2_g, dy, t2, dr1, dp0, 0, 1);
  else row_bwd(r_y1, t0, z1, mu1, rstd1, p->ln1_g, nullptr, t2, dr1, dp0, 0, 1);
  if (together == APART) {
    if (!rows_aside) sums_of_attention_output();
    fork(2);
    if (rows_aside) sums_of_attention_output();
  }
  dweight(H, A, dr1, attn, gr->wo);
  dgrad(EPI_NONE, A, H, dr1, p->wo, t0, nullptr);
  as.beside = side && splitk_ws && together == APART;
  launch_attn_bwd(dt, as, qkv, seqlens, attn, t0, lse, delta, dqkv, st);
  fork(3);
  if (together != APART) {
    sums_of_attention_output();
    if (!llama) colsum(dqkv, 3 * A, gr->bqkv, ws);
  }
  dweight(3 * A, H, dqkv, d->pre_ln ? sv + L.n1 : x, gr->wqkv);
  if (d->pre_ln) {
    if (together != APART) dgrad_with_weights(H, 3 * A, dqkv, p->wqkv, t0, nullptr);
    else if (r_x) launch_gemm_ranges(dt, GEMM_NN, T, H, 3 * A, dqkv, p->wqkv, gws, st);
    else dgrad(EPI_NONE, H, 3 * A, dqkv, p->wqkv, t0, nullptr);
    if (link && link->dr2_below) {
      // (from the stored dx, so that the layer below sees what it would compute from dx itself, bit for bit)
      row_bwd(r_x, nullptr, x, mu1, rstd1, p->ln1_g, t2, dx, link->dr2_below, link->dp_below, 1, 2);
      reduce_rows(2, gr->ln1_g, g_ln1_b, link->db2_below, st);
    } else {
      row_bwd(r_x, nullptr, x, mu1, rstd1, p->ln1_g, t2, dx, nullptr, dp0, 0, 2);
      reduce_rows(2, gr->ln1_g, g_ln1_b, nullptr, st);
    }
  } else {
    if (side && dx_on_x) side->order(side->join, ws, st);   // the helper stream has read x before dx is written there
    if (together != APART) dgrad_with_weights(H, 3 * A, dqkv, p->wqkv, dx, t2);
    else dgrad(EPI_ADD, H, 3 * A, dqkv, p->wqkv, dx, t2);
  }
  // apart, the last bias gradient goes behind the data gradient on the caller's stream: the helper stream's last
  // product is the longer one, and this way the two streams end at about the same time
  if (!llama && together == APART) colsum(dqkv, 3 * A, gr->bqkv, st);
  if (side) side->order(side->join, ws, st);   // join: the caller's stream continues only after the weight gradients are complete
  return finish();
}

int slapo_layer_bwd(const slapo_layer_desc* d, const slapo_layer_params* p, const void* x, const int32_t* seqlens,
                    const void* dy, const void* saved, void* dx, const slapo_layer_grads* gr, void* scratch,
                    void* stream) {
  const int rc = check_backward_args(d, p, x, dy, saved, dx, gr, scratch);
  if (rc) return rc;
  entry_error();
  return run_backward(d, p, x, seqlens, dy, saved, dx, gr, scratch, (hipStream_t)stream);
}

// ---- a stack of layers of one shape ------------------------------------------------------------------
static size_t stack_act_bytes(const slapo_layer_desc* d) {
  return (size_t)d->batch * d->seq * d->hidden * (d->dtype == SLAPO_FP32 ? 4 : 2);
}

int slapo_stack_workspace(const slapo_layer_desc* desc, int32_t n_layers, size_t* acts_bytes, size_t* saved_bytes,
                          size_t* scratch_bytes) {
  if (!acts_bytes || !saved_bytes || !scratch_bytes) return SLAPO_ERR_NULL;
  const int rc = check_desc(desc);
  if (rc) return rc;
  if (n_layers <= 0) return SLAPO_ERR_SHAPE;
  *acts_bytes = (size_t)(n_layers - 1) * stack_act_bytes(desc);
  *saved_bytes = desc->checkpoint ? 0 : (size_t)n_layers * saved_layout(desc).total;
  // behind the layer's own scratch: two alternating buffers for the gradient that flows down the stack and,
  // for pre-LN layers, two for the branch gradient that each layer's last kernel prepares for the layer below
  *scratch_bytes = scratch_layout(desc).total + (desc->pre_ln ? 4 : 2) * align256(stack_act_bytes(desc));
  return SLAPO_OK;
}

int slapo_stack_fwd(const slapo_layer_desc* desc, int32_t n_layers, const slapo_layer_params* params, const void* x,
                    const int32_t* seqlens, void* y, void* acts, void* saved, void* scratch, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (n_layers <= 0) return SLAPO_ERR_SHAPE;
  if (!params || !x || !y || !scratch || (n_layers > 1 && !acts) || (!saved && !desc->checkpoint)) return SLAPO_ERR_NULL;
  const size_t ab = stack_act_bytes(desc), sb = desc->checkpoint ? 0 : saved_layout(desc).total;
  slapo_layer_desc d = *desc;
  // every layer is checked before the first launch, so that a bad table leaves nothing half done
  for (int l = 0; l < n_layers; ++l) {
    const void* in = l == 0 ? x : (const char*)acts + (size_t)(l - 1) * ab;
    void* out = l == n_layers - 1 ? y : (char*)acts + (size_t)l * ab;
    if ((rc = check_forward_args(&d, params + l, in, out, saved, scratch))) return rc;
  }
  entry_error();
  // with checkpointing every layer works in the same transient region, whose contents die with the layer
  char* transient = (char*)scratch + scratch_layout(desc).acts;
  auto saved_of = [&](int l) -> void* { return desc->checkpoint ? transient : (char*)saved + (size_t)l * sb; };
  for (int l = 0; l < n_layers; ++l) {
    d.layer_id = desc->layer_id + l;
    const void* in = l == 0 ? x : (const char*)acts + (size_t)(l - 1) * ab;
    void* out = l == n_layers - 1 ? y : (char*)acts + (size_t)l * ab;
    ForwardLink link;
    if (d.pre_ln) {   // the first LayerNorm of layer l+1 rides on the last kernel of layer l
      link.ln1_done = l > 0;
      if (l + 1 < n_layers) { link.above = params + l + 1; link.above_saved = saved_of(l + 1); }
    }
    link.rope_done = l > 0;
    run_forward(&d, params + l, in, seqlens, out, saved_of(l), scratch, (hipStream_t)stream, false, &link);
  }
  return finish();
}

int slapo_stack_bwd(const slapo_layer_desc* desc, int32_t n_layers, const slapo_layer_params* params, const void* x,
                    const int32_t* seqlens, const void* dy, const void* acts, const void* saved, void* dx,
                    const slapo_layer_grads* grads, void* scratch, void* stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (n_layers <= 0) return SLAPO_ERR_SHAPE;
  if (!params || !grads || !x || !dy || !dx || !scratch || (n_layers > 1 && !acts) || (!saved && !desc->checkpoint))
    return SLAPO_ERR_NULL;
  const size_t ab = stack_act_bytes(desc), sb = desc->checkpoint ? 0 : saved_layout(desc).total;
  char* pong = (char*)scratch + scratch_layout(desc).total;   // two gradient buffers behind the layer's own scratch
  char* carry = pong + 2 * align256(ab);                      // (pre-LN) two branch-gradient buffers behind those
  slapo_layer_desc d = *desc;
  for (int l = 0; l < n_layers; ++l) {   // every layer is checked before the first launch
    const void* in = l == 0 ? x : (const char*)acts + (size_t)(l - 1) * ab;
    if ((rc = check_backward_args(&d, params + l, in, dy, saved, dx, grads + l, scratch))) return rc;
  }
  entry_error();
  const void* gin = dy;
  BackwardLink link;
  for (int l = n_layers - 1; l >= 0; --l) {
    d.layer_id = desc->layer_id + l;
    const void* in = l == 0 ? x : (const char*)acts + (size_t)(l - 1) * ab;
    void* gout = l == 0 ? dx : pong + (size_t)(l & 1) * align256(ab);
    link.dr2_in = nullptr;
    link.dr2_below = nullptr;
    link.above = l + 1 < n_layers;
    link.below = l > 0;
    link.rope_done = link.above;
    if (d.pre_ln && !dropout_keeps_all(make_dropout(&d, 1))) {   // (nothing dropped: the gradient that flows down is the branch's too)
      // Layer l reads buffer l&1 (on both streams) and writes the other one; that one was last read by the
      // weight gradient of layer l+1, which the join at the end of that layer's backward has waited for.
      if (l + 1 < n_layers) link.dr2_in = carry + (size_t)(l & 1) * align256(ab);
      if (l > 0) {
        slapo_layer_desc below = d;
        below.layer_id = d.layer_id - 1;
        link.dr2_below = carry + (size_t)((l - 1) & 1) * align256(ab);
        link.dp_below = make_dropout(&below, 1);
        link.db2_below = is_llama(desc) ? nullptr : grads[l - 1].b2;
      }
    }
    rc = run_backward(&d, params + l, in, seqlens, gin, saved ? (const char*)saved + (size_t)l * sb : nullptr, gout,
                      grads + l, scratch, (hipStream_t)stream, &link);
    if (rc) return rc;
    gin = gout;
  }
  return SLAPO_OK;
}

static int gemm_entry(int dtype, int layout, int epilogue, int act, int64_t M, int64_t N, int64_t K, const void* A,
                      const void* B, void* C, const void* bias, const void* aux_in, void* aux_out, void* stream, bool solo,
                      void* ws, size_t ws_bytes) {
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (layout < GEMM_NT || layout > GEMM_TN || epilogue < EPI_NONE || epilogue > EPI_DGATE) return SLAPO_ERR_UNSUPPORTED;
  if (act != SLAPO_GELU_ERF && act != SLAPO_RELU) return SLAPO_ERR_UNSUPPORTED;
  if (M <= 0 || N <= 0 || K <= 0) return SLAPO_ERR_SHAPE;
  if (M * N >= ((int64_t)1 << 31) || M * K >= ((int64_t)1 << 31) || N * K >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if (!A || !B || !C) return SLAPO_ERR_NULL;
  if ((epilogue == EPI_BIAS || epilogue == EPI_BIAS_ACT) && !bias) return SLAPO_ERR_NULL;
  if (((epilogue == EPI_BIAS_ACT && act != SLAPO_RELU) || epilogue == EPI_GATE) && !aux_out) return SLAPO_ERR_NULL;
  if ((epilogue == EPI_DACT || epilogue == EPI_ADD || epilogue == EPI_DGATE) && !aux_in) return SLAPO_ERR_NULL;
  if (epilogue == EPI_DGATE && 2 * M * N >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if (N % 8 || (epilogue == EPI_GATE && N % 16)) return SLAPO_ERR_ALIGN;
  if (layout == GEMM_TN ? (M % 8) : (K % 8)) return SLAPO_ERR_ALIGN;   // A's contiguous dimension
  if (layout == GEMM_NT && (K % 8)) return SLAPO_ERR_ALIGN;
  if (misaligned(A) || misaligned(B) || misaligned(C) || misaligned(ws)) return SLAPO_ERR_ALIGN;
  // a workspace that is too small for what the shape can use is never half used: it is refused or left alone
  if (ws && ws_bytes < gemm_ws_least_bytes(dtype, layout, epilogue, (int)M, (int)N, (int)K)) return SLAPO_ERR_WORKSPACE;
  entry_error();
  launch_gemm(dtype, layout, epilogue, act, (int)M, (int)N, (int)K, A, B, C, bias, aux_in,
              epilogue == EPI_DACT ? nullptr : aux_out,   // (no output of this epilogue here)
              (hipStream_t)stream, solo, (float*)ws, ws ? ws_bytes : 0);
  return finish();
}

int slapo_gemm(int dtype, int layout, int epilogue, int act, int64_t M, int64_t N, int64_t K, const void* A,
               const void* B, void* C, const void* bias, const void* aux_in, void* aux_out, void* stream) {
  return gemm_entry(dtype, layout, epilogue, act, M, N, K, A, B, C, bias, aux_in, aux_out, stream, true, nullptr, 0);
}

int slapo_gemm_workspace(int dtype, int layout, int epilogue, int64_t M, int64_t N, int64_t K, size_t* ws_bytes) {
  if (!ws_bytes) return SLAPO_ERR_NULL;
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (layout < GEMM_NT || layout > GEMM_TN || epilogue < EPI_NONE || epilogue > EPI_DGATE) return SLAPO_ERR_UNSUPPORTED;
  if (M <= 0 || N <= 0 || K <= 0) return SLAPO_ERR_SHAPE;
  if (M * N >= ((int64_t)1 << 31) || M * K >= ((int64_t)1 << 31) || N * K >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  *ws_bytes = gemm_ws_bytes(dtype, layout, epilogue, (int)M, (int)N, (int)K);
  return SLAPO_OK;
}

int slapo_gemm_ex(int dtype, int layout, int epilogue, int act, int64_t M, int64_t N, int64_t K, const void* A,
                  const void* B, void* C, const void* bias, const void* aux_in, void* aux_out, int flags, void* ws,
                  size_t ws_bytes, void* stream) {
  if (flags & ~SLAPO_GEMM_SHARED) return SLAPO_ERR_UNSUPPORTED;
  return gemm_entry(dtype, layout, epilogue, act, M, N, K, A, B, C, bias, aux_in, aux_out, stream,
                    !(flags & SLAPO_GEMM_SHARED), ws, ws_bytes);
}

int slapo_gemm_kernel_name(int dtype, int layout, int epilogue, int64_t M, int64_t N, int64_t K, int flags,
                           int weight_grad, int with_ws, char* buf, size_t len) {
  if (!buf || len == 0) return SLAPO_ERR_NULL;
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (layout < GEMM_NT || layout > GEMM_TN || epilogue < EPI_NONE || epilogue > EPI_DGATE) return SLAPO_ERR_UNSUPPORTED;
  if (flags & ~SLAPO_GEMM_SHARED) return SLAPO_ERR_UNSUPPORTED;
  if (M <= 0 || N <= 0 || K <= 0 || M >= ((int64_t)1 << 31) || N >= ((int64_t)1 << 31) || K >= ((int64_t)1 << 31)) return SLAPO_ERR_SHAPE;
  if (weight_grad && layout != GEMM_TN) return SLAPO_ERR_UNSUPPORTED;
  describe_gemm(dtype, layout, epilogue, (int)M, (int)N, (int)K, !(flags & SLAPO_GEMM_SHARED), weight_grad != 0, with_ws != 0, buf, len);
  return SLAPO_OK;
}

static int check_weight_grad_shape(int dtype, int64_t M, int64_t N, int64_t K) {
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (M <= 0 || N <= 0 || K <= 0) return SLAPO_ERR_SHAPE;
  if (M * N >= ((int64_t)1 << 31) || M * K >= ((int64_t)1 << 31) || N * K >= ((int64_t)1 << 31)) return SLAPO_ERR_UNSUPPORTED;
  if (M % 8 || N % 8) return SLAPO_ERR_ALIGN;
  return SLAPO_OK;
}

int slapo_weight_grad_workspace(int dtype, int64_t M, int64_t N, int64_t K, size_t* ws_bytes) {
  if (!ws_bytes) return SLAPO_ERR_NULL;
  const int rc = check_weight_grad_shape(dtype, M, N, K);
  if (rc) return rc;
  *ws_bytes = weight_grad_ws_bytes(dtype, (int)M, (int)N, (int)K);
  return SLAPO_OK;
}

int slapo_weight_grad(int dtype, int accumulate, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C,
                      void* ws, void* stream) {
  const int rc = check_weight_grad_shape(dtype, M, N, K);
  if (rc) return rc;
  if (!A || !B || !C) return SLAPO_ERR_NULL;
  if (!ws && weight_grad_ws_least_bytes(dtype, (int)M, (int)N, (int)K)) return SLAPO_ERR_NULL;
  if (misaligned(A) || misaligned(B) || misaligned(C) || misaligned(ws)) return SLAPO_ERR_ALIGN;
  entry_error();
  launch_weight_grad(dtype, accumulate ? 1 : 0, (int)M, (int)N, (int)K, A, B, C, (float*)ws, (hipStream_t)stream);
  return finish();
}

// ---- the weight gradient for callers that cannot allocate ---------------------------------------------
// Same computation as slapo_weight_grad, with the fp32 partial tiles of the K-range path in a fixed array in
// device memory that belongs to the library instead of a caller-provided workspace. The array's name is only a
// host-side handle: its device address is looked up once per device (with that device current) and kept, and
// that pointer is what the kernels are given.
}  // extern "C"

namespace {
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)16 << 20;
static __device__ __align__(256) unsigned char g_static_scratch[STATIC_SCRATCH_BYTES];

// device address of this device's copy of g_static_scratch, or nullptr (with *status set) if it cannot be had
float* static_scratch(int* status) {
  static void* table[16] = {};
  static std::mutex mu;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) { *status = SLAPO_ERR_HIP; return nullptr; }
  if (dev < 0 || dev >= 16) { *status = SLAPO_ERR_UNSUPPORTED; return nullptr; }
  std::lock_guard<std::mutex> lock(mu);
  if (!table[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      *status = SLAPO_ERR_HIP;
      return nullptr;
    }
    table[dev] = ptr;
  }
  return (float*)table[dev];
}
}  // namespace

extern "C" {

int slapo_weight_grad_static(int dtype, int accumulate, int64_t M, int64_t N, int64_t K, const void* A, const void* B,
                             void* C, void* stream) {
  const int rc = check_weight_grad_shape(dtype, M, N, K);
  if (rc) return rc;
  if (!A || !B || !C) return SLAPO_ERR_NULL;
  if (misaligned(A) || misaligned(B) || misaligned(C)) return SLAPO_ERR_ALIGN;
  if (weight_grad_ws_least_bytes(dtype, (int)M, (int)N, (int)K) > STATIC_SCRATCH_BYTES) return SLAPO_ERR_WORKSPACE;
  const size_t wants = weight_grad_ws_bytes(dtype, (int)M, (int)N, (int)K);
  float* ws = nullptr;
  if (wants && wants <= STATIC_SCRATCH_BYTES) {   // shapes that run as one plain GEMM touch no scratch at all
    int st = SLAPO_OK;
    ws = static_scratch(&st);
    if (!ws) return st;
  }
  entry_error();
  launch_weight_grad(dtype, accumulate ? 1 : 0, (int)M, (int)N, (int)K, A, B, C, ws, (hipStream_t)stream);
  return finish();
}

int slapo_attn_fwd(const slapo_layer_desc* d, const void* qkv, const int32_t* seqlens, void* out, float* lse,
                   void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (!qkv || !out || !lse) return SLAPO_ERR_NULL;
  if (misaligned(qkv) || misaligned(out)) return SLAPO_ERR_ALIGN;
  const AttnShape as = make_attn_shape(d);
  entry_error();
  launch_attn_fwd(d->dtype, as, qkv, seqlens, out, lse, (hipStream_t)stream);
  return finish();
}

int slapo_attn_bwd(const slapo_layer_desc* d, const void* qkv, const int32_t* seqlens, const void* out,
                   const void* dout, const float* lse, float* delta, void* dqkv, void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (!qkv || !out || !dout || !lse || !delta || !dqkv) return SLAPO_ERR_NULL;
  if (misaligned(qkv) || misaligned(out) || misaligned(dout) || misaligned(dqkv)) return SLAPO_ERR_ALIGN;
  const AttnShape as = make_attn_shape(d);
  entry_error();
  launch_attn_bwd(d->dtype, as, qkv, seqlens, out, dout, lse, delta, dqkv, (hipStream_t)stream);
  return finish();
}

int slapo_bdrln_fwd(const slapo_layer_desc* d, int site, int64_t T, const void* r, const void* bias, const void* res,
                    const void* gamma, const void* beta, void* z_out, void* out, float* mu, float* rstd,
                    void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (T <= 0 || site < 0 || site > 1) return SLAPO_ERR_SHAPE;
  const bool llama = is_llama(d);   // RMSNorm: no offset, no mean; no biases
  if (!res) return SLAPO_ERR_NULL;
  if (r && ((!bias && !llama) || !z_out)) return SLAPO_ERR_NULL;
  if (gamma && (!out || !rstd || (!llama && (!beta || !mu)))) return SLAPO_ERR_NULL;
  if (!r && !gamma) return SLAPO_ERR_NULL;
  if (misaligned(r) || misaligned(bias) || misaligned(res) || misaligned(gamma) || misaligned(beta) ||
      misaligned(z_out) || misaligned(out)) return SLAPO_ERR_ALIGN;
  entry_error();
  launch_bdrln_fwd(d->dtype, T, d->hidden, r, bias, res, gamma, beta, z_out, out, mu, rstd,
                   make_dropout(d, site), d->ln_eps, llama ? 1 : 0, (hipStream_t)stream);
  return finish();
}

int slapo_bdrln_bwd_blocks(int64_t T) { return bdrln_bwd_blocks(T); }

int slapo_bdrln_bwd(const slapo_layer_desc* d, int site, int64_t T, const void* dout, const void* z, const float* mu,
                    const float* rstd, const void* gamma, const void* dres_in, void* dz_out, void* dr_out,
                    float* partials, void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (T <= 0 || site < 0 || site > 1) return SLAPO_ERR_SHAPE;
  if (!dout || !partials) return SLAPO_ERR_NULL;
  if (gamma && (!z || !rstd || (!mu && !is_llama(d)))) return SLAPO_ERR_NULL;
  if (!dz_out && !dr_out) return SLAPO_ERR_NULL;
  if (misaligned(dout) || misaligned(z) || misaligned(gamma) || misaligned(dres_in) || misaligned(dz_out) ||
      misaligned(dr_out) || misaligned(partials)) return SLAPO_ERR_ALIGN;
  entry_error();
  launch_bdrln_bwd(d->dtype, T, d->hidden, dout, z, mu, rstd, gamma, dres_in, dz_out, dr_out, partials,
                   make_dropout(d, site), is_llama(d) ? 1 : 0, (hipStream_t)stream);
  return finish();
}

int slapo_rope(const slapo_layer_desc* d, void* qkv, float* table, int inverse, void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (!is_llama(d)) return SLAPO_ERR_UNSUPPORTED;
  if (!qkv || !table) return SLAPO_ERR_NULL;
  if (misaligned(qkv) || misaligned(table)) return SLAPO_ERR_ALIGN;
  const int hd = attn_width(d) / d->heads;
  entry_error();
  launch_rope_table(d->seq, hd, d->rope_base, table, (hipStream_t)stream);
  launch_rope(d->dtype, (int64_t)d->batch * d->seq, d->seq, attn_width(d), hd, table, qkv, inverse ? 1 : 0, (hipStream_t)stream);
  return finish();
}

int slapo_colsum_blocks(int64_t T) { return colsum_blocks(T); }

int slapo_colsum_partials(int dtype, int64_t T, int64_t N, const void* a, float* partials, void* stream) {
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (T <= 0 || N <= 0) return SLAPO_ERR_SHAPE;
  if (!a || !partials) return SLAPO_ERR_NULL;
  if (N % 8 || misaligned(a) || misaligned(partials)) return SLAPO_ERR_ALIGN;
  entry_error();
  launch_colsum_partials(dtype, T, N, a, partials, (hipStream_t)stream);
  return finish();
}

int slapo_colreduce_partials(int dtype, int64_t nblk, int64_t stride, int64_t N, const float* partials, void* out,
                             int accumulate, void* stream) {
  if (dtype != SLAPO_BF16 && dtype != SLAPO_FP32 && dtype != SLAPO_FP16) return SLAPO_ERR_UNSUPPORTED;
  if (nblk <= 0 || N <= 0 || stride < N) return SLAPO_ERR_SHAPE;
  if (!partials || !out) return SLAPO_ERR_NULL;
  entry_error();
  launch_colreduce_partials(dtype, nblk, stride, N, partials, out, accumulate, (hipStream_t)stream);
  return finish();
}

int slapo_dropout_mask(const slapo_layer_desc* d, int site, int64_t T, uint8_t* mask, void* stream) {
  const int rc = check_desc(d);
  if (rc) return rc;
  if (T <= 0 || site < 0 || site > 1) return SLAPO_ERR_SHAPE;
  if (!mask) return SLAPO_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(mask) & 7u) != 0) return SLAPO_ERR_ALIGN;
  entry_error();
  launch_dropout_mask(T * d->hidden, mask, make_dropout(d, site), (hipStream_t)stream);
  return finish();
}

}  // extern "C"
