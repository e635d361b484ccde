// Stage 3 of the decode step: GQA decode attention over the selected pages only (System
// Overview: attention runs over the union of resident and newly fetched entries).  See
// kvd_attn_body.h for the split-K frame.
//
// One kernel, three layouts that differ in how a lane finds its operands:
//  * pages of a multiple of 16 tokens are kept in the slot pool in an operand-ready tile layout (see
//    kvd_tile_layout.h), so that every wave load is 1 KiB contiguous and lands directly in MFMA operand
//    registers: S^T = K Q^T with 16x16x32 MFMAs, O^T += V^T P^T with 16x16x16 MFMAs whose B operand is
//    the softmaxed C tile of the first;
//  * pages of 4 or 8 tokens take the same kernel over the packed layout: 16 / P pages per tile;
//  * pages of any other size keep natural [token][dim] slots, of which a tile takes 16 consecutive tokens.
#include <math.h>

#include <mutex>

#include "kvd_attn_body.h"
#include "kvd_device.h"
#include "kvd_internal.h"
#include "kvd_tile_layout.h"

// Scratch of kvd_sparse_decode_attn_noalloc: the arrival tickets of the units, then the split
// partials (max and sum per query head, then the accumulators).  Every GPU the library runs on
// holds its own copy of this array from the moment the code is loaded until the process ends.
constexpr size_t kNoAllocScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace kvd {

constexpr int kMergeThreads = 256;

template <int G>
__global__ __launch_bounds__(kMergeThreads) void combine_kernel(AttnArgs a) {
  __shared__ float lds[kMergeFloats];
  merge_splits<G, kMergeThreads, false>(a, blockIdx.x + a.u0, lds);
}

// 512 threads and up to 256 registers per lane: one workgroup per CU, three tile buffers (24 KiB)
// in flight per wave; the grid is sized to about one workgroup per CU (see kvd_create).
constexpr int kAttnMfmaThreads = 512;
template <bool BF16, int G, int LAYOUT>
__global__ __launch_bounds__(kAttnMfmaThreads, 2) void attend_mfma_kernel(AttnArgs a) {
  __shared__ AttnSmem<G, kAttnMfmaThreads / kWave, LAYOUT == kLayoutNatural ? KVD_MAX_TOPK : kAttnIdxCap> sm;
  attend_mfma_body<BF16, G, kAttnMfmaThreads, false, LAYOUT>(a, sm, blockIdx.y + a.u0, blockIdx.x);
}

template <bool BF16, int G>
static void launch_attend(int layout, const AttnArgs& a, dim3 grid, hipStream_t s, hipEvent_t between) {
  if (layout == kLayoutPacked)
    hipLaunchKernelGGL((attend_mfma_kernel<BF16, G, kLayoutPacked>), grid, dim3(kAttnMfmaThreads), 0, s, a);
  else if (layout == kLayoutTiles)
    hipLaunchKernelGGL((attend_mfma_kernel<BF16, G, kLayoutTiles>), grid, dim3(kAttnMfmaThreads), 0, s, a);
  else
    hipLaunchKernelGGL((attend_mfma_kernel<BF16, G, kLayoutNatural>), grid, dim3(kAttnMfmaThreads), 0, s, a);
  if (between != nullptr) (void)hipEventRecord(between, s);   // no kernel follows when the merge is fused
  if (a.S > 1 && !a.fuse_merge)
    hipLaunchKernelGGL((combine_kernel<G>), dim3(grid.y), dim3(kMergeThreads), 0, s, a);
}

template <bool BF16>
static bool dispatch_group(int G, int layout, const AttnArgs& a, dim3 grid, hipStream_t s, hipEvent_t between) {
  switch (G) {
    case 1: launch_attend<BF16, 1>(layout, a, grid, s, between); return true;
    case 2: launch_attend<BF16, 2>(layout, a, grid, s, between); return true;
    case 3: launch_attend<BF16, 3>(layout, a, grid, s, between); return true;
    case 4: launch_attend<BF16, 4>(layout, a, grid, s, between); return true;
    case 5: launch_attend<BF16, 5>(layout, a, grid, s, between); return true;
    case 6: launch_attend<BF16, 6>(layout, a, grid, s, between); return true;
    case 7: launch_attend<BF16, 7>(layout, a, grid, s, between); return true;
    case 8: launch_attend<BF16, 8>(layout, a, grid, s, between); return true;
    default: return false;
  }
}

}  // namespace kvd

// Split-K factor where the caller leaves it open: one 512-thread workgroup runs per CU, so at most one workgroup per
// CU in the grid; the few of a second round take as long again.  In the one-launch step (beside_selection) the units' selection
// workgroups hold CUs of their own until their entries are out: these are left to them where that costs an attention
// workgroup no more than a quarter of its length, unless the splits are 8 or 16, which launches of several layers deal out
// evenly.  us per step with the nearest number to a workgroup per CU, with at most one, and without the selections' CUs: one
// launch, 24 units of 2048 pages S = 11, 10 and 9 23.3, 20.2 and 19.7, 40 of 363 6, 6 and 5 18.3, 18.3 and 17.2, 56 of 2969
// 5, 4 and 3 39.1, 33.5 and 34.8, 96 of 1250 3, 2 and 1 38.5, 33.1 and 38.2; 32 of 1001 8, 8 and 7 20.2, 20.2 and 19.8, but per layer
// of 8 layers x 16 units of 1024 pages 7.6 with 16 and 8.5 with 15, of 3 x 32 of 2048 14.6 with 8 and 16.0 with 7 (contexts of
// one layer keep 8 and 16 too, and lose 2 % by it); over natural slots, where a workgroup takes one split also in launches of several layers, so that 8 and 16 are
// nothing special (dealt_out false), 24 units x 53 pages of 24 tokens 25.5 with 11 and 23.6
// with 10, 32 x 85 of 24 24.3 with 8 and 23.7 with 7, 96 x 102 pages of 20 49.4 with 3 and 41.0 with 2.  But
//  - a split keeps at least `least` tiles of 16 tokens for its eight waves: 16 in the stand-alone kernel over tiles (where
//    fewer made no difference), 8 in the one-launch step with pages of up to 16 tokens and at least 32 tiles (8 units
//    of 64 pages: 16.7 us with two tiles per wave, 15.9 with one; 2 splits instead of 1 gain nothing, and with larger
//    pages a split's share comes in steps of several tiles: 20 units of 21 pages of 64 tokens 21.1 and 21.8), 4 over
//    natural slots, where a tile costs a wave more (2 units of 40 pages of 12 tokens: 23.8 us with 16, 18.8 with 4);
//  - beyond 16 splits a split keeps 32 tiles: the last split to arrive fetches the partials of all the others, and that costs
//    more than shorter splits save.  With room for 32 splits per unit, that is up to 8 units, up to 32 splits keep 18 tiles
//    each.  us per step of one launch, pages of 16 tokens, with 16 splits, this and 32: 4 units of 320 pages 18.5, 18.3 and
//    18.5, of 448 20.2, 19.2 and 19.6, of 576 22.3, 20.5 and 20.5; 8 units of 320 19.6, 19.9 and 20.8, of 448 21.1, 21.2 and
//    21.8, of 512 22.0, 21.7 and 22.1, of 640 23.7, 23.6 and 23.5; as a chain, 2 units of 1024 27.5, 24.1 and 24.5.  With 16
//    splits and with 18 tiles each where there is less room: 9 units of 320 19.8 and 20.2, of 512 22.3 and 22.1, 10 of 512 22.9
//    and 23.2, 12 of 448 22.6 and 23.3, 14 of 576 25.7 and 26.5;
//  - no split is left without pages.
int kvd_attn_splits(int least, int U, int k, int P, int cus, bool beside_selection, bool dealt_out) {
  const int tiles = (k * P + 15) / 16;                 // of a unit's selection
  int S = cus / U;
  if (beside_selection && S >= 5 && !(dealt_out && S % 8 == 0)) S = (cus - U) / U;
  if (S > tiles / least) S = tiles / least;
  int longest = tiles / 32;
  if (cus / U >= 32 && longest < 32) longest = tiles / 18 < 32 ? tiles / 18 : 32;
  if (S > 16 && S > longest) S = longest > 16 ? longest : 16;
  if (S > KVD_MAX_SPLITS) S = KVD_MAX_SPLITS;
  if (S > k) S = k;
  if (S < 1) S = 1;
  const int per_split = (k + S - 1) / S;
  return (k + per_split - 1) / per_split;
}

kvd::AttnArgs kvd_attn_args(kvd_ctx* c, int layer, const void* q, const int32_t* sel_pages, const int32_t* sel_slots,
                            float* out, float* lse, int u0) {
  using namespace kvd;
  AttnArgs a;
  a.u0 = u0;
  a.q = reinterpret_cast<const uint16_t*>(q);
  a.pool = c->pool + (size_t)layer * c->U * c->Cmax * c->page_bytes;
  a.sel_pages = sel_pages;
  a.sel_slots = sel_slots;
  a.sel_entry = nullptr;                               // (only the one-launch step hands the selection over in entries)
  a.error = c->error_dev;
  a.wait_limit = c->wait_limit_ticks;
  a.seq_len = c->d_seq_len;
  a.part_acc = c->d_part_acc;
  a.part_ml = c->d_part_ml;
  a.ticket = c->d_attn_ticket;
  a.out = out;
  a.lse = lse;
  a.k = c->k; a.P = c->P; a.Cmax = c->Cmax; a.Hq = c->Hq; a.Hkv = c->Hkv; a.G = c->G; a.S = c->S;
  a.per_split = (c->k + c->S - 1) / c->S;
  a.take = 1;
  a.fuse_merge = c->fuse_merge;
  a.page_bytes = (unsigned)c->page_bytes;
  a.scale_log2 = c->scale * kLog2e;
  return a;
}

hipError_t kvd_launch_attend(kvd_ctx* c, int layer, const void* q, const int32_t* sel_pages,
                             const int32_t* sel_slots, float* out, float* lse, int u0, int u1, hipStream_t s,
                             hipEvent_t between) {
  using namespace kvd;
  if (u1 <= u0) return hipSuccess;
  const AttnArgs a = kvd_attn_args(c, layer, q, sel_pages, sel_slots, out, lse, u0);
  dim3 grid(c->S, u1 - u0);
  const bool ok = c->bf16 ? dispatch_group<true>(c->G, c->tiled, a, grid, s, between)
                          : dispatch_group<false>(c->G, c->tiled, a, grid, s, between);
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------
// The attention stage for callers that cannot allocate
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mutex;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU (the array's name is only a host-side handle)
int g_scratch_cus[kMaxDevices];

// Device address of this GPU's copy of `scratch` and its number of compute units, looked up once
// per device with that device current.
hipError_t noalloc_device_state(void** ptr, int* cus) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    int n = 0;
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    g_scratch_cus[dev] = n > 0 ? n : 256;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  *cus = g_scratch_cus[dev];
  return hipSuccess;
}

size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }

}  // namespace

extern "C" int kvd_sparse_decode_attn_noalloc(const void* q, const void* slot_pool, const int32_t* sel_pages,
                                              const int32_t* sel_slots, const int32_t* seq_len, float* out, float* lse,
                                              int32_t batch, int32_t n_q_heads, int32_t n_kv_heads, int32_t page_size,
                                              int32_t topk_pages, int32_t capacity_max, int32_t kv_dtype,
                                              float softmax_scale, int32_t attn_splits, void* stream) {
  using namespace kvd;
  if (!q || !slot_pool || !sel_pages || !sel_slots || !seq_len || !out) return KVD_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(q) & 15u) || (reinterpret_cast<uintptr_t>(slot_pool) & 15u)) return KVD_ERR_ARG;
  if (kv_dtype != KVD_F16 && kv_dtype != KVD_BF16) return KVD_ERR_DTYPE;
  if (batch < 1 || n_q_heads < 1 || n_kv_heads < 1 || n_q_heads % n_kv_heads != 0) return KVD_ERR_SHAPE;
  const int G = n_q_heads / n_kv_heads;
  if (G > KVD_MAX_GROUP) return KVD_ERR_SHAPE;
  if (page_size < 1 || page_size > KVD_MAX_PAGE) return KVD_ERR_SHAPE;
  if (topk_pages < 1 || topk_pages > KVD_MAX_TOPK) return KVD_ERR_SHAPE;
  if (capacity_max < 1 || capacity_max > KVD_MAX_CAPACITY) return KVD_ERR_SHAPE;
  if ((long long)batch * n_kv_heads > 65535) return KVD_ERR_SHAPE;
  if (attn_splits < 0 || attn_splits > KVD_MAX_SPLITS) return KVD_ERR_SHAPE;
  if (!(softmax_scale >= 0.f) || isinf(softmax_scale)) return KVD_ERR_ARG;
  void* base = nullptr;
  int cus = 0;
  // (the number of compute units is only needed to choose the splits: sizes that cannot fit
  // whatever the device are refused before any device is touched)
  if (attn_splits == 0 && noalloc_device_state(&base, &cus) != hipSuccess) {
    (void)hipGetLastError();
    return KVD_ERR_HIP;
  }
  const int U = batch * n_kv_heads;
  const int layout = slot_layout_of(page_size);
  int S = attn_splits == 0 ? kvd_attn_splits(layout == kLayoutNatural ? kNaturalLeast : 16, U, topk_pages, page_size, cus) : attn_splits;
  if (S > topk_pages) S = topk_pages;
  // the scratch array, cut into tickets [U], (max, sum) [U][S][G][2] and accumulators [U][S][G][D]
  const size_t rows = (size_t)U * S * G;
  const size_t off_ml = round256((size_t)U * sizeof(int32_t));
  const size_t off_acc = off_ml + round256(rows * 2 * sizeof(float));
  const size_t need = off_acc + rows * kHeadDim * sizeof(float);
  if (need > kNoAllocScratchBytes) return KVD_ERR_CAPACITY;
  if (base == nullptr && noalloc_device_state(&base, &cus) != hipSuccess) {
    (void)hipGetLastError();
    return KVD_ERR_HIP;
  }
  unsigned char* sp = static_cast<unsigned char*>(base);
  hipStream_t s = static_cast<hipStream_t>(stream);

  AttnArgs a;
  a.u0 = 0;
  a.q = reinterpret_cast<const uint16_t*>(q);
  a.pool = static_cast<const char*>(slot_pool);
  a.sel_pages = sel_pages;
  a.sel_slots = sel_slots;
  a.sel_entry = nullptr;
  a.error = nullptr;
  a.wait_limit = 0;
  a.seq_len = seq_len;
  a.ticket = reinterpret_cast<int32_t*>(sp);
  a.part_ml = reinterpret_cast<float*>(sp + off_ml);
  a.part_acc = reinterpret_cast<float*>(sp + off_acc);
  a.out = out;
  a.lse = lse;
  a.k = topk_pages; a.P = page_size; a.Cmax = capacity_max; a.Hq = n_q_heads; a.Hkv = n_kv_heads; a.G = G; a.S = S;
  a.per_split = (topk_pages + S - 1) / S;
  a.take = 1;
  a.fuse_merge = 1;
  a.page_bytes = (unsigned)((size_t)2 * page_size * kHeadDim * 2);
  a.scale_log2 = (softmax_scale > 0.f ? softmax_scale : 1.0f / sqrtf((float)kHeadDim)) * kLog2e;
  // the tickets must start at zero whatever an earlier call left there (a fill kernel, so that
  // the call can be captured into a HIP graph)
  if (S > 1 && kvd_launch_fill_i32(a.ticket, 0, (size_t)U, s) != hipSuccess) {
    (void)hipGetLastError();
    return KVD_ERR_HIP;
  }
  const dim3 grid(S, U);
  const bool ok = kv_dtype == KVD_BF16 ? dispatch_group<true>(G, layout, a, grid, s, nullptr)
                                       : dispatch_group<false>(G, layout, a, grid, s, nullptr);
  if (!ok) return KVD_ERR_SHAPE;
  if (hipGetLastError() != hipSuccess) return KVD_ERR_HIP;
  return KVD_OK;
}
