// Moving pages from the host store's natural layout (K[P][D] then V[P][D]) into the slot layouts of kvd_tile_layout.h.
#pragma once
#include "kvd_device.h"
#include "kvd_internal.h"
#include "kvd_tile_layout.h"

namespace kvd {

// 16 bytes at `off` of the `bytes` bytes from `base` on (the same for the whole wave); beyond them a load gives zero and a store
// does nothing.  HANDOFF: the bytes are read by another workgroup of the same launch, so they are written through (a
// device-scope store).
__device__ __forceinline__ uint4 buffer_load16(const char* base, u32 bytes, u32 off) {
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)bytes, 0x00020000), (int)off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool HANDOFF>
__device__ __forceinline__ void buffer_store16(char* base, u32 bytes, u32 off, const uint4& v) {
  const u32x4_t x = {v.x, v.y, v.z, v.w};
  __builtin_amdgcn_raw_buffer_store_b128(x, __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000), (int)off, 0, HANDOFF ? 16 : 0);
}

// One 16-token tile by a group of 256 threads in two phases with a barrier (the caller's) between them.
// Phase A (gt = thread index in the group): fetch one 16-byte unit of K and of V (token gt / 16 of
// the tile, dims 8 (gt % 16) ..), store the K unit at its permuted place, park the V unit in LDS
// (`vt`: 16 x 128 elements, natural order).
__device__ __forceinline__ void tile_copy_phase_a(const char* __restrict__ src_page, int P, int tile,
                                                  char* __restrict__ dst_tile, uint16_t* vt, int gt) {
  const int row = gt >> 4, ch = gt & 15;
  const char* ksrc = src_page + ((size_t)(tile * kTileTokens + row) * kRowBytes) + ch * 16;
  const uint4 kq = *reinterpret_cast<const uint4*>(ksrc);
  const uint4 vq = *reinterpret_cast<const uint4*>(ksrc + (size_t)P * kRowBytes);
  // K: chunk c = ch / 4, lane = row + 16 * (ch % 4)
  *reinterpret_cast<uint4*>(dst_tile + ((ch >> 2) * 64 + (ch & 3) * 16 + row) * 16) = kq;
  *reinterpret_cast<uint4*>(vt + row * kHeadDim + ch * 8) = vq;
}

// Phase B: thread gt assembles destination unit gt of the V part (chunk c, lane i + 16 g): four
// tokens 4g..4g+3 of dim 32c + i, then of dim 32c + 16 + i.
__device__ __forceinline__ void tile_copy_phase_b(char* __restrict__ dst_tile, const uint16_t* vt, int gt) {
  const int c = gt >> 6, g = (gt >> 4) & 3, i = gt & 15;
  uint16_t e[8];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int k = 0; k < 4; ++k) e[hh * 4 + k] = vt[(4 * g + k) * kHeadDim + 32 * c + 16 * hh + i];
  uint4 outv;
  outv.x = (u32)e[0] | ((u32)e[1] << 16);
  outv.y = (u32)e[2] | ((u32)e[3] << 16);
  outv.z = (u32)e[4] | ((u32)e[5] << 16);
  outv.w = (u32)e[6] | ((u32)e[7] << 16);
  *reinterpret_cast<uint4*>(dst_tile + kTilePartBytes + gt * 16) = outv;
}

// Four tokens of a page from the host store's natural layout into a slot of 16-token tiles or of a packed page, by one wave
// (unit (c, g, t) of a tile's K and unit (c, tg, i) of its V are at the same places as those of a packed page of 16 tokens).
// Every lane moves one 16-byte unit of K and one of V, which the wave turns around through `vt` (4 x 128 elements of LDS of its
// own).  A wave waits for nobody, and loads are apart from stores so that several groups can be on their way.
struct PageGroup { uint4 k, v; };
__device__ __forceinline__ void page_group_load(const char* src_page, u32 bytes, int P, int group, PageGroup& x) {
  const u32 lane = threadIdx.x & (kWave - 1), at = (4u * (u32)group + (lane >> 4)) * kRowBytes + (lane & 15) * 16;
  x.k = buffer_load16(src_page, bytes, at);
  x.v = buffer_load16(src_page, bytes, at + (u32)P * kRowBytes);
}
// T: tokens of a tile (16, or the 4 or 8 of a packed page)
template <bool HANDOFF>
__device__ __forceinline__ void page_group_store(char* slot, u32 bytes, int T, int group, uint16_t* vt, const PageGroup& x) {
  const u32 lane = threadIdx.x & (kWave - 1), t0 = 4u * (u32)group & (u32)(T - 1), tile = (4u * (u32)group - t0) * 2 * kRowBytes;
  buffer_store16<HANDOFF>(slot, bytes, tile + ((lane & 15) * (u32)T + t0 + (lane >> 4)) * 16, x.k);
  wave_lds_fence();                                    // (the group before this one has been read)
  *reinterpret_cast<uint4*>(vt + (lane >> 4) * kHeadDim + (lane & 15) * 8) = x.v;
  wave_lds_fence();
  // V unit (c, t0 / 4, i): the four tokens of dim 32c + i, then of dim 32c + 16 + i
  const u32 c = lane >> 4, i = lane & 15;
  uint16_t e[8];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int k = 0; k < 4; ++k) e[hh * 4 + k] = vt[k * kHeadDim + 32 * c + 16 * hh + i];
  uint4 outv;
  outv.x = (u32)e[0] | ((u32)e[1] << 16);
  outv.y = (u32)e[2] | ((u32)e[3] << 16);
  outv.z = (u32)e[4] | ((u32)e[5] << 16);
  outv.w = (u32)e[6] | ((u32)e[7] << 16);
  buffer_store16<HANDOFF>(slot, bytes, tile + (u32)T * kRowBytes + ((c * ((u32)T >> 2) + (t0 >> 2)) * 16 + i) * 16, outv);
}
template <class T>
__device__ __forceinline__ T* wave_uniform(T* p) {
  const u64 v = reinterpret_cast<u64>(p);
  return reinterpret_cast<T*>(((u64)(u32)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) | (u32)__builtin_amdgcn_readfirstlane((int)(u32)v));
}
__device__ __forceinline__ void packed_copy_group(const char* src_page, int P, int group, char* slot, uint16_t* vt) {
  src_page = wave_uniform(src_page);
  slot = wave_uniform(slot);
  PageGroup x;
  page_group_load(src_page, (u32)P * 2 * kRowBytes, P, group, x);
  page_group_store<false>(slot, (u32)P * 2 * kRowBytes, P, group, vt, x);
}

}  // namespace kvd
