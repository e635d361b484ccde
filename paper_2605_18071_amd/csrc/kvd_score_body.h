// Scoring of page summaries against the pooled query, one wave at a time (Background, "KV Cache
// Offloading": the query is multiplied with the index representatives; System Overview: the
// representative is the page's mean key).  Shared by the stand-alone scoring kernel and by the
// single-launch layer-step kernel.
#pragma once
#include "kvd_device.h"
#include "kvd_internal.h"

namespace kvd {

// One wave scores pages [wave_base, wave_base + 64 * passes) of one unit in passes of 64.  A wave
// load covers 4 summary rows (4 x 256 B): lane (r, c) = (lane / 16, lane % 16) holds dims
// 8c..8c+7 of row r.  The 16 partial dot products of a row are summed with DPP row rotations;
// after 16 loads lane (r, c) keeps the score of page base + 4c + r and the wave stores 64
// consecutive scores.  The query's rows and the first summaries are on their way together: with a load and a wait per row
// the summaries were waited for with the first row and each further row took a trip to the L2, with nothing streaming
// (us per step so and with all loads ahead: 128 units x 2048 pages, G = 7, 46.6 and 43.9; 32 units x 2084 pages, G = 7, as a
// chain 30.9 and 29.2; 4 layers of 32 x 1001 pages, G = 4, 114.1 and 111.6; 128 x 8192 pages 96.3 and 94.7).  16 loads
// ahead of the first pass instead of 8 gained nothing (43.8 to 44.2, 29.4, 111.3, 95.5).
//   summ_u   [NP][D]  summaries of the unit
//   q_group  [G][D]   the unit's G query heads
//   scores_u [NP]
// HANDOFF: the scores are consumed by another workgroup of the same launch, so they are stored
// with device-scope write-through stores.
template <bool BF16, bool HANDOFF>
__device__ __forceinline__ void score_wave(const uint16_t* __restrict__ summ_u, const uint16_t* __restrict__ q_group,
                                           float* __restrict__ scores_u, int NP, int G, float scale, int wave_base,
                                           int passes) {
  const int lane = threadIdx.x & (kWave - 1);
  const int r = lane >> 4, c = lane & 15;
  if (wave_base >= NP) return;
  const uint16_t* srow = summ_u + c * 8;

  // All of the query's rows are asked for at once and before the first summaries: loads return in order, so the wait for
  // the rows leaves the summaries in flight.  Rows beyond the group are out of the buffer's bounds and read as zero,
  // which the sums do not notice.
  const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(q_group), 0, G * kRowBytes, 0x00020000);
  u32x4_t qraw[KVD_MAX_GROUP];
#pragma unroll
  for (int g = 0; g < KVD_MAX_GROUP; ++g) qraw[g] = __builtin_amdgcn_raw_buffer_load_b128(q_rsrc, c * 16 + g * kRowBytes, 0, 0);

  uint4 raw[8];
  auto issue = [&](int base, int half) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      int page = base + 4 * (half * 8 + i) + r;
      page = page < NP ? page : NP - 1;
      raw[i] = load_stream16(srow + (size_t)page * kHeadDim);
    }
  };
  issue(wave_base, 0);
  __builtin_amdgcn_sched_barrier(0);                   // (the conversions of the query stay behind the loads)

  float qbar[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) qbar[e] = 0.f;
#pragma unroll
  for (int g = 0; g < KVD_MAX_GROUP; ++g) {
    float f[8];
    cvt8<BF16>(make_uint4(qraw[g].x, qraw[g].y, qraw[g].z, qraw[g].w), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) qbar[e] += f[e];
  }
  const float fg = (float)G;
#pragma unroll
  for (int e = 0; e < 8; ++e) qbar[e] = qbar[e] / fg;

  for (int pass = 0; pass < passes; ++pass) {
    const int base = wave_base + pass * 64;
    if (base >= NP) break;
    float mine = 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint4 cur[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) cur[i] = raw[i];
      // next batch in flight while this one is reduced
      if (half == 0) issue(base, 1);
      else if (pass + 1 < passes && base + 64 < NP) issue(base + 64, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float f[8];
        cvt8<BF16>(cur[i], f);
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaf(qbar[e], f[e], acc);
        acc = row16_allreduce_sum(acc);
        if (c == half * 8 + i) mine = acc;
      }
    }
    const int page = base + 4 * c + r;
    if (page < NP) {
      if (HANDOFF) store_agent(scores_u + page, mine * scale);
      else scores_u[page] = mine * scale;
    }
  }
}

}  // namespace kvd
