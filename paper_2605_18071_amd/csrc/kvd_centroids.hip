// The hierarchical index (System Overview: the page means form higher-level centroids for
// similarity grouping; Pipeline Optimization: the number of centroids is a tunable of the index).
//
// Build (set-up helper, not on the decode path): Lloyd's k-means over the page summaries of every
// unit, in fp64 so that its decisions can be checked against a plain CPU implementation: initial
// centroids = the pages at evenly spaced positions, nearest centroid by squared Euclidean distance
// (ties to the lower centroid), new centroid = mean of the cluster's summaries summed in ascending
// page order (an empty cluster keeps its centroid), a fixed number of rounds; the stored centroid
// is rounded once to the KV dtype and each cluster's pages are listed in ascending order.
//
// Decode: the scoring kernel runs over the centroids instead of the page summaries (half the
// bytes when there are half as many centroids as pages); cluster_select_kernel then takes whole
// clusters in (score descending, cluster ascending) order until the page budget is used up, the
// first cluster that does not fit giving its lowest pages; sink / recent pages are in first and
// are not counted as members of their clusters.
#include "kvd_cluster_body.h"
#include "kvd_device.h"
#include "kvd_internal.h"

namespace kvd {

// ---------------------------------------------------------------------------------------------
// build
// ---------------------------------------------------------------------------------------------
template <bool BF16>
__device__ __forceinline__ double widen_kv(uint16_t raw) {
  return (double)(BF16 ? as_f32((u32)raw << 16) : (float)__builtin_bit_cast(_Float16, raw));
}

// What the assignment screens with, per 16 centroids: [2 parts][4 chunks of 32 dims][64 lanes][8 elements], lane i + 16 g of
// chunk c holding dims 32c + 8g .. +7 of centroid i, which is the A operand of a 16x16x32 MFMA as a wave loads it (1 KiB
// contiguous per chunk).  Part 0 is the centroid, less the unit's shift, rounded to the KV dtype, part 1 the rest
// rounded once more.
constexpr int kScreenTile = 2 * 4 * kWave * 8;            // elements
struct ScreenArgs {
  uint16_t* frag;       // [U][tiles][kScreenTile]
  float* neg_half;      // [U][16 * tiles] minus half the squared norm (of the same); minus infinity beyond the last centroid
  uint16_t* shift;      // [U][D] see kmeans_shift_kernel
  int tiles;            // ceil(Nc / 16)
  int32_t* hard;        // [U][NP] pages of the round that kmeans_exhaustive_kernel decides, in any order
  int32_t* n_hard;      // [U] how many; zero before a round
};

template <bool BF16>
__device__ __forceinline__ u32 narrow_screen(double x) {
  const float f = (float)x;
  return BF16 ? (u32)__builtin_bit_cast(uint16_t, (__bf16)f) : (u32)__builtin_bit_cast(uint16_t, (_Float16)f);
}

// One wave, centroid c of unit u, lane l holding dims 2l and 2l + 1.
template <bool BF16>
__device__ __forceinline__ void store_screen(const ScreenArgs& sa, int u, int c, double x0, double x1) {
  const int lane = threadIdx.x & (kWave - 1);
  const u32 shift = *reinterpret_cast<const u32*>(sa.shift + (size_t)u * kHeadDim + 2 * lane);
  x0 -= widen_kv<BF16>((uint16_t)shift);
  x1 -= widen_kv<BF16>((uint16_t)(shift >> 16));
  // (by way of fp32: a second rounding of 2^-24 does not matter to the screening's bound, and four conversions of 64-bit
  // integer arithmetic were half of what kmeans_update_kernel did)
  const u32 h0 = narrow_screen<BF16>(x0), h1 = narrow_screen<BF16>(x1);
  const u32 l0 = narrow_screen<BF16>(x0 - widen_kv<BF16>((uint16_t)h0)), l1 = narrow_screen<BF16>(x1 - widen_kv<BF16>((uint16_t)h1));
  const int d = 2 * lane, at = ((d >> 5) * kWave + ((d & 31) >> 3) * 16 + (c & 15)) * 8 + (d & 7);
  uint16_t* tile = sa.frag + ((size_t)u * sa.tiles + (c >> 4)) * kScreenTile;
  *reinterpret_cast<u32*>(tile + at) = h0 | (h1 << 16);
  *reinterpret_cast<u32*>(tile + kScreenTile / 2 + at) = l0 | (l1 << 16);
  double n = x0 * x0 + x1 * x1;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) n += __shfl_xor(n, m, kWave);
  if (lane == 0) sa.neg_half[(size_t)u * sa.tiles * 16 + c] = (float)(-0.5 * n);
}

// The shift that the screening takes off all points and centroids of a unit: its bound grows with their norms, and
// keys often have a large component in common, which makes no difference to a distance.  A dim whose values all lie
// between some a > 0 and 3a (or between -3a and -a) is shifted by the middle of the extremes rounded to the KV
// dtype, which every value is within a factor of two of, and every mean of them, so that all differences are exact; other
// dims by zero.  Values below 2^-12 (fp16) and 2^-40 are left alone, so that halves of them are still normal numbers.
// Block (x, u): dims 8x .. 8x+7 of unit u.  (ms of a build of 4 rounds, 8192 pages against 4096 centroids, a common
// component 200 times the spread, without and with the shift: one unit 5.2 and 1.3, eight units 18.5 and 1.6; 20 us of it are
// this kernel's.)
constexpr int kShiftThreads = 256;
template <bool BF16>
__global__ __launch_bounds__(kShiftThreads) void kmeans_shift_kernel(const uint16_t* __restrict__ summ, ScreenArgs sa,
                                                                   const int32_t* __restrict__ seq_len, int NP, int P, int Hkv) {
  constexpr int NW = kShiftThreads / kWave;
  __shared__ float least[NW][8], most[NW][8];
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  int n_valid = (seq_len[u / Hkv] + P - 1) / P;
  n_valid = n_valid < NP ? n_valid : NP;
  const uint16_t* col = summ + (size_t)u * NP * kHeadDim + 8 * blockIdx.x;
  float lo[8], hi[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { lo[e] = INFINITY; hi[e] = -INFINITY; }
  for (int p = tid; p < n_valid; p += kShiftThreads) {
    float f[8];
    cvt8<BF16>(*reinterpret_cast<const uint4*>(col + (size_t)p * kHeadDim), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = fminf(lo[e], f[e]); hi[e] = fmaxf(hi[e], f[e]); }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    lo[e] = wave_allreduce_min(lo[e]);
    hi[e] = wave_allreduce_max(hi[e]);
    if (lane == 0) { least[w][e] = lo[e]; most[w][e] = hi[e]; }
  }
  __syncthreads();
  if (tid < 8) {
    float a = least[0][tid], b = most[0][tid];
#pragma unroll
    for (int i = 1; i < NW; ++i) { a = fminf(a, least[i][tid]); b = fmaxf(b, most[i][tid]); }
    const float small = BF16 ? 0x1p-40f : 0x1p-12f;
    const bool alike = (a >= small && b <= 3.f * a && b < INFINITY) || (b <= -small && a >= 3.f * b && a > -INFINITY);
    sa.shift[(size_t)u * kHeadDim + 8 * blockIdx.x + tid] = alike ? f64_to_kv<BF16>(0.5 * ((double)a + (double)b)) : (uint16_t)0;
  }
}

constexpr int kCentroidWaves = 4;     // centroids per block of the kernels that write them

// cent64 [U][Nc][D] <- summaries of the pages floor((c + 1/2) * n_valid / Nc)
template <bool BF16>
__global__ __launch_bounds__(kCentroidWaves* kWave) void kmeans_init_kernel(const uint16_t* __restrict__ summ,
                                                                           double* __restrict__ cent64, ScreenArgs sa,
                                                                           const int32_t* __restrict__ seq_len, int NP, int Nc,
                                                                           int P, int Hkv) {
  const int c = blockIdx.x * kCentroidWaves + threadIdx.x / kWave, u = blockIdx.y, lane = threadIdx.x & (kWave - 1);
  if (c >= sa.tiles * 16) return;
  if (c == 0 && lane == 0) sa.n_hard[u] = 0;
  if (c >= Nc) {                                            // the last tile's empty places
    if (lane == 0) sa.neg_half[(size_t)u * sa.tiles * 16 + c] = -INFINITY;
    uint16_t* tile = sa.frag + ((size_t)u * sa.tiles + (c >> 4)) * kScreenTile;
    for (int k = lane; k < kScreenTile / 16; k += kWave) tile[((k >> 3) * 16 + (c & 15)) * 8 + (k & 7)] = 0;
    return;
  }
  int n_valid = (seq_len[u / Hkv] + P - 1) / P;
  n_valid = n_valid < NP ? n_valid : NP;
  const int page = (int)(((double)c + 0.5) * (double)n_valid / (double)Nc);
  const u32 raw = *reinterpret_cast<const u32*>(summ + ((size_t)u * NP + page) * kHeadDim + 2 * lane);
  const double x0 = widen_kv<BF16>((uint16_t)raw), x1 = widen_kv<BF16>((uint16_t)(raw >> 16));
  *reinterpret_cast<double2*>(cent64 + ((size_t)u * Nc + c) * kHeadDim + 2 * lane) = make_double2(x0, x1);
  store_screen<BF16>(sa, u, c, x0, x1);
}

// Nearest centroid of every page, exactly as the definition has it: squared distance summed in
// fp64 in dim order, ties to the lower centroid.  Computing all of them in fp64 is bound by the
// fp64 rate (8 units of 8192 pages against 4096 centroids: 4.4 ms a round); so
// the distances are first bounded on the matrix cores, where a round is 275 GFLOP of 16-bit MFMA (two sweeps of 137):
//   v = x . (c_hi + c_lo) - |c|^2 / 2        (the larger, the nearer; x and c less the unit's shift)
// in fp32, each within E of its true value, E = 2^-14 (|x| C + C^2 / 2) + 2^-20 |x| with C the unit's
// largest centroid norm.  That covers the part of c that two 16-bit parts leave out (2^-18 |x| |c| for
// bf16; for fp16 2^-24, or 2^-25 per dim among its subnormals), and 256 fp32 roundings of sums no
// larger than |x| |c| + |c|^2 / 2 (2^-16 of that).  The nearest centroid is among those whose v is
// within 2 E of the largest: one of them, as a rule, and then it is the answer; several are compared
// in fp64, in the definition's order of operations; more than kAssignCap (exact ties, or data whose
// differences the screening cannot see) and the page is compared with every centroid in fp64.  So it is
// where E would not hold for the range of fp32: norms above 2^60 could carry v or E to infinity, and a
// largest centroid norm below 2^-45 leaves v among the subnormals.
//
// Block (x, u): points 256x .. 256x+255 of unit u.  Wave w takes 64 of them (B operands kept in
// registers) and one half of the centroid tiles, which the block stages through LDS, two of each half at a time and double
// buffered: each tile is read once per 256 points and feeds 32 MFMAs per wave.  The first round goes through the tiles
// twice, for the largest v of every point and then for the candidates.  Later rounds start from v of the centroid that the
// point had before, which the largest v is not below, and go through the tiles once: what is within the slack of the
// largest v so far is listed, and the list is filtered when the largest of all is known (a list that is too short sends its
// block through the tiles again).  (us a round of 8 x 8192 pages against 4096 centroids: two sweeps with one tile of a
// half at a time and its norms read when they are needed 295, two as they are now 256, one 159.)
constexpr int kAssignThreads = 512;
constexpr int kAssignBlock = 256;     // points per block
constexpr int kAssignCap = 8;         // candidates per point that are compared one by one

typedef float f32x4_c __attribute__((ext_vector_type(4)));
template <bool BF16>
__device__ __forceinline__ f32x4_c mfma_16x16x32(const uint4& a, const uint4& b, f32x4_c c) {
  if (BF16) {
    typedef __bf16 v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8, a), __builtin_bit_cast(v8, b), c, 0, 0, 0);
  } else {
    typedef _Float16 v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8, a), __builtin_bit_cast(v8, b), c, 0, 0, 0);
  }
}

// a number that the KV dtype holds exactly, as its bits
template <bool BF16>
__device__ __forceinline__ u32 narrow_exact(float f) {
  return BF16 ? __float_as_uint(f) >> 16 : (u32)__builtin_bit_cast(uint16_t, (_Float16)f);
}

constexpr int kAssignList = 24;       // candidates per point that a single sweep may collect before the largest v is known
constexpr int kAssignTiles = 2;       // tiles of each half staged at a time

struct AssignSmem {
  uint4 tile[2][2][kAssignTiles][kScreenTile / 8];          // [buffer][half of the centroids]
  float best[2][kAssignBlock];                              // largest v of a point in each half
  float norm[kAssignThreads / kWave];
  int n_cand[kAssignBlock];
  int again;                                                // some point's list is too short
  uint16_t cand[kAssignBlock][kAssignList];
  float cand_v[kAssignBlock][kAssignList];
};

template <bool BF16>
__global__ __launch_bounds__(kAssignThreads, 2) void kmeans_assign_kernel(const uint16_t* __restrict__ summ,
                                                                         const double* __restrict__ cent64, ScreenArgs sa,
                                                                         int32_t* __restrict__ assign,   // [U][NP]
                                                                         const int32_t* __restrict__ seq_len, int NP, int Nc,
                                                                         int P, int Hkv, int first_round) {
  __shared__ AssignSmem sm;
  const int u = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  int n_valid = (seq_len[u / Hkv] + P - 1) / P;
  n_valid = n_valid < NP ? n_valid : NP;
  const int p0 = blockIdx.x * kAssignBlock;
  if (p0 >= n_valid) return;
  const uint16_t* summ_u = summ + (size_t)u * NP * kHeadDim;
  const double* cent_u = cent64 + (size_t)u * Nc * kHeadDim;
  int32_t* assign_u = assign + (size_t)u * NP;
  const float* neg_u = sa.neg_half + (size_t)u * sa.tiles * 16;
  const uint4* frag_u = reinterpret_cast<const uint4*>(sa.frag) + (size_t)u * sa.tiles * (kScreenTile / 8);
  const int half = w >> 2, pw = (w & 3) * 64, j = lane & 15, g = lane >> 4;

  const uint16_t* shift_u = sa.shift + (size_t)u * kHeadDim + 8 * g;

  // B operands: lane (j, g) of group q holds dims 32c + 8g .. +7 of point pw + 16 q + j
  uint4 x[4][4];
  float slack[4];                                           // 2 E of the point
  float floor_v[4];                                         // what the point's largest v is not below, less the slack
  bool in_range[4];                                         // E holds
  {
    float cmax2 = 0.f;                                      // largest squared norm of the unit's centroids
    for (int c = tid; c < Nc; c += kAssignThreads) cmax2 = fmaxf(cmax2, -2.f * neg_u[c]);
    cmax2 = wave_allreduce_max(cmax2);
    if (lane == 0) sm.norm[w] = cmax2;
    if (tid == 0) sm.again = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAssignThreads / kWave; ++i) cmax2 = fmaxf(cmax2, sm.norm[i]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = p0 + pw + 16 * q + j;
      const uint16_t* row = summ_u + (size_t)(p < n_valid ? p : n_valid - 1) * kHeadDim + 8 * g;
      float n = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint4 raw = *reinterpret_cast<const uint4*>(row + 32 * c), shift = *reinterpret_cast<const uint4*>(shift_u + 32 * c);
        float f[8], sh[8];
        cvt8<BF16>(raw, f);
        cvt8<BF16>(shift, sh);
        u32* packed = reinterpret_cast<u32*>(&x[q][c]);
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float f0 = f[e] - sh[e], f1 = f[e + 1] - sh[e + 1];
          n = fmaf(f0, f0, n);
          n = fmaf(f1, f1, n);
          packed[e / 2] = narrow_exact<BF16>(f0) | (narrow_exact<BF16>(f1) << 16);
        }
      }
      n += __shfl_xor(n, 16, kWave);
      n += __shfl_xor(n, 32, kWave);
      // (2^-14 instead of the 2^-15.5 that the terms above add up to leaves room for the roundings of E itself)
      in_range[q] = n <= 0x1p120f && cmax2 <= 0x1p120f && cmax2 >= 0x1p-90f;
      const float xn = sqrtf(n);
      slack[q] = 2.f * (6.103515625e-5f * (xn * sqrtf(cmax2) + 0.5f * cmax2) + 9.5367431640625e-7f * xn);
      floor_v[q] = -INFINITY;
    }
    if (!first_round) {
      // v of the centroid that the point had before, summed in another order: within 2 E of what the sweep will find for it
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p = p0 + pw + 16 * q + j;
        int c0 = assign_u[p < n_valid ? p : n_valid - 1];
        c0 = c0 < 0 ? 0 : (c0 < Nc ? c0 : Nc - 1);
        const uint4* row = frag_u + (size_t)(c0 >> 4) * (kScreenTile / 8) + (c0 & 15) + 16 * g;
        float dot = 0.f;
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float f[8], e[8];
            cvt8<BF16>(x[q][c], f);
            cvt8<BF16>(row[(part * 4 + c) * kWave], e);
#pragma unroll
            for (int k = 0; k < 8; ++k) dot = fmaf(f[k], e[k], dot);
          }
        dot += __shfl_xor(dot, 16, kWave);
        dot += __shfl_xor(dot, 32, kWave);
        const float at_least = (dot + neg_u[c0]) - 2.f * slack[q];
        // (a cluster with a page that is no number has no v: no floor then; no v compares with a NaN)
        floor_v[q] = at_least == at_least ? at_least : -INFINITY;
      }
    }
  }
  for (int i = tid; i < kAssignBlock; i += kAssignThreads) sm.n_cand[i] = 0;

  // iteration i stages tiles 2i, 2i + 1 of the lower half and the same of the upper half, which begins with tile n_half
  // (the last tile again where there are fewer: the waves of that half then skip it)
  const int n_half = (sa.tiles + 1) / 2, n_iter = (n_half + kAssignTiles - 1) / kAssignTiles;
  static_assert(kAssignTiles == 2, "what is on its way is held in variables of their own, not in an array");
  uint4 lower0, lower1, upper0, upper1;
  float4 nh0, nh1;                                          // the norms of this wave's next tiles
  auto tile_at = [&](int h, int i, int k) -> int {
    const int t = h * n_half + i * kAssignTiles + k;
    return t < sa.tiles ? t : sa.tiles - 1;
  };
  auto fetch = [&](int i) {
    lower0 = frag_u[(size_t)tile_at(0, i, 0) * (kScreenTile / 8) + tid];
    lower1 = frag_u[(size_t)tile_at(0, i, 1) * (kScreenTile / 8) + tid];
    upper0 = frag_u[(size_t)tile_at(1, i, 0) * (kScreenTile / 8) + tid];
    upper1 = frag_u[(size_t)tile_at(1, i, 1) * (kScreenTile / 8) + tid];
    nh0 = *reinterpret_cast<const float4*>(neg_u + tile_at(half, i, 0) * 16 + 4 * g);
    nh1 = *reinterpret_cast<const float4*>(neg_u + tile_at(half, i, 1) * 16 + 4 * g);
  };
  static_assert(kScreenTile / 8 == kAssignThreads, "one 16-byte unit of a tile per thread");
  // f(t, v): v[q] = the values of rows 4g .. 4g+3 of tile t for this lane's point of group q
  auto sweep = [&](auto f) {
    auto product = [&](int i, int k, const float4& nh) {
      const int in_half = i * kAssignTiles + k, t = half * n_half + in_half;
      if (in_half >= n_half || t >= sa.tiles) return;
      const f32x4_c start = f32x4_c{nh.x, nh.y, nh.z, nh.w};
      f32x4_c v[4] = {start, start, start, start};
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint4 a = sm.tile[i & 1][half][k][(part * 4 + c) * kWave + lane];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = mfma_16x16x32<BF16>(a, x[q][c], v[q]);
        }
      f(t, v);
    };
    fetch(0);
    for (int i = 0; i < n_iter; ++i) {
      sm.tile[i & 1][0][0][tid] = lower0;
      sm.tile[i & 1][0][1][tid] = lower1;
      sm.tile[i & 1][1][0][tid] = upper0;
      sm.tile[i & 1][1][1][tid] = upper1;
      const float4 n0 = nh0, n1 = nh1;
      if (i + 1 < n_iter) fetch(i + 1);
      __syncthreads();                                      // (buffer i & 1 is written again two iterations on, after the next barrier)
      product(i, 0, n0);
      product(i, 1, n1);
    }
    __syncthreads();
  };
  auto largest = [](const f32x4_c& v) -> float { return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])); };
  auto collect = [&](int t, const f32x4_c (&v)[4], const float (&least)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!(largest(v[q]) >= least[q])) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v[q][e] >= least[q] && t * 16 + 4 * g + e < Nc) {
          const int at = atomicAdd(&sm.n_cand[pw + 16 * q + j], 1);
          if (at < kAssignList) {
            sm.cand[pw + 16 * q + j][at] = (uint16_t)(t * 16 + 4 * g + e);
            sm.cand_v[pw + 16 * q + j][at] = v[q][e];
          }
        }
    }
  };

  bool two_sweeps = first_round != 0;
  float top[4];
  if (!two_sweeps) {
    // one sweep: whatever is within the slack of the largest v so far, or of the floor; the largest v of all is in the list
#pragma unroll
    for (int q = 0; q < 4; ++q) top[q] = floor_v[q];
    sweep([&](int t, const f32x4_c (&v)[4]) {
      collect(t, v, top);
#pragma unroll
      for (int q = 0; q < 4; ++q) top[q] = fmaxf(top[q], largest(v[q]) - slack[q]);
    });
    for (int i = tid; i < kAssignBlock; i += kAssignThreads)
      if (sm.n_cand[i] > kAssignList) sm.again = 1;
    __syncthreads();
    if (sm.again) {
      // a list did not hold them all (every wave sees it): as in the first round, with what this sweep has found
      two_sweeps = true;
      __syncthreads();
      for (int i = tid; i < kAssignBlock; i += kAssignThreads) sm.n_cand[i] = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) top[q] += slack[q];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) top[q] = -INFINITY;
    sweep([&](int, const f32x4_c (&v)[4]) {
#pragma unroll
      for (int q = 0; q < 4; ++q) top[q] = fmaxf(top[q], largest(v[q]));
    });
  }
  if (two_sweeps) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      top[q] = fmaxf(top[q], __shfl_xor(top[q], 16, kWave));
      top[q] = fmaxf(top[q], __shfl_xor(top[q], 32, kWave));
      if (g == 0) sm.best[half][pw + 16 * q + j] = top[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) top[q] = fmaxf(top[q], sm.best[half ^ 1][pw + 16 * q + j]) - slack[q];
    sweep([&](int t, const f32x4_c (&v)[4]) { collect(t, v, top); });
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (g == 0 && half == 0) sm.best[0][pw + 16 * q + j] = in_range[q] ? slack[q] : -1.f;   // (for the point's thread)
  __syncthreads();

  if (tid < kAssignBlock && p0 + tid < n_valid) {
    int n = sm.n_cand[tid];
    const float within = sm.best[0][tid];
    int kept = 0;
    bool open = n < 1 || n > kAssignList || !(within >= 0.f);
    if (!open) {
      float most = sm.cand_v[tid][0];
      for (int k = 1; k < n; ++k) most = fmaxf(most, sm.cand_v[tid][k]);
      for (int k = 0; k < n; ++k)
        if (sm.cand_v[tid][k] >= most - within) sm.cand[tid][kept++] = sm.cand[tid][k];
      open = kept > kAssignCap;
      n = kept;
    }
    if (open) {
      sa.hard[(size_t)u * NP + atomicAdd(&sa.n_hard[u], 1)] = p0 + tid;
    } else {
      int bc = sm.cand[tid][0];
      if (n > 1) {
        const uint16_t* row = summ_u + (size_t)(p0 + tid) * kHeadDim;
        double bd = INFINITY;
        bc = 0x7fffffff;
        for (int k = 0; k < n; ++k) {
          const int c = sm.cand[tid][k];
          const double* crow = cent_u + (size_t)c * kHeadDim;
          double acc = 0.0;
          for (int d = 0; d < kHeadDim; d += 2) {
            const u32 raw = *reinterpret_cast<const u32*>(row + d);
            const double2 cv = *reinterpret_cast<const double2*>(crow + d);
            const double e0 = widen_kv<BF16>((uint16_t)raw) - cv.x, e1 = widen_kv<BF16>((uint16_t)(raw >> 16)) - cv.y;
            acc = fma(e0, e0, acc);
            acc = fma(e1, e1, acc);
          }
          if (acc < bd || (acc == bd && c < bc)) { bd = acc; bc = c; }
        }
      }
      assign_u[p0 + tid] = bc < Nc ? bc : 0;
    }
  }
}

// The pages that the screening leaves open against all centroids of their unit in fp64.  A launch of its own, so
// that they spread over the chip however they lie among the blocks of the screening, 4 blocks per CU over all units.
// A block takes 16 pages at a time, so that a centroid is read once for 16, or 4 where all of a unit's blocks have
// no more than that to do: bound by the latency of one block's run through the centroids.  (ms of a build of
// 4 rounds, 8192 pages against 4096 centroids, done by the block of the screening that met the page, and so: one unit,
// nearly all pages open 24.8 and 5.2, every vector 40 times 16.4 and 4.2, few pages open 3.2 and 2.0; eight units 26.4
// and 18.5, 18.4 and 13.6, 3.5 and 4.0.)
constexpr int kExhaustiveThreads = 256, kExhaustivePages = 16, kExhaustiveFew = 4;
struct ExhaustiveSmem {
  static constexpr int NW = kExhaustiveThreads / kWave;
  double pts[kExhaustivePages][kHeadDim];
  double best_d[kExhaustivePages][NW];
  int best_c[kExhaustivePages][NW];
};

template <bool BF16, int PAGES>
__device__ __forceinline__ void assign_exhaustive(ExhaustiveSmem& sm, const uint16_t* __restrict__ summ_u, const double* __restrict__ cent_u,
                                                  int32_t* __restrict__ assign_u, const int32_t* __restrict__ hard, int n_hard, int Nc) {
  constexpr int NW = ExhaustiveSmem::NW;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  for (int first = blockIdx.x * PAGES; first < n_hard; first += gridDim.x * PAGES) {
    const int n = n_hard - first < PAGES ? n_hard - first : PAGES;
    __syncthreads();                                        // (the pages before these are done)
    for (int i = tid; i < PAGES * kHeadDim; i += kExhaustiveThreads) {
      const int pi = i / kHeadDim, d = i % kHeadDim;
      sm.pts[pi][d] = pi < n ? widen_kv<BF16>(summ_u[(size_t)hard[first + pi] * kHeadDim + d]) : 0.0;
    }
    __syncthreads();
    double bd[PAGES];
    int bc[PAGES];
#pragma unroll
    for (int i = 0; i < PAGES; ++i) { bd[i] = INFINITY; bc[i] = 0x7fffffff; }
    for (int c = tid; c < Nc; c += kExhaustiveThreads) {
      const double* crow = cent_u + (size_t)c * kHeadDim;
      double acc[PAGES];
#pragma unroll
      for (int i = 0; i < PAGES; ++i) acc[i] = 0.0;
      for (int d = 0; d < kHeadDim; d += 2) {
        const double2 cv = *reinterpret_cast<const double2*>(crow + d);
#pragma unroll
        for (int i = 0; i < PAGES; ++i) {
          const double e0 = sm.pts[i][d] - cv.x, e1 = sm.pts[i][d + 1] - cv.y;
          acc[i] = fma(e0, e0, acc[i]);
          acc[i] = fma(e1, e1, acc[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < PAGES; ++i)
        if (acc[i] < bd[i]) { bd[i] = acc[i]; bc[i] = c; }  // centroids come in ascending order per thread
    }
    // smallest (distance, centroid) per page over the block
#pragma unroll
    for (int i = 0; i < PAGES; ++i) {
      double d = bd[i];
      int c = bc[i];
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        const double od = __shfl_xor(d, m, kWave);
        const int oc = __shfl_xor(c, m, kWave);
        if (od < d || (od == d && oc < c)) { d = od; c = oc; }
      }
      if (lane == 0) { sm.best_d[i][w] = d; sm.best_c[i][w] = c; }
    }
    __syncthreads();
    if (tid < n) {
      double d = sm.best_d[tid][0];
      int c = sm.best_c[tid][0];
      for (int j = 1; j < NW; ++j) {
        const double od = sm.best_d[tid][j];
        const int oc = sm.best_c[tid][j];
        if (od < d || (od == d && oc < c)) { d = od; c = oc; }
      }
      assign_u[hard[first + tid]] = c < Nc ? c : 0;   // (no distance is a number: any cluster, within bounds)
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(kExhaustiveThreads) void kmeans_exhaustive_kernel(const uint16_t* __restrict__ summ,
                                                                             const double* __restrict__ cent64, ScreenArgs sa,
                                                                             int32_t* __restrict__ assign, int NP, int Nc) {
  __shared__ ExhaustiveSmem sm;
  const int u = blockIdx.y, n_hard = sa.n_hard[u];
  const uint16_t* summ_u = summ + (size_t)u * NP * kHeadDim;
  const double* cent_u = cent64 + (size_t)u * Nc * kHeadDim;
  int32_t* assign_u = assign + (size_t)u * NP;
  const int32_t* hard = sa.hard + (size_t)u * NP;
  if (n_hard <= kExhaustiveFew * (int)gridDim.x)
    assign_exhaustive<BF16, kExhaustiveFew>(sm, summ_u, cent_u, assign_u, hard, n_hard, Nc);
  else
    assign_exhaustive<BF16, kExhaustivePages>(sm, summ_u, cent_u, assign_u, hard, n_hard, Nc);
}

constexpr int kCsrThreads = 1024;

constexpr int kRankMost = 128;        // members of a cluster up to which each finds its own place among them

// One block per unit: cluster_start [Nc+1] and cluster_pages [NP] (pages of every cluster in
// ascending order) from assign; page_cluster [NP], if given, receives the assignment too.  Latency-bound
// and alone on its CU, so everything happens in LDS: the counts, their scan, the members in arrival
// order, and each page's place = the number of smaller pages among its cluster's members.  The reads
// for that grow with the square of a cluster's size, so a cluster of more than kRankMost pages is
// gone through by one wave instead, in page order.
__global__ __launch_bounds__(kCsrThreads) void kmeans_csr_kernel(const int32_t* __restrict__ assign,
                                                                int32_t* __restrict__ cluster_start,   // [U][Nc+1]
                                                                int32_t* __restrict__ cluster_pages,   // [U][NP]
                                                                int32_t* __restrict__ page_cluster,    // [U][NP] or null
                                                                const int32_t* __restrict__ seq_len, int NP, int Nc,
                                                                int P, int Hkv) {
  __shared__ uint16_t as[KVD_FAST_MAX_PAGES], members[KVD_FAST_MAX_PAGES];
  __shared__ int cur[KVD_MAX_CENTROIDS];                    // counts; then the next place of a cluster; in the end its end
  __shared__ int scan_smem[kCsrThreads / kWave + 1];
  __shared__ int large[KVD_FAST_MAX_PAGES / kRankMost], n_large;
  const int u = blockIdx.x, tid = threadIdx.x;
  int n_valid = (seq_len[u / Hkv] + P - 1) / P;
  n_valid = n_valid < NP ? n_valid : NP;
  const int32_t* as_u = assign + (size_t)u * NP;
  int32_t* start = cluster_start + (size_t)u * (Nc + 1);
  int32_t* pages = cluster_pages + (size_t)u * NP;
  int32_t* pc = page_cluster != nullptr ? page_cluster + (size_t)u * NP : nullptr;
  for (int c = tid; c < Nc; c += kCsrThreads) cur[c] = 0;
  if (tid == 0) n_large = 0;
  __syncthreads();
  for (int p = tid; p < NP; p += kCsrThreads) {
    const int c = p < n_valid ? as_u[p] : -1;
    if (pc != nullptr) pc[p] = c;
    if (c < 0) { pages[p] = -1; continue; }
    as[p] = (uint16_t)c;
    atomicAdd(&cur[c], 1);
  }
  __syncthreads();
  // exclusive scan of the counts, 1024 clusters at a time
  int base = 0;
  for (int c0 = 0; c0 < Nc; c0 += kCsrThreads) {
    const int c = c0 + tid, cnt = c < Nc ? cur[c] : 0;
    int total;
    const int at = base + block_exclusive_scan<kCsrThreads>(cnt, scan_smem, total);
    base += total;
    if (c < Nc) {
      start[c] = at;
      cur[c] = at;
      if (cnt > kRankMost) large[atomicAdd(&n_large, 1)] = c;
    }
  }
  if (tid == 0) start[Nc] = base;
  __syncthreads();
  for (int p = tid; p < n_valid; p += kCsrThreads) members[atomicAdd(&cur[as[p]], 1)] = (uint16_t)p;
  __syncthreads();
  for (int p = tid; p < n_valid; p += kCsrThreads) {
    const int c = as[p], b = c > 0 ? cur[c - 1] : 0, e = cur[c];
    if (e - b > kRankMost) continue;
    int before = 0;
    for (int i = b; i < e; ++i) before += members[i] < p ? 1 : 0;
    pages[b + before] = p;
  }
  const int lane = tid & (kWave - 1);
  for (int i = tid / kWave; i < n_large; i += kCsrThreads / kWave) {
    const int c = large[i];
    int at = c > 0 ? cur[c - 1] : 0;
    for (int p0 = 0; p0 < n_valid; p0 += kWave) {
      const int p = p0 + lane;
      const u64 mine = __ballot(p < n_valid && as[p] == c);
      if ((mine >> lane) & 1ull) pages[at + __popcll(mine & ((1ull << lane) - 1ull))] = p;
      at += __popcll(mine);
    }
  }
}

// One wave per centroid, two dims per lane: new centroid = mean of the members' summaries in ascending page order.
template <bool BF16>
__global__ __launch_bounds__(kCentroidWaves* kWave) void kmeans_update_kernel(const uint16_t* __restrict__ summ,
                                                                             double* __restrict__ cent64, ScreenArgs sa,
                                                                             const int32_t* __restrict__ cluster_start,
                                                                             const int32_t* __restrict__ cluster_pages, int NP,
                                                                             int Nc) {
  const int c = blockIdx.x * kCentroidWaves + threadIdx.x / kWave, u = blockIdx.y, lane = threadIdx.x & (kWave - 1);
  if (c >= Nc) return;
  if (c == 0 && lane == 0) sa.n_hard[u] = 0;                // for the next round
  const int b = cluster_start[(size_t)u * (Nc + 1) + c], e = cluster_start[(size_t)u * (Nc + 1) + c + 1];
  double2* cent = reinterpret_cast<double2*>(cent64 + ((size_t)u * Nc + c) * kHeadDim) + lane;
  double2 x;
  if (e == b) {
    x = *cent;                                              // an empty cluster keeps its centroid
  } else {
    const int32_t* pages = cluster_pages + (size_t)u * NP;
    double a0 = 0.0, a1 = 0.0;
    for (int i0 = b; i0 < e; i0 += kWave) {
      // a wave's worth of members at a time, the rows of four on their way together
      const int n = e - i0 < kWave ? e - i0 : kWave;
      const int mine = pages[i0 + (lane < n ? lane : n - 1)];
      for (int i = 0; i < n; i += 4) {
        u32 raw[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int page = __builtin_amdgcn_readlane(mine, i + k < n ? i + k : n - 1);
          raw[k] = *reinterpret_cast<const u32*>(summ + ((size_t)u * NP + page) * kHeadDim + 2 * lane);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i + k < n) {
            a0 += widen_kv<BF16>((uint16_t)raw[k]);
            a1 += widen_kv<BF16>((uint16_t)(raw[k] >> 16));
          }
      }
    }
    x = make_double2(a0 / (double)(e - b), a1 / (double)(e - b));
    *cent = x;
  }
  store_screen<BF16>(sa, u, c, x.x, x.y);
}

template <bool BF16>
__global__ __launch_bounds__(kHeadDim) void kmeans_store_kernel(const double* __restrict__ cent64, uint16_t* __restrict__ centroids,
                                                               int Nc) {
  const size_t i = ((size_t)blockIdx.y * Nc + blockIdx.x) * kHeadDim + threadIdx.x;
  centroids[i] = f64_to_kv<BF16>(cent64[i]);
}

// ---------------------------------------------------------------------------------------------
// decode: clusters -> pages (see kvd_cluster_body.h)
// ---------------------------------------------------------------------------------------------
constexpr int kClusterThreads = 1024;

// One block per unit.
__global__ __launch_bounds__(kClusterThreads) void cluster_select_kernel(const float* __restrict__ scores,
                                                                        const int32_t* __restrict__ cluster_start,
                                                                        const int32_t* __restrict__ cluster_pages,
                                                                        int32_t* __restrict__ sel_pages,
                                                                        const int32_t* __restrict__ seq_len, int NP, int Nc,
                                                                        int P, int k, int sink, int recent, int Hkv, int u0) {
  extern __shared__ __align__(16) unsigned char cs_raw[];
  ClusterSelectSmem<kClusterThreads>& sm = *reinterpret_cast<ClusterSelectSmem<kClusterThreads>*>(cs_raw);
  cluster_select_body<kClusterThreads, false>(scores, cluster_start, cluster_pages, sel_pages, seq_len, NP, Nc, P, k, sink,
                                              recent, Hkv, blockIdx.x + u0, sm);
}

// page_cluster [NP] of unit blockIdx.x from its cluster lists: -1, then the cluster of every listed page.
__global__ __launch_bounds__(kCsrThreads) void cluster_inverse_kernel(const int32_t* __restrict__ cluster_start,
                                                                     const int32_t* __restrict__ cluster_pages,
                                                                     int32_t* __restrict__ page_cluster, int NP, int Nc) {
  const int u = blockIdx.x, tid = threadIdx.x;
  const int32_t* start = cluster_start + (size_t)u * (Nc + 1);
  const int32_t* pages = cluster_pages + (size_t)u * NP;
  int32_t* pc = page_cluster + (size_t)u * NP;
  for (int p = tid; p < NP; p += kCsrThreads) pc[p] = -1;
  __syncthreads();
  for (int c = tid; c < Nc; c += kCsrThreads) {
    int b = start[c], e = start[c + 1];
    b = b < 0 ? 0 : b;
    e = e > NP ? NP : e;
    for (int i = b; i < e; ++i) {
      const int p = pages[i];
      if (p >= 0 && p < NP) pc[p] = c;
    }
  }
}

}  // namespace kvd

bool kvd_centroid_mode(const kvd_ctx* c) { return c->Nc > 0; }

hipError_t kvd_prepare_cluster_select(void) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kvd::cluster_select_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(kvd::ClusterSelectSmem<kvd::kClusterThreads>));
}

hipError_t kvd_launch_cluster_select(kvd_ctx* c, int layer, const float* scores, int32_t* sel_pages, int u0, int u1,
                                     hipStream_t s) {
  using namespace kvd;
  if (u1 <= u0) return hipSuccess;
  const size_t lu = (size_t)layer * c->U;
  hipLaunchKernelGGL(cluster_select_kernel, dim3(u1 - u0), dim3(kClusterThreads), sizeof(ClusterSelectSmem<kClusterThreads>), s, scores,
                     c->cluster_start + lu * (c->Nc + 1), c->cluster_pages + lu * c->NP, sel_pages, c->d_seq_len, c->NP, c->Nc,
                     c->P, c->k, c->cfg.sink_pages, c->cfg.recent_pages, c->Hkv, u0);
  return hipGetLastError();
}

hipError_t kvd_launch_cluster_inverse(kvd_ctx* c, int layer, hipStream_t s) {
  using namespace kvd;
  const size_t lu = (size_t)layer * c->U;
  hipLaunchKernelGGL(cluster_inverse_kernel, dim3(c->U), dim3(kCsrThreads), 0, s, c->cluster_start + lu * (c->Nc + 1),
                     c->cluster_pages + lu * c->NP, c->d_page_cluster + lu * c->NP, c->NP, c->Nc);
  return hipGetLastError();
}

// k-means over the layer's page summaries; assign_trace (device, [iterations][U][NP], or null)
// receives the assignment of every round.  Synchronous.
hipError_t kvd_run_build_centroids(kvd_ctx* c, int layer, int iterations, int32_t* assign_trace, hipStream_t s) {
  using namespace kvd;
  const size_t lu = (size_t)layer * c->U;
  const uint16_t* summ = reinterpret_cast<const uint16_t*>(c->summaries) + lu * c->NP * kHeadDim;
  uint16_t* cent = reinterpret_cast<uint16_t*>(c->centroids) + lu * c->Nc * kHeadDim;
  int32_t* cstart = c->cluster_start + lu * (c->Nc + 1);
  int32_t* cpages = c->cluster_pages + lu * c->NP;
  ScreenArgs sa;
  sa.tiles = (c->Nc + 15) / 16;
  // one temporary block: fp64 centroids, screening tiles, half norms, assignment, shifts, pages left open by the screening
  const size_t n_cent = (size_t)c->U * c->Nc, n_tiles = (size_t)c->U * sa.tiles, n_points = (size_t)c->U * c->NP;
  size_t at = 0;
  auto place = [&](size_t bytes) { const size_t o = at; at += (bytes + 255) & ~(size_t)255; return o; };
  const size_t o_cent = place(n_cent * kHeadDim * sizeof(double)), o_frag = place(n_tiles * kScreenTile * 2),
               o_neg = place(n_tiles * 16 * sizeof(float)), o_assign = place(n_points * sizeof(int32_t)),
               o_shift = place((size_t)c->U * kHeadDim * 2), o_hard = place(n_points * sizeof(int32_t)), o_n_hard = place((size_t)c->U * sizeof(int32_t));
  // Kept with the context up to 64 MB (its size is the same in every call): allocating and freeing it took 20 to 100 us of one
  // (4 units x 152 pages and 76 centroids, 5 rounds, with its summaries 306 us with and 286 without).  Two calls at once, from two
  // threads, have one each: the kept one is taken out of the context meanwhile.
  constexpr size_t kKept = (size_t)64 << 20;
  hipError_t e = hipSuccess;
  char* temp = __atomic_exchange_n(&c->build_temp, static_cast<char*>(nullptr), __ATOMIC_ACQ_REL);
  if (temp == nullptr) e = hipMalloc(reinterpret_cast<void**>(&temp), at);
  if (e == hipSuccess) {
    double* cent64 = reinterpret_cast<double*>(temp + o_cent);
    int32_t* assign = reinterpret_cast<int32_t*>(temp + o_assign);
    sa.frag = reinterpret_cast<uint16_t*>(temp + o_frag);
    sa.neg_half = reinterpret_cast<float*>(temp + o_neg);
    sa.shift = reinterpret_cast<uint16_t*>(temp + o_shift);
    sa.hard = reinterpret_cast<int32_t*>(temp + o_hard);
    sa.n_hard = reinterpret_cast<int32_t*>(temp + o_n_hard);
    int open_blocks = (4 * c->n_cus + c->U - 1) / c->U;
    if (open_blocks > (c->NP + kExhaustiveFew - 1) / kExhaustiveFew) open_blocks = (c->NP + kExhaustiveFew - 1) / kExhaustiveFew;
    const dim3 per_centroid(c->Nc, c->U), per_tile_row((sa.tiles * 16 + kCentroidWaves - 1) / kCentroidWaves, c->U);
    const dim3 per_points((c->NP + kAssignBlock - 1) / kAssignBlock, c->U), centroid_block(kCentroidWaves * kWave);
#define KVD_DT(KERNEL, ...)                                                    \
  do {                                                                         \
    if (c->bf16) hipLaunchKernelGGL((KERNEL<true>), __VA_ARGS__);              \
    else hipLaunchKernelGGL((KERNEL<false>), __VA_ARGS__);                     \
  } while (0)
    KVD_DT(kmeans_shift_kernel, dim3(kHeadDim / 8, c->U), dim3(kShiftThreads), 0, s, summ, sa, c->d_seq_len, c->NP, c->P, c->Hkv);
    KVD_DT(kmeans_init_kernel, per_tile_row, centroid_block, 0, s, summ, cent64, sa, c->d_seq_len, c->NP, c->Nc, c->P, c->Hkv);
    for (int it = 0; it < iterations && e == hipSuccess; ++it) {
      KVD_DT(kmeans_assign_kernel, per_points, dim3(kAssignThreads), 0, s, summ, cent64, sa, assign, c->d_seq_len, c->NP, c->Nc,
             c->P, c->Hkv, it == 0 ? 1 : 0);
      KVD_DT(kmeans_exhaustive_kernel, dim3(open_blocks, c->U), dim3(kExhaustiveThreads), 0, s, summ, cent64, sa, assign, c->NP, c->Nc);
      if (assign_trace != nullptr)
        e = hipMemcpyAsync(assign_trace + (size_t)it * c->U * c->NP, assign, (size_t)c->U * c->NP * sizeof(int32_t),
                           hipMemcpyDeviceToDevice, s);
      hipLaunchKernelGGL(kmeans_csr_kernel, dim3(c->U), dim3(kCsrThreads), 0, s, assign, cstart, cpages,
                         it + 1 == iterations ? c->d_page_cluster + lu * c->NP : nullptr, c->d_seq_len, c->NP, c->Nc, c->P, c->Hkv);
      KVD_DT(kmeans_update_kernel, per_tile_row, centroid_block, 0, s, summ, cent64, sa, cstart, cpages, c->NP, c->Nc);
    }
    KVD_DT(kmeans_store_kernel, per_centroid, dim3(kHeadDim), 0, s, cent64, cent, c->Nc);
#undef KVD_DT
    if (e == hipSuccess) e = hipGetLastError();
    const hipError_t e2 = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e2;
  }
  if (e == hipSuccess && at <= kKept) temp = __atomic_exchange_n(&c->build_temp, temp, __ATOMIC_ACQ_REL);
  if (temp != nullptr) (void)hipFree(temp);
  return e;
}
