// GQA decode attention over the selected pages of one unit by one workgroup (System Overview:
// attention runs over the union of resident and newly fetched entries).  The selected pages of a
// unit are split over several workgroups (split-K); each streams its K/V pages from the slot pool
// once and keeps an fp32 online softmax per query head; the split partials are merged by
// log-sum-exp, either by the last workgroup of the unit to finish or by a second kernel.
// Shared by the stand-alone attention kernels and the single-launch layer-step kernel.
#pragma once
#include <type_traits>

#include "kvd_device.h"
#include "kvd_internal.h"
#include "kvd_tile_layout.h"

namespace kvd {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct AttnArgs {
  const uint16_t* q;         // [B][Hq][D]
  const char* pool;          // [U][Cmax] slots of the layer
  const int32_t* sel_pages;  // [U][k]
  const int32_t* sel_slots;  // [U][k]
  u64* sel_entry;            // [U][k]: what a HANDOFF caller reads instead of the two (see pack_sel_entry); cleared after use
  int32_t* error;            // host-visible word, raised when the wait for the entries runs out
  long long wait_limit;      // bound of that wait in ticks of the 100 MHz wall clock
  const int32_t* seq_len;    // [B]
  float* part_acc;           // [U][S][G][D]
  float* part_ml;            // [U][S][G][2]
  int32_t* ticket;           // [U], zero between launches
  float* out;                // [B][Hq][D]
  float* lse;                // [B][Hq] or null
  int k, P, Cmax, Hq, Hkv, G, S, per_split, fuse_merge, u0;
  int take;                  // consecutive splits that a workgroup takes (other than 1 only in launches of several layers)
  unsigned page_bytes;
  float scale_log2;          // softmax scale * log2(e)
};

// GMAX query heads per KV head at most, NW waves per workgroup.  What a wave leaves of a split is G rows of kPartStride
// floats: the accumulators, then maximum and sum.  `part` holds one split of the waves; a caller with more LDS behind it may
// have a workgroup take several splits (part_of).
constexpr int kPartStride = kHeadDim + 4;   // (a multiple of 16 bytes)
template <int GMAX, int NW, int CAP = kAttnIdxCap>
struct AttnSmem {
  int32_t page[CAP], slot[CAP];
  int is_last;
  __align__(16) float part[NW * GMAX * kPartStride];
  __device__ __forceinline__ float* part_of(int v, int w, int g, int G) { return part + ((v * NW + w) * G + g) * kPartStride; }
};

// GT > 0: the group size is the compile-time GT; GT == 0: it is a.G (at most KVD_MAX_GROUP).
template <int GT>
__device__ __forceinline__ int group_size(const AttnArgs& a) { return GT > 0 ? GT : a.G; }
template <int GT>
struct GroupMax { static constexpr int value = GT > 0 ? GT : KVD_MAX_GROUP; };

// Log-sum-exp merge of the S split partials of unit u into out / lse, by one workgroup of NT threads: the largest of the
// maxima, then the sums in the order of the splits, each times 2^(its maximum - the largest).  Bound by the trips to memory.
// Up to 8 splits every thread fetches all it needs at once and works the weights out for itself.  With more, the maxima and
// sums go through LDS (`lds`, kMergeFloats), where a weight is computed once per split and head, while the accumulators are on
// their way, up to 32 at a time.  (us per step with batches of 8 for any number and so: 2 units with 15 splits, G = 7, 17.1
// and 15.8; 8 with 16 splits of 32 tiles 31.9 and 31.4; but through LDS 8 units with 8 splits 13.4 and 13.7.)  HANDOFF: the
// partials were written by other workgroups of the same launch.
constexpr int kMergeFloats = (3 * KVD_MAX_SPLITS + 1) * KVD_MAX_GROUP;
template <int GT, int NT, bool HANDOFF>
__device__ __forceinline__ void merge_splits(const AttnArgs& a, int u, float* lds) {
  const int G = group_size<GT>(a), S = a.S;
  const int tid = threadIdx.x;
  const int b = u / a.Hkv, h = u % a.Hkv;
  if (S <= 8) {
    for (int idx = tid; idx < G * kHeadDim; idx += NT) {
      const int g = idx / kHeadDim, d = idx % kHeadDim;
      const float* ml = a.part_ml + ((size_t)u * S * G + g) * 2;
      const float* pa = a.part_acc + ((size_t)u * S * G + g) * kHeadDim + d;
      float mv[8], lv[8], av[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int s = i < S ? i : S - 1;
        if (HANDOFF) {
          mv[i] = load_agent(ml + (size_t)s * G * 2);
          lv[i] = load_agent(ml + (size_t)s * G * 2 + 1);
          av[i] = load_agent(pa + (size_t)s * G * kHeadDim);
        } else {
          mv[i] = ml[(size_t)s * G * 2];
          lv[i] = ml[(size_t)s * G * 2 + 1];
          av[i] = pa[(size_t)s * G * kHeadDim];
        }
      }
      float M = -INFINITY, L = 0.f, A = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) M = fmaxf(M, mv[i]);
      const float Ms = M == -INFINITY ? 0.f : M;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i < S) {
          const float sc = exp2f(mv[i] - Ms);
          L += lv[i] * sc;
          A += av[i] * sc;
        }
      const size_t row = (size_t)b * a.Hq + (size_t)h * G + g;
      a.out[row * kHeadDim + d] = A / L;
      if (a.lse != nullptr && d == 0) a.lse[row] = (M + log2f(L)) * kLn2;
    }
    return;
  }
  auto merge = [&](auto batch) {
    constexpr int N = decltype(batch)::value;            // splits whose accumulators are fetched at a time
    const int SP = (S + N - 1) / N * N;
    float* mx = lds;                                     // [G][SP] maxima
    float* weight = lds + SP * G;                        // [G][SP]
    float* sum = lds + 2 * SP * G;                       // [G][SP]
    float* top = lds + 3 * SP * G;                       // [G]
    const u64* ml = reinterpret_cast<const u64*>(a.part_ml) + (size_t)u * S * G;
    for (int i = tid; i < SP * G; i += NT) {
      const int s = i / G, at = (i % G) * SP + s;
      u64 v = ((u64)0 << 32) | as_u32(-INFINITY);
      if (s < S) v = HANDOFF ? load_agent(ml + i) : ml[i];
      mx[at] = as_f32((u32)v);
      sum[at] = as_f32((u32)(v >> 32));
    }
    const __amdgpu_buffer_rsrc_t acc = __builtin_amdgcn_make_buffer_rsrc(a.part_acc + (size_t)u * S * G * kHeadDim, 0, S * G * kHeadDim * 4, 0x00020000);
    for (int idx0 = 0; idx0 < G * kHeadDim; idx0 += NT) {
      const int idx = idx0 + tid, g = idx / kHeadDim, d = idx % kHeadDim;
      float av[N];
      // (splits beyond S read as zero: the whole offset is in the operand that the buffer's bounds are checked against, which
      // the scalar offset is not)
      auto fetch = [&](int s0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
          av[i] = as_f32(__builtin_amdgcn_raw_buffer_load_b32(acc, (idx + (s0 + i) * G * kHeadDim) * 4, 0, HANDOFF ? 16 : 0));
      };
      fetch(0);
      if (idx0 == 0) {
        __syncthreads();
        for (int i = tid; i < SP * G; i += NT) {
          const int gi = i / SP;
          float m = -INFINITY;
          for (int s = 0; s < S; ++s) m = fmaxf(m, mx[gi * SP + s]);
          weight[i] = exp2f(mx[i] - (m == -INFINITY ? 0.f : m));
          if (i == gi * SP) top[gi] = m;
        }
        __syncthreads();
      }
      if (idx >= G * kHeadDim) continue;
      float L = 0.f, A = 0.f;
      for (int s0 = 0; s0 < SP; s0 += N) {
        if (s0 > 0) fetch(s0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float sc = weight[g * SP + s0 + i];
          L += sum[g * SP + s0 + i] * sc;
          A += av[i] * sc;
        }
      }
      const size_t row = (size_t)b * a.Hq + (size_t)h * G + g;
      a.out[row * kHeadDim + d] = A / L;
      if (a.lse != nullptr && d == 0) a.lse[row] = (top[g] + log2f(L)) * kLn2;
    }
  };
  if (S <= 16) merge(std::integral_constant<int, 16>());
  else merge(std::integral_constant<int, 32>());
}

// Workgroup epilogue.  The waves have left what they have of splits [split, split + n) in `sm`; merge them and write
// the splits' partials.  With fuse_merge the partials travel with device-scope stores and the
// last workgroup of the unit to arrive (a ticket counter) merges all S of them; a workgroup that has taken all S
// merges them itself, in the same order and with the same operations, so that the output does not depend on how many splits
// a workgroup takes.
// Returns true in the workgroup that completed the unit's output (with a separate merge kernel:
// never).
// SEVERAL: a workgroup may have taken more than one split.
template <int GT, int NT, bool SEVERAL, class Smem>
__device__ __forceinline__ bool finish_splits(const AttnArgs& a, Smem& sm, int u, int split, int n_taken) {
  const int n = SEVERAL ? n_taken : 1;
  constexpr int NW = NT / kWave;
  const int G = group_size<GT>(a);
  const int tid = threadIdx.x;
  const int b = u / a.Hkv, h = u % a.Hkv;
  const bool fused = a.fuse_merge != 0;
  __syncthreads();
  for (int idx = tid; idx < G * kHeadDim; idx += NT) {
    const int g = idx / kHeadDim, d = idx % kHeadDim;
    float MM = -INFINITY, LL = 0.f, AA = 0.f;            // over the splits, when they are all here (as merge_splits has it)
    if (SEVERAL && n == a.S)
      for (int v = 0; v < n; ++v)
#pragma unroll
        for (int w = 0; w < NW; ++w) MM = fmaxf(MM, sm.part_of(v, w, g, G)[kHeadDim]);
    for (int v = 0; v < n; ++v) {
      float m[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) m[w] = sm.part_of(v, w, g, G)[kHeadDim];
      float M = m[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, m[w]);
      const float Ms = M == -INFINITY ? 0.f : M;
      float L = 0.f, A = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float* p = sm.part_of(v, w, g, G);
        const float sc = exp2f(m[w] - Ms);
        L += p[kHeadDim + 1] * sc;
        A += p[d] * sc;
      }
      if (a.S == 1) {
        MM = M; LL = L; AA = A;
      } else if (SEVERAL && n == a.S) {
        const float sc = exp2f(M - (MM == -INFINITY ? 0.f : MM));
        LL += L * sc;
        AA += A * sc;
      } else {
        const size_t base = ((size_t)u * a.S + split + v) * G + g;
        if (fused) {
          store_agent(&a.part_acc[base * kHeadDim + d], A);
          if (d == 0) {
            store_agent(&a.part_ml[base * 2], M);
            store_agent(&a.part_ml[base * 2 + 1], L);
          }
        } else {
          a.part_acc[base * kHeadDim + d] = A;
          if (d == 0) {
            a.part_ml[base * 2] = M;
            a.part_ml[base * 2 + 1] = L;
          }
        }
      }
    }
    if (n == a.S) {
      const size_t row = (size_t)b * a.Hq + (size_t)h * G + g;
      a.out[row * kHeadDim + d] = AA / LL;
      if (a.lse != nullptr && d == 0) a.lse[row] = (MM + log2f(LL)) * kLn2;
    }
  }
  if (n == a.S) {
    // (a HANDOFF caller's entries were read into LDS before the first barrier: blank them for the next launch)
    if (a.sel_entry != nullptr)
      for (int i = tid; i < a.k; i += NT) store_agent(&a.sel_entry[(size_t)u * a.k + i], 0ull);
    return true;
  }
  if (!fused) return false;
  wave_drain_memory();                               // this wave's partials have been acknowledged
  __syncthreads();
  if (tid == 0) {
    const int arrivals = SEVERAL ? (a.S + a.take - 1) / a.take : a.S;
    const int t = __hip_atomic_fetch_add(&a.ticket[u], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sm.is_last = (t == arrivals - 1) ? 1 : 0;
    if (t == arrivals - 1) store_agent(&a.ticket[u], 0);  // ready for the next launch
  }
  __syncthreads();
  if (!sm.is_last) return false;
  merge_splits<GT, NT, true>(a, u, sm.part);
  // every split of the unit has read its entries: blank them for the next launch
  if (a.sel_entry != nullptr)
    for (int i = tid; i < a.k; i += NT) store_agent(&a.sel_entry[(size_t)u * a.k + i], 0ull);
  return true;
}

// ---------------------------------------------------------------------------------------------
// MFMA attention
// ---------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <bool BF16>
__device__ __forceinline__ f32x4 mfma_qk(const uint4& kfrag, const uint4& qfrag, f32x4 c) {
  if (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kfrag), __builtin_bit_cast(bf16x8, qfrag), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kfrag), __builtin_bit_cast(f16x8, qfrag), c, 0, 0, 0);
}

// The same instruction for the P.V product of 16 tokens with P in two parts: c + v0 p0 + v1 p1.
template <bool BF16>
__device__ __forceinline__ f32x4 mfma_pv2(const uint2& v0, const uint2& v1, const uint2& p0, const uint2& p1, f32x4 c) {
  return mfma_qk<BF16>(make_uint4(v0.x, v0.y, v1.x, v1.y), make_uint4(p0.x, p0.y, p1.x, p1.y), c);
}

template <bool BF16>
__device__ __forceinline__ f32x4 mfma_pv(const uint2& vfrag, const uint2& pfrag, f32x4 c) {
  if (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vfrag), __builtin_bit_cast(s16x4, pfrag), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, vfrag), __builtin_bit_cast(f16x4, pfrag), c, 0, 0, 0);
}

// Workgroup (split, u) of NT threads takes split `split`, or (SEVERAL) a.take splits from there on, one after the other: wave w takes 16-token tiles w, w +
// NW, ... of each one's pages, without a pause between two splits, and leaves a partial of its own for each.  Per tile: 4 loads give the K operand (lane (i, g) = token i, dims
// 32c+8g..+7), 4 loads the V^T operands; S^T[token][head] = sum_c mfma(K_c, Q^T_c); the C tile of
// lane (j, g) holds head j, tokens 4g..4g+3, which is exactly the B operand of
// O^T[dim][head] += V^T[dim][token] P^T[token][head].  Heads sit in the 16 MFMA columns; columns
// >= G carry zeros and are never read.  For bf16 the probabilities are split into a high and a
// low bf16 part (two MFMAs) so that P keeps 16 bits of mantissa; fp16 P has 11 bits and needs one.
// HANDOFF: the selection was written by another workgroup of the same launch.
// LAYOUT kLayoutPacked: pages of 4 or 8 tokens in the packed slot layout: a tile is made of 16 / P consecutive
// entries of the split, every lane fetching its 16-byte units from the slot of its own page, and
// every token of the tile is valid or not on its own (a page beyond the selection's end, a made-up
// page, the ragged last page of a sequence).
// LAYOUT kLayoutNatural: pages of any other size, K and V rows as the host has them.  A tile is 16
// consecutive tokens of the split's pages put one after the other, whichever pages they lie in.  What the
// other layouts prepare in the slot is had here by the choice of rows: row i of the K operand is token
// 4 (i % 4) + i / 4 of the tile, so that lane (j, g) of the C tile holds the logits of tokens g, 4 + g, 8 + g
// and 12 + g; lane (i, g) fetches 16 bytes of the V rows of the same four tokens, eight dims of each, and the
// halves of dim 8i + e, put together in pairs, are its V^T operand of the e-th MFMA (16 byte permutes a
// tile, no LDS), whose C tile then holds dims 8 (4g + 0..3) + e.  P keeps all its 24 bits: in three 16-bit parts where
// these hold them (bf16 above 2^-100; fp16 parts of 2^15 P above 2^-15, so that the third ends at fp16's smallest
// number), and in fp32 MFMAs (16x16x4, four times the cycles) for a tile that has a smaller one.  (us per step, three
// parts and fp32 throughout: 32 units x 85 pages of 24 tokens, G = 7, fp16 31.2 and 32.1; 32 units x 102 pages of
// 20 tokens, bf16 26.5 and 28.3.  With two fp16 parts the first was 30.6; in fp32 VALU arithmetic 50.6 and 36.5.
// Of the shapes measured that was faster only with one query head to a KV head, for small ones above all: 4 units x 14
// pages of 40 tokens 17.5 and 18.4, 16 x 26 of 20 19.4 and 20.3, 8 x 170 of 12 22.2 and 22.7, 64 x 102 of 20 30.7 and 31.4,
// but 256 x 51 of 20 44.9 and 41.0.)
// Returns 1 in the workgroup that completed the unit's output, 0 in the others, -1 (from all
// threads, no output) when a HANDOFF wait ran out.  inputs_ready_tick (one thread passes it)
// receives the wall clock at which the split's entries were all there.
template <bool BF16, int GT, int NT, bool HANDOFF, int LAYOUT = kLayoutTiles, bool SEVERAL = false, class Smem>
__device__ __forceinline__ int attend_mfma_body(const AttnArgs& a, Smem& sm, int u, int split, long long* inputs_ready_tick = nullptr) {
  constexpr int NW = NT / kWave;
  constexpr bool PACKED = LAYOUT == kLayoutPacked, NATURAL = LAYOUT == kLayoutNatural;
  constexpr float kPScale = NATURAL && !BF16 ? 32768.f : 1.f;   // of the probabilities that multiply V
  const int G = group_size<GT>(a);
  const int b = u / a.Hkv, h = u % a.Hkv;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  const int j = lane & 15, g = lane >> 4;

  // Q^T operand: lane (j, g) holds Q[head j][32c + 8g .. +7] for c = 0..3 (zeros for j >= G)
  uint4 qfrag[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) qfrag[c] = make_uint4(0u, 0u, 0u, 0u);
  if (j < G) {
    const uint16_t* qrow = a.q + ((size_t)b * a.Hq + (size_t)h * G + j) * kHeadDim + 8 * g;
#pragma unroll
    for (int c = 0; c < 4; ++c) qfrag[c] = *reinterpret_cast<const uint4*>(qrow + 32 * c);
  }

  f32x4 o[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;

  const int seq = a.seq_len[b];
  const int tiles_per_page = a.P >> 4;                  // (PACKED: 0; pages_per_tile counts instead)
  const int pages_per_tile = PACKED ? 16 / a.P : 1;
  // splits [split, split + n_splits), whose entries are [first, last)
  const int n_splits = !SEVERAL ? 1 : split + a.take < a.S ? a.take : a.S - split;
  const int first = split * a.per_split;
  const int last = (split + n_splits) * a.per_split < a.k ? (split + n_splits) * a.per_split : a.k;
  auto tiles_of = [&](int v) -> int {                  // of the v-th of them
    const int n = last - first - v * a.per_split < a.per_split ? last - first - v * a.per_split : a.per_split;
    return PACKED ? (n + pages_per_tile - 1) / pages_per_tile : NATURAL ? (n * a.P + 15) >> 4 : n * tiles_per_page;
  };
  // T / P for a token of the split (below 2^20): the product with the reciprocal rounded up, off by less than T P / 2^32
  const u32 recip = NATURAL ? 0xffffffffu / (u32)a.P + 1u : 0u;   // (P = 1: 2^32 wraps to 0, handled below)
  const int32_t* sel = a.sel_pages + (size_t)u * a.k;
  const int32_t* slots = a.sel_slots + (size_t)u * a.k;
  const char* pool_u = a.pool + (size_t)u * a.Cmax * a.page_bytes;

  // the split's (page, slot) entries go to LDS once, so that issuing a tile's loads never waits on
  // a global index load.  HANDOFF: they come from the unit's selection workgroup of the same launch,
  // one 64-bit word each, and a thread polls its word until it has been published (a word is
  // published when the page is in its slot); the wait is bounded and its verdict shared.
  const int n_entries = last - first;
  // (HANDOFF callers keep splits within kAttnIdxCap, and over natural slots there is room for any)
  const bool idx_in_lds = HANDOFF || NATURAL || n_entries <= kAttnIdxCap;
  if (HANDOFF) {
    const u64* ent = a.sel_entry + (size_t)u * a.k + first;
    if (tid == 0) sm.is_last = 0;                      // (here: -1 once some thread's wait has run out)
    __syncthreads();
    int failed = 0;
    long long t0 = 0;
    for (int i = tid; i < n_entries && i < kAttnIdxCap; i += NT) {
      u64 v = load_agent(ent + i);
      while (!(v >> 63)) {
        if (t0 == 0) t0 = wall_clock64();
        __builtin_amdgcn_s_sleep(2);
        v = load_agent(ent + i);
        if (!(v >> 63) && wall_clock64() - t0 > a.wait_limit) { failed = 1; break; }
      }
      const int slot16 = (int)((v >> 32) & 0xffffu);
      sm.page[i] = (int32_t)(u32)v;
      sm.slot[i] = slot16 == 0xffff ? -1 : slot16;
    }
    if (failed) sm.is_last = -1;
    __syncthreads();
    if (sm.is_last < 0) return -1;
    if (inputs_ready_tick != nullptr) *inputs_ready_tick = wall_clock64();
  } else {
    if (idx_in_lds) {
      for (int i = tid; i < n_entries; i += NT) {
        sm.page[i] = sel[first + i];
        sm.slot[i] = slots[first + i];
      }
    }
    __syncthreads();
  }

  // software pipeline: three tile buffers rotate, so the operands of the next two tiles of this
  // wave (16 KiB) are in flight while one tile is computed
  struct Tile { uint4 k[4], v[4]; u32 valid; int split; };   // valid: bit i = token i of the tile takes part
  auto issue_tile = [&](Tile& tl, int split_v, int t, bool there = true) {   // (there: looked at over natural slots)
    // the split's entries in LDS, and behind `first`
    const int e_base = SEVERAL ? split_v * a.per_split : 0;
    const int e_end = SEVERAL && e_base + a.per_split < n_entries ? e_base + a.per_split : n_entries;
    tl.valid = 0;
    if (PACKED) {
      // lane (i, g): K units of token i of the tile = token i % P of entry i / P; V units of tokens
      // 4g..4g+3 = token group (4g % P) / 4 of entry 4g / P
      auto entry = [&](int e, int& page, int& slot) {
        page = -1; slot = -1;
        if (e < e_end) {
          if (idx_in_lds) { page = sm.page[e]; slot = sm.slot[e]; }
          else { page = sel[first + e]; slot = slots[first + e]; }
        }
        if (slot >= a.Cmax) slot = -1;
      };
      const int shift = a.P == 8 ? 3 : 2;               // (P is 4 or 8; a unit's slots span less than 4 GB)
      const int e0 = e_base + t * pages_per_tile;
      int kp, ks, vp, vs;
      entry(e0 + (j >> shift), kp, ks);
      entry(e0 + ((4 * g) >> shift), vp, vs);
      const int ktok = j & (a.P - 1);
      const bool kok = kp >= 0 && ks >= 0 && kp * a.P + ktok < seq;
      // the tile's valid tokens: lanes 0..15 (g = 0) speak for tokens 0..15
      const u32 valid = (u32)(__ballot(kok) & 0xffffull);
      tl.valid = valid;
      if (valid == 0) return;
#pragma unroll
      for (int c = 0; c < 4; ++c) { tl.k[c] = make_uint4(0u, 0u, 0u, 0u); tl.v[c] = make_uint4(0u, 0u, 0u, 0u); }
      if (kok) {
        const u32 kb = (u32)ks * a.page_bytes + (u32)(g * a.P + ktok) * 16u;
#pragma unroll
        for (int c = 0; c < 4; ++c) tl.k[c] = load_stream16(pool_u + (kb + (u32)(c * 64 * a.P)));
      }
      if (vp >= 0 && vs >= 0 && ((valid >> (4 * g)) & 15u)) {
        const u32 tg = (u32)((4 * g) & (a.P - 1)) >> 2;
        const u32 vb = (u32)vs * a.page_bytes + (u32)a.P * kRowBytes + (tg * 16u + (u32)j) * 16u;
#pragma unroll
        for (int c = 0; c < 4; ++c) tl.v[c] = load_stream16(pool_u + (vb + (u32)(c * 64 * a.P)));
      }
      return;
    }
    if constexpr (NATURAL) {
      // token d of the tile: row (16 t + d) % P of entry (16 t + d) / P.  Each lane looks up the token of its K row, and
      // learns where its V rows are from the lanes 4g .. 4g+3, which have looked up their tokens.  (us per step with five
      // lookups per lane and so: 160 units x 85 pages of 12 tokens, G = 2 and 7, 49.7, 52.0 and 37.5, 40.0; 40 x 300
      // pages of 6 34.8 and 31.4; 96 x 102 pages of 20 41.0 and 40.4; 16 x 26 pages of 20 20.0 and 20.3.  Ways of their own
      // for pages of more and of up to 16 tokens: the last gained nothing, large ones lost 10 % to the longer code.)
      // The loads have no branch around them, a token that is not there an address that is: where one path loads a register
      // and another does not, the compiler has all loads waited for before the next ones, and one tile is in flight instead of
      // three (32 units x 2084 pages of 24 tokens, G = 7, 24.3 us a step and 23.6 so).
      const int t_u = there ? __builtin_amdgcn_readfirstlane(t) : 0, end = there ? e_end : 0;
      const int e0_v = (int)((u32)(((u64)(16 * t_u) * recip) >> 32)) + (a.P == 1 ? 16 * t_u : 0), row0 = 16 * t_u - e0_v * a.P;
      const int e0 = e_base + e0_v;
      auto entry = [&](int e, int& page, int& slot) {
        const int at = e < end ? e : 0;
        page = sm.page[at];
        slot = sm.slot[at];
        slot = e >= end || slot >= a.Cmax ? -1 : slot;
        page = e >= end ? -1 : page;
      };
      int page, slot, row = row0 + 4 * (j & 3) + (j >> 2);
      if (a.P > 16) {                                    // the tile lies in entries e0 and e0 + 1
        int page1, slot1;
        entry(e0, page, slot);
        entry(e0 + 1, page1, slot1);
        page = __builtin_amdgcn_readfirstlane(page); slot = __builtin_amdgcn_readfirstlane(slot);
        page1 = __builtin_amdgcn_readfirstlane(page1); slot1 = __builtin_amdgcn_readfirstlane(slot1);
        const bool next = row >= a.P;
        row -= next ? a.P : 0;
        page = next ? page1 : page;
        slot = next ? slot1 : slot;
      } else {
        const int de = a.P == 1 ? row : (int)__umulhi((u32)row, recip);
        row -= de * a.P;
        entry(e0 + de, page, slot);
      }
      const bool kok = page >= 0 && slot >= 0 && page * a.P + row < seq;
      const u32 valid = (u32)(__ballot(kok) & 0xffffull);   // bit i: the token of row i takes part
      tl.valid = valid;
      const int krow = slot * 2 * a.P + row;             // of the unit's slots, in rows of 256 bytes (below 2^25)
      int vrow[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) vrow[m] = __shfl(krow, 4 * g + m, kWave) + a.P;
      // a token that takes no part reads the query's first row, which is there and in no slot (its logit is not used, and its V is blanked)
      const char* nowhere = reinterpret_cast<const char*>(a.q + ((size_t)b * a.Hq + (size_t)h * G) * kHeadDim);
      // (each 128-byte line is the business of two of the K loads: no streaming hint)
      const char* kb = (kok ? pool_u + (size_t)krow * kRowBytes : nowhere) + g * 16;
#pragma unroll
      for (int c = 0; c < 4; ++c) tl.k[c] = *reinterpret_cast<const uint4*>(kb + c * 64);
      const u32 mine = (valid >> (4 * g)) & 15u;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        tl.v[m] = load_stream16(((mine >> m) & 1u ? pool_u + (size_t)vrow[m] * kRowBytes : nowhere) + j * 16);
      return;
    }
    const int e = e_base + t / tiles_per_page, tile = t % tiles_per_page;
    int page, slot;
    if (idx_in_lds) {
      page = sm.page[e];
      slot = sm.slot[e];
    } else {
      page = sel[first + e];
      slot = slots[first + e];
    }
    page = __builtin_amdgcn_readfirstlane(page);
    slot = __builtin_amdgcn_readfirstlane(slot);
    if (page < 0 || slot < 0 || slot >= a.Cmax) return;
    int ntok = seq - page * a.P - tile * 16;
    ntok = ntok < 16 ? ntok : 16;
    if (ntok <= 0) return;
    tl.valid = ntok >= 16 ? 0xffffu : ((1u << ntok) - 1u);
    const uint4* tb = reinterpret_cast<const uint4*>(pool_u + (size_t)slot * a.page_bytes + (size_t)tile * kTileBytes) + lane;
#pragma unroll
    for (int c = 0; c < 4; ++c) tl.k[c] = load_stream16(tb + c * 64);
#pragma unroll
    for (int c = 0; c < 4; ++c) tl.v[c] = load_stream16(tb + 256 + c * 64);
  };
  // exact: P.V in fp32 whatever the probabilities
  auto compute = [&](Tile& tl, auto exact) {
    const u32 valid = tl.valid;
    if (!NATURAL && valid == 0) return;
    if (NATURAL && valid != 0xffffu) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!((valid >> (4 * g + e)) & 1u)) tl.v[e] = make_uint4(0u, 0u, 0u, 0u);
    }
    const u32 mine = (valid >> (4 * g)) & 15u;          // this lane's four tokens 4g..4g+3
    if (!NATURAL && valid != 0xffffu) {
      // a tile with tokens that take no part (the ragged end of a sequence, whose slot holds whatever
      // the store had there since a page is copied whole; with PACKED also a missing page): a
      // probability of zero does not silence a NaN or an infinity, so those tokens' V elements are
      // blanked.  Lane (., g) holds tokens 4g..4g+3 of a dim in each half of a V fragment, two
      // tokens per 32-bit word.
      const u32 m0 = ((mine & 1u) ? 0x0000ffffu : 0u) | ((mine & 2u) ? 0xffff0000u : 0u);
      const u32 m1 = ((mine & 4u) ? 0x0000ffffu : 0u) | ((mine & 8u) ? 0xffff0000u : 0u);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        tl.v[c].x &= m0; tl.v[c].y &= m1;
        tl.v[c].z &= m0; tl.v[c].w &= m1;
      }
    }
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (NATURAL) {
      // (four partial sums: an fp32 rounding at the size of the whole sum three times fewer)
      f32x4 part[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) part[c] = mfma_qk<BF16>(tl.k[c], qfrag[c], s);
      s = (part[0] + part[1]) + (part[2] + part[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) s = mfma_qk<BF16>(tl.k[c], qfrag[c], s);
    }
    float x[4];
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (NATURAL) s[e] = ((mine >> e) & 1u) ? s[e] : -INFINITY;
      x[e] = NATURAL || ((mine >> e) & 1u) ? s[e] * a.scale_log2 : -INFINITY;
      mx = fmaxf(mx, x[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    const float m_new = fmaxf(m, mx);
    const float ms = m_new == -INFINITY ? 0.f : m_new;   // (a head with no logit above minus infinity yet: no weight, no NaN)
    if (__any(m_new > m)) {
      const float alpha = exp2f(m - ms);
      l *= alpha;
#pragma unroll
      for (int c = 0; c < 8; ++c) o[c] *= alpha;
      m = m_new;
    }
    float p[4];
    const bool coarse = fabsf(ms) > 4194304.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // (natural layout: without the rounding of x, which is larger than that of the difference; but not for logits
      // beyond 2^22, where the rounding of their maximum would leave that token far from a probability of one)
      p[e] = exp2f(!NATURAL || coarse ? x[e] - ms : fmaf(s[e], a.scale_log2, -ms));
      l += p[e];
    }
    if constexpr (NATURAL) {
      u32 least = 0xffffffffu;                           // bits of the smallest probability that is not zero, less one
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u32 bits = __float_as_uint(p[e]) - 1u;
        least = least < bits ? least : bits;
        p[e] *= kPScale;
      }
      const u32* v0 = reinterpret_cast<const u32*>(&tl.v[0]);
      const u32* v1 = reinterpret_cast<const u32*>(&tl.v[1]);
      const u32* v2 = reinterpret_cast<const u32*>(&tl.v[2]);
      const u32* v3 = reinterpret_cast<const u32*>(&tl.v[3]);
      if (decltype(exact)::value || __any(least < __float_as_uint(BF16 ? 0x1p-100f : 0x1p-15f) - 1u)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const u32 word = (i == 0 ? v0 : i == 1 ? v1 : i == 2 ? v2 : v3)[e >> 1];
            const uint16_t h = (uint16_t)((e & 1) ? word >> 16 : word);
            const float ve = BF16 ? as_f32((u32)h << 16) : (float)__builtin_bit_cast(_Float16, h);
            sum = __builtin_amdgcn_mfma_f32_16x16x4f32(ve, p[i], sum, 0, 0, 0);
          }
          o[e] += sum;
        }
        return;
      }
      uint2 parts[3];
      typedef std::conditional_t<BF16, __bf16, _Float16> half_t;
      typedef half_t half4 __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const half4 part = {(half_t)p[0], (half_t)p[1], (half_t)p[2], (half_t)p[3]};
        parts[i] = __builtin_bit_cast(uint2, part);
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] -= (float)part[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const u32 pick = (e & 1) ? 0x07060302u : 0x05040100u;   // the high or the low halves of two words
        const uint2 v = make_uint2(__builtin_amdgcn_perm(v1[e >> 1], v0[e >> 1], pick), __builtin_amdgcn_perm(v3[e >> 1], v2[e >> 1], pick));
        o[e] = mfma_pv2<BF16>(v, v, parts[0], parts[1], o[e]);
        o[e] = mfma_pv2<BF16>(v, v, parts[2], make_uint2(0u, 0u), o[e]);
      }
    } else if (BF16) {
      const bf16x4 hi = {(__bf16)p[0], (__bf16)p[1], (__bf16)p[2], (__bf16)p[3]};
      const bf16x4 lo = {(__bf16)(p[0] - (float)hi[0]), (__bf16)(p[1] - (float)hi[1]), (__bf16)(p[2] - (float)hi[2]),
                         (__bf16)(p[3] - (float)hi[3])};
      const uint2 ph = __builtin_bit_cast(uint2, hi), pl = __builtin_bit_cast(uint2, lo);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint2 v0 = make_uint2(tl.v[c].x, tl.v[c].y), v1 = make_uint2(tl.v[c].z, tl.v[c].w);
        o[2 * c] = mfma_pv<true>(v0, ph, o[2 * c]);
        o[2 * c + 1] = mfma_pv<true>(v1, ph, o[2 * c + 1]);
        o[2 * c] = mfma_pv<true>(v0, pl, o[2 * c]);
        o[2 * c + 1] = mfma_pv<true>(v1, pl, o[2 * c + 1]);
      }
    } else {
      const f16x4 hp = {(_Float16)p[0], (_Float16)p[1], (_Float16)p[2], (_Float16)p[3]};
      const uint2 ph = __builtin_bit_cast(uint2, hp);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint2 v0 = make_uint2(tl.v[c].x, tl.v[c].y), v1 = make_uint2(tl.v[c].z, tl.v[c].w);
        o[2 * c] = mfma_pv<false>(v0, ph, o[2 * c]);
        o[2 * c + 1] = mfma_pv<false>(v1, ph, o[2 * c + 1]);
      }
    }
  };
  // what this wave has of the split is left for the epilogue
  auto leave = [&](int v) {
    // per-lane sums cover tokens 4g..4g+3 of every tile: add the four lane groups of a head
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    if (j < G) {
      // O^T C tiles: lane (j, g) register e of tile c holds dim 16c + 4g + e of head j (natural layout: 8 (4g + e) + c)
      float* p = sm.part_of(v, w, j, G);
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) p[NATURAL ? 8 * (4 * g + e) + c : 16 * c + 4 * g + e] = o[c][e] * (1.f / kPScale);
      if (g == 0) { p[kHeadDim] = m; p[kHeadDim + 1] = l; }
    }
  };
  auto start_over = [&]() {
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    m = -INFINITY; l = 0.f;
  };
  // the wave's tiles in order, split by split; ends with the accumulators of the last split
  auto run = [&](auto exact) {
    if constexpr (SEVERAL) {
      int iv = 0, it = w, n_it = tiles_of(0), cv = 0;    // the next tile to ask for; the split that the accumulators are of
      auto issue = [&](Tile& tl) {
        while (it >= n_it && iv < n_splits) {
          ++iv;
          it = w;
          n_it = iv < n_splits ? tiles_of(iv) : 0;
        }
        tl.split = iv;
        if (iv == n_splits) return;
        issue_tile(tl, iv, it);
        it += NW;
      };
      auto next = [&](Tile& tl) -> bool {                // false: there is no tile left
        while (cv < tl.split && cv < n_splits - 1) {
          leave(cv++);
          start_over();
        }
        if (tl.split == n_splits) return false;
        compute(tl, exact);
        return true;
      };
      Tile ta, tb2, tc;
      issue(ta);
      issue(tb2);
      for (;;) {
        issue(tc);
        if (!next(ta)) break;
        issue(ta);
        if (!next(tb2)) break;
        issue(tb2);
        if (!next(tc)) break;
      }
    } else {
      const int n_tiles = tiles_of(0);
      if constexpr (NATURAL) {
        auto issue = [&](Tile& tl, int t) { issue_tile(tl, 0, t, t < n_tiles); };
        // Behind a tile without a valid token a launch's own selection, which is in the pages' order, has padding only: the wave
        // is done.  (us per step of sequences with fewer pages than are selected, without and with it: 64 units, 50 of 300 pages of
        // 12 tokens 28.1 and 25.6, 16 x 150 of 1000 of 20 31.3 and 31.0; full selections 0 to 0.4 % slower.  The tiles counted to the
        // sequence's end beforehand instead 26.0 and 30.8, but 0.5 % slower where they are full, and 2 % in launches of 8 layers.)
        auto none = [&](const Tile& next, int t) { return t >= n_tiles || (HANDOFF && next.valid == 0); };
        if (w >= n_tiles) return;
        Tile ta, tb2, tc;
        issue(ta, w);
        // a tile to a wave, where the loads of two more that are not there cost their time (us per step with and without them:
        // 4 units x 500 pages of 40 tokens 15.1 and 14.3, 2 x 170 of 12 14.2 and 13.4, 16 x 1000 of 20 16.2 and 15.3)
        if (!decltype(exact)::value && n_tiles <= NW) {
          compute(ta, exact);
          return;
        }
        issue(tb2, w + NW);
        for (int t = w;; t += 3 * NW) {
          issue(tc, t + 2 * NW);
          compute(ta, exact);
          if (none(tb2, t + NW)) break;
          issue(ta, t + 3 * NW);
          compute(tb2, exact);
          if (none(tc, t + 2 * NW)) break;
          issue(tb2, t + 4 * NW);
          compute(tc, exact);
          if (none(ta, t + 3 * NW)) break;
        }
        return;
      }
      auto issue = [&](Tile& tl, int t) {
        tl.valid = 0;
        if (t < n_tiles) issue_tile(tl, 0, t);
      };
      Tile ta, tb2, tc;
      issue(ta, w);
      issue(tb2, w + NW);
      for (int t = w; t < n_tiles; t += 3 * NW) {
        issue(tc, t + 2 * NW);
        compute(ta, exact);
        issue(ta, t + 3 * NW);
        compute(tb2, exact);
        issue(tb2, t + 4 * NW);
        compute(tc, exact);
      }
    }
  };
  run(std::false_type());
  if constexpr (NATURAL) {
    // (here a workgroup takes one split.)  An infinity in V times a lower part of P, which may be zero or negative, is not the infinity that P times V
    // is.  Sums that are not finite are therefore formed again in fp32.
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) sum += (o[c][0] * 0.f + o[c][1] * 0.f) + (o[c][2] * 0.f + o[c][3] * 0.f);
    if (__any(sum != 0.f)) {                             // (0 x infinity and 0 x NaN are NaN)
      start_over();
      run(std::true_type());
    }
  }
  leave(n_splits - 1);
  return finish_splits<GT, NT, SEVERAL>(a, sm, u, split, n_splits) ? 1 : 0;
}

}  // namespace kvd
