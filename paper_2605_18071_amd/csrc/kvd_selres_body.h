// Selection, cache-directory update and fetch for one unit by one workgroup of NT threads:
// exact Top-K selection of the scored pages (Background: "retrieving only the Top-K"), the
// directory update for the same unit (Attention-Based Cache Management with LRU replacement),
// and the fetch of the unit's missed pages from the pinned host store (only out-of-cache entries
// move — Roofline section).  Shared by the stand-alone kernel and the single-launch layer-step
// kernel.
//
// Selection and victim choice are both "the n smallest of distinct 64-bit keys" problems: an LDS
// histogram over a monotone bucket function narrows the answer to
// one bucket, whose few members are ranked exactly.  The items stay in registers; only a bucket
// with more than 1024 members (degenerate inputs, e.g. all scores equal) falls back to radix
// refinement.  What bounds it is the chain of instructions and barriers that one workgroup goes through (cycles until the
// entries are out, 512 threads and up to 2048 pages: 11600 with block scans, a threshold handed around through LDS and
// one store at a time from the lanes that own the pages, 7400 to 9300 so), hence: each wave reads the whole histogram and
// finds the bucket for itself; a list is ranked only when the decisive bucket does not go in whole; what is selected goes to
// LDS at its place and out from there, by full waves.  (us per step before and after: 8 units x 256 pages 14.7 and 13.5, 4
// layers of 32 x 1001 pages 111.6 and 108.5, 20 x 335 pages 30.1 and 28.8.  The wait between scoring and selection is no
// matter of cold code: a rehearsal of the selection on the scores of the step before, while those of this step come in,
// made it no faster.)  The page -> slot map of the unit is rebuilt in LDS from the slot array at every
// launch, so a lookup never waits on a dependent global load; every global load the block needs
// is issued in its first instructions.
#pragma once
#include <type_traits>

#include "kvd_device.h"
#include "kvd_internal.h"
#include "kvd_page_copy.h"

namespace kvd {

struct NothingToDo { __device__ void operator()() const {} };

constexpr int kListCap = 1024;
constexpr uint16_t kAbsent = 0xffffu;

struct FastArgs {
  const float* scores;        // [U][NP]
  const int32_t* seq_len;     // [B]
  int32_t* sel_pages;         // [U][k]: written by the selection, read when only resolving
  const int32_t* capacity;    // [U] of the layer
  int32_t* resident;          // [U]
  int32_t* slot_page;         // [U][Cmax]
  int32_t* slot_stamp;        // [U][Cmax]
  int32_t* sel_slots;         // [U][k]
  u64* sel_entry;             // [U][k] or null: (valid, slot, page) entries for the attention workgroups of the same launch; zero between launches
  int32_t* hit_mask;          // [U][k]
  int32_t* evicted;           // [U][k]
  int32_t* counts;            // [U][3]
  int32_t* miss_list;         // [U][k][2]
  int32_t* miss_count;        // [U]
  unsigned long long* stats;  // hits, misses, evictions
  const char* store;          // host store of the layer, [U][NP] pages (device-visible address)
  char* pool;                 // slot pool of the layer, [U][Cmax] slots
  int NP, P, k, Cmax, sink, recent, Hkv, step, u0, do_gather, tiled;
  int lookahead;              // victims by lowest current-step score (needs `scores`) instead of by age
  int la_pool;                // look-ahead pool in pages (0 = every scored page): resident pages outside the step's la_pool
                              // best-scoring pages leave first, least recently selected first
  const int32_t* page_cluster;  // [U][NP] or null: the victims' scores are those of the pages' clusters
  int score_stride;           // scores of unit u start at scores + u * score_stride (NP, or the number of centroids)
  unsigned page_bytes;
  int shallow_fetch;          // many units fetch at the same time: each with less on its way
};

// What the attention workgroups of the same launch read instead of sel_pages / sel_slots: one
// 64-bit word per selected entry, bit 63 = published, bits 32..47 the slot (0xffff = none), the
// low word the page (-1 = padding).  A word is published once the page's bytes are in its slot.
__device__ __forceinline__ u64 pack_sel_entry(int page, int slot) {
  return (1ull << 63) | ((u64)((u32)slot & 0xffffu) << 32) | (u64)(u32)page;
}

// This step's score of a resident page as lookahead eviction sees it: the page's own score, or with
// the hierarchical index the score of its cluster (-inf for a page of no cluster: it leaves first).
template <bool HANDOFF>
__device__ __forceinline__ float victim_score(const FastArgs& a, int u, int page) {
  int at = page;
  if (a.page_cluster != nullptr) {
    at = a.page_cluster[(size_t)u * a.NP + page];
    if (at < 0) return -INFINITY;
  }
  const float* sc = a.scores + (size_t)u * a.score_stride + at;
  return HANDOFF ? load_agent(sc) : *sc;
}

// BIG: units of up to KVD_BIG_MAX_PAGES pages and KVD_BIG_MAX_CAPACITY slots; the map alone is 128 of the
// CU's 160 KiB, and page numbers no longer leave a 16-bit value free for "none".
template <int NT, bool BIG = false>
struct FastSmem {
  static constexpr int NW = NT / kWave;
  static constexpr int kMaxPages = BIG ? KVD_BIG_MAX_PAGES : KVD_FAST_MAX_PAGES;
  static constexpr int kMaxCapacity = BIG ? KVD_BIG_MAX_CAPACITY : KVD_FAST_MAX_CAPACITY;
  typedef std::conditional_t<BIG, u32, uint16_t> page_t;
  static constexpr page_t kNoPage = (page_t)~(page_t)0;
  union {
    struct {
      u32 hist[kRadixBins];
      u64 cand[kListCap];
    } sel;
    uint16_t vt[NW][4 * kHeadDim];                       // V of the four tokens that a wave turns around during the fetch
  } a;
  uint16_t p2s[kMaxPages];                               // page -> slot of this unit, kAbsent = not resident
  union {
    page_t sel[KVD_MAX_TOPK + (BIG ? 0 : kWave)];        // selected pages (kNoPage = padding)
    u32 miss[KVD_MAX_TOPK];                              // then: page (low half) and entry of the selection of the i-th miss
    static_assert(BIG || sizeof(page_t) * (KVD_MAX_TOPK + kWave) <= sizeof(u32) * KVD_MAX_TOPK, "room behind sel for what is not selected");
  };
  uint16_t assign[KVD_MAX_TOPK];                         // slot handed to the i-th miss
  u32 hit_bitmap[kMaxCapacity / 32];
  int scan[2][NW];
  float2 red[NW];                                        // extremes over the waves
  int red_cnt[NW];
  u64 thr;
  int cand_n, tied_n, bin, below, n_ev, late;
  SelectSmem generic;
};

__device__ __forceinline__ u32 fast_descending_key(float s) {
  const u32 x = as_u32(s + 0.0f);                    // -0 -> +0 so that the two zeros tie
  const u32 asc = (x & 0x80000000u) ? ~x : (x | 0x80000000u);
  return ~asc;
}
// Key of the selection order (best page first); it also decides membership of the look-ahead pool.
__device__ __forceinline__ u64 selection_order_key(float s, int page) {
  return ((u64)fast_descending_key(s) << 32) | (u32)page;
}

// Exclusive prefix sum over the block with one barrier: the wave totals alternate between two
// LDS rows (`flip` is the caller's per-thread call counter), so a call never overwrites totals
// that slower waves may still be reading from the call before.
template <int NT, bool BIG>
__device__ __forceinline__ int fast_scan(int v, FastSmem<NT, BIG>& sm, int& flip, int& total) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int inc = wave_inclusive_scan(v);
  int* row = sm.scan[flip & 1];
  ++flip;
  if (lane == kWave - 1) row[w] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int t = row[i];
    base += i < w ? t : 0;
    tot += t;
  }
  total = tot;
  return base + inc - v;
}

// The histogram is filled (no barrier since): sm.bin = the bucket that holds the need-th smallest
// item, sm.below = the items in the buckets before it.  Ends with the block synchronised.
template <int NT, bool BIG>
__device__ __forceinline__ void find_bucket(int need, FastSmem<NT, BIG>& sm, int& flip) {
  const int tid = threadIdx.x;
  u32* hist = sm.a.sel.hist;
  __syncthreads();
  constexpr int BPT = kRadixBins / NT;
  int local = 0;
#pragma unroll
  for (int j = 0; j < BPT; ++j) local += (int)hist[tid * BPT + j];
  int total;
  int ex = fast_scan<NT>(local, sm, flip, total);
  if (ex < need && need <= ex + local) {             // exactly one thread
    int b = tid * BPT;
    for (int j = 0; j < BPT; ++j, ++b) {
      const int c = (int)hist[b];
      if (need <= ex + c) break;
      ex += c;
    }
    sm.bin = b;
    sm.below = ex;
  }
  __syncthreads();
}

// A histogram of 128 * W buckets, two 16-bit counts to a word (of at most 32768 items): lane l
// of a wave reads the 2 W buckets from 2 W l on with W / 4 16-byte loads without bank conflicts.
template <int W>
__device__ __forceinline__ int packed_bin_word(int bucket) {
  const int l = bucket / (2 * W), word = (bucket >> 1) & (W - 1);
  return (((word >> 2) * kWave + l) << 2) | (word & 3);
}
template <int W>
__device__ __forceinline__ void packed_bin_add(u32* hist, int bucket, u32 n = 1u) {
  atomicAdd(&hist[packed_bin_word<W>(bucket)], n << (16 * (bucket & 1)));
}
// The bucket that holds the need-th smallest item, the items before it and those in it, the same in every lane.  Each
// wave finds out for itself: no barrier and nothing handed around.  The histogram is complete (a barrier before).
template <int W>
__device__ __forceinline__ void packed_bin_find(const u32* hist, int need, int& bin, int& below, int& count) {
  const int lane = threadIdx.x & (kWave - 1);
  u32 sum = 0;
#pragma unroll
  for (int i = 0; i < W / 4; ++i) {
    const uint4 v = reinterpret_cast<const uint4*>(hist)[i * kWave + lane];
    sum += (v.x + v.y) + (v.z + v.w);                   // (both halves at once: no half of the total reaches 2^16)
  }
  const int local = (int)((sum & 0xffffu) + (sum >> 16));
  const int inc = wave_inclusive_scan(local);
  const u64 reached = __ballot(inc >= need);
  const int l = reached ? __ffsll((unsigned long long)reached) - 1 : kWave - 1;
  const int before = __builtin_amdgcn_readlane(inc - local, l);
  // lane j < 2 W: the j-th bucket of lane l
  const int b = 2 * W * l + (lane & (2 * W - 1));
  const u32 word = hist[packed_bin_word<W>(b)];
  const int c = lane < 2 * W ? (int)((lane & 1) ? word >> 16 : word & 0xffffu) : 0;
  const int cum = before + wave_inclusive_scan(c);
  const u64 at = __ballot(cum >= need);
  const int j = at ? __ffsll((unsigned long long)at) - 1 : 0;
  bin = 2 * W * l + j;
  count = __builtin_amdgcn_readlane(c, j);
  below = __builtin_amdgcn_readlane(cum, j) - count;
}

// The r-th smallest of the m <= 64 keys in the list, which is complete; each wave finds it for itself.
__device__ __forceinline__ u64 kth_of_list(const u64* list, int m, int r) {
  const int lane = threadIdx.x & (kWave - 1);
  const u64 mine = lane < m ? list[lane] : ~0ull;
  auto key_of_lane = [&](int x) -> u64 {
    return ((u64)(u32)__builtin_amdgcn_readlane((int)(mine >> 32), x) << 32) | (u32)__builtin_amdgcn_readlane((int)(u32)mine, x);
  };
  int rank = 0;
  for (int x = 0; x < m; ++x) rank += key_of_lane(x) < mine ? 1 : 0;
  const u64 at = __ballot(lane < m && rank == r - 1);
  return key_of_lane(__ffsll((unsigned long long)at) - 1);   // (1 <= r <= m: there is one)
}

// The r-th smallest of the m candidates in the list (no barrier since they were put there).
template <int NT, bool BIG>
__device__ __forceinline__ u64 rank_candidates(int m, int r, FastSmem<NT, BIG>& sm) {
  __syncthreads();
  for (int c = threadIdx.x; c < m; c += NT) {
    const u64 mine = sm.a.sel.cand[c];
    int rank = 0;
    for (int x = 0; x < m; ++x) rank += sm.a.sel.cand[x] < mine ? 1 : 0;
    if (rank == r - 1) sm.thr = mine;
  }
  __syncthreads();
  return sm.thr;
}

// Items j = 0..n_items-1 (at most IPT) of every thread: bkt(j) in [0, 2047], or -1 for "not a candidate"; key(j)
// distinct; key1 < key2 implies bkt1 <= bkt2.  sm.a.sel.hist must be zero and sm.cand_n zero on
// entry (with a barrier since).  Returns the need-th smallest key among the candidates
// (1 <= need <= number of candidates).  `refine(bin, r)` is called by all threads when the
// decisive bucket holds more than kListCap items and must return the r-th smallest key of that
// bucket.  Other waves may still be reading the list on return: a barrier comes before sm.a is written again.
template <int NT, int IPT, bool BIG, class KeyOf, class BktOf, class Refine>
__device__ __forceinline__ u64 two_level_select(KeyOf key, BktOf bkt, int n_items, int need, FastSmem<NT, BIG>& sm, int& flip,
                                                Refine refine) {
  constexpr int UNROLL = BIG ? 1 : IPT;               // (BIG: the items are read again from memory, not held in registers)
  int held[BIG ? 1 : IPT];                             // every item's bucket
#pragma unroll UNROLL
  for (int j = 0; j < IPT; ++j) {
    if (j >= n_items) break;
    const int bj = bkt(j);
    if (!BIG) held[j] = bj;
    if (bj < 0) continue;
    if (BIG) atomicAdd(&sm.a.sel.hist[bj], 1u);
    else packed_bin_add<16>(sm.a.sel.hist, bj);
  }
  int bin, below, m;
  if (BIG) {
    find_bucket<NT>(need, sm, flip);
    bin = sm.bin; below = sm.below; m = (int)sm.a.sel.hist[bin];
  } else {
    __syncthreads();
    packed_bin_find<16>(sm.a.sel.hist, need, bin, below, m);
  }
  const int r = need - below;
  if (m > kListCap) return refine(bin, r);
#pragma unroll UNROLL
  for (int j = 0; j < IPT; ++j) {
    if (j >= n_items) break;
    if ((BIG ? bkt(j) : held[j]) == bin) sm.a.sel.cand[atomicAdd(&sm.cand_n, 1)] = key(j);
  }
  if (m <= kWave / 2) {
    __syncthreads();
    return kth_of_list(sm.a.sel.cand, m, r);
  }
  return rank_candidates<NT>(m, r, sm);
}

// Victim key of lookahead eviction: ascending in (score, -page), so that the lowest score leaves
// first and, among equal scores, the higher page.
__device__ __forceinline__ u64 lookahead_victim_key(float s, int page) {
  const u32 x = as_u32(s + 0.0f);
  const u32 asc = (x & 0x80000000u) ? ~x : (x | 0x80000000u);
  return ((u64)asc << 32) | (u32)(~(u32)page);
}

// With a finite look-ahead pool the victim order is: pages outside the pool by (stamp, page), then
// pool pages by (score, -page).  One 64-bit key carries both (pages are below 2^24): bit 63 = in
// the pool, then the 32-bit stamp or score key, then the page or its complement.
__device__ __forceinline__ u64 pooled_victim_key(bool in_pool, float s, int stamp, int page) {
  if (!in_pool) return ((u64)((u32)stamp ^ 0x80000000u) << 24) | (u64)((u32)page & 0xffffffu);
  const u32 x = as_u32(s + 0.0f);
  const u32 asc = (x & 0x80000000u) ? ~x : (x | 0x80000000u);
  return (1ull << 63) | ((u64)asc << 24) | (u64)((~(u32)page) & 0xffffffu);
}
// page_scale: 32 / NP.  (A 64-bit division here, twice for each of a thread's eight slots, took 4 of the 6.2 us that the victim
// choice of a unit of 750 pages and 340 slots took.)
__device__ __forceinline__ int victim_bucket(int step, int stamp, int page, float page_scale) {
  // one group of 32 buckets per age (step - stamp) below 64, split by page range; everything older
  // shares bucket 0; the newest class (age <= 1) shares bucket 2047
  const long long age = (long long)step - (long long)stamp;
  const int in_class = (int)fminf((float)page * page_scale, 31.f);   // (monotone in the page)
  const int a = age >= 64 ? 64 : (int)(age <= 1 ? 1 : age);
  return a >= 64 ? 0 : a <= 1 ? 2047 : 2048 - 32 * a + in_class;
}

// Top-K selection of a unit of more pages than the ordinary form holds (see select_resolve_body for
// the rules).  Three passes over the scores: for the extremes, for the histogram, and for which pages
// lie before the decisive bucket and which in it.  HELD: at most 8 quads per lane (NP <= 32 NT), read once, 16
// bytes per lane, and kept in registers; with more pages every pass reads them, the later ones from the L2 (32 units
// of 32768 pages: 86.0 us a step with three reads, 84.6 with one).  A wave owns 256 * nq consecutive pages, of which a lane holds
// two 64-bit masks.  One workgroup per unit, so the passes are bound by what one CU reads from its L2 and
// by instruction issue.  32 units of 32768 pages and 8192 slots:
// selection, directory update and fetch of an all-hit step 23 us, against 115 us as the size-agnostic kernels,
// which refine their keys over global memory pass by pass (select 90, resolve 20, fetch 5).
template <int NT, bool HELD>
__device__ __forceinline__ void select_big(const FastArgs& a, int u, int seq, FastSmem<NT, true>& sm, int& flip) {
  constexpr int NW = NT / kWave;
  static_assert(KVD_BIG_MAX_PAGES <= NT * 64, "one mask bit per page of a lane");
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave, k = a.k;
  int n_valid = (seq + a.P - 1) / a.P;
  n_valid = n_valid < a.NP ? n_valid : a.NP;
  const int k_eff = k < n_valid ? k : n_valid;
  const int recent_from = n_valid - a.recent;
  const float* sc = a.scores + (size_t)u * a.NP;
  const int nq = (n_valid + 4 * NT - 1) / (4 * NT);
  const int wave_p0 = w * (4 * kWave) * nq;
  const bool vec = (a.NP & 3) == 0;
  auto quad = [&](int q, float (&s)[4]) {              // this lane's q-th four pages
    const int p = wave_p0 + q * (4 * kWave) + 4 * lane;
    if (vec) {                                         // (NP a multiple of 4: the four pages are all there or none)
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < a.NP) v = *reinterpret_cast<const float4*>(sc + p);
      s[0] = v.x; s[1] = v.y; s[2] = v.z; s[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = p + e < a.NP ? sc[p + e] : 0.f;
    }
  };
  auto upto = [&](int q, int bound) -> u32 {           // bits of the q-th four pages below `bound`
    const int n = bound - (wave_p0 + q * (4 * kWave) + 4 * lane);
    return (1u << (n < 0 ? 0 : (n > 4 ? 4 : n))) - 1u;
  };
  auto free_of = [&](int q) -> u32 { return upto(q, recent_from) & ~upto(q, a.sink); };
  float held[HELD ? 8 : 1][4];
  if constexpr (HELD) {
#pragma unroll
    for (int q = 0; q < 8; ++q) quad(q < nq ? q : 0, held[q]);
  }
  // calls f(q, scores, free bits) for this lane's pages, four quads' loads in flight
  auto for_quads = [&](auto f) {
    if constexpr (HELD) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q < nq) f(q, held[q], free_of(q));
      return;
    }
    for (int q0 = 0; q0 < nq; q0 += 4) {
      float s[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) quad(q0 + i < nq ? q0 + i : q0, s[i]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (q0 + i < nq) f(q0 + i, s[i], free_of(q0 + i));
    }
  };
  u64 take = 0;                                        // bit 4q + e: the q-th four pages' e-th is selected
  float fmin = INFINITY, fmax = -INFINITY;
  int n_forced = 0;
  for_quads([&](int q, const float (&s)[4], u32 fr) {
    const u32 forced = upto(q, n_valid) & ~fr;
    take |= (u64)forced << (4 * q);
    n_forced += __popc(forced);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      fmin = fminf(fmin, (fr >> e) & 1u ? s[e] : INFINITY);
      fmax = fmaxf(fmax, (fr >> e) & 1u ? s[e] : -INFINITY);
    }
  });
  fmin = wave_allreduce_min(fmin);
  fmax = wave_allreduce_max(fmax);
  n_forced = wave_inclusive_scan(n_forced);
  if (lane == kWave - 1) { sm.red[w] = make_float2(fmin, fmax); sm.red_cnt[w] = n_forced; }
  __syncthreads();
  n_forced = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    fmin = fminf(fmin, sm.red[i].x);
    fmax = fmaxf(fmax, sm.red[i].y);
    n_forced += sm.red_cnt[i];
  }
  const int k_free = k_eff - n_forced;
  if (k_free > 0) {
    const float range = fmax - fmin;
    const float inv = range > 0.f ? 2047.0f / range : 0.f;
    auto bucket_of = [&](float v) -> int { return (int)fminf(fmaxf((fmax - v) * inv, 0.f), 2047.f); };
    for_quads([&](int, const float (&s)[4], u32 fr) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((fr >> e) & 1u) atomicAdd(&sm.a.sel.hist[bucket_of(s[e])], 1u);
    });
    find_bucket<NT>(k_free, sm, flip);
    const int bin = sm.bin, r = k_free - sm.below, m = (int)sm.a.sel.hist[bin];
    const bool listed = m <= kListCap;
    u64 tied = 0;                                      // pages of the decisive bucket
    for_quads([&](int q, const float (&s)[4], u32 fr) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!((fr >> e) & 1u)) continue;
        const int b = bucket_of(s[e]);
        if (b < bin) take |= 1ull << (4 * q + e);
        if (b == bin) {
          tied |= 1ull << (4 * q + e);
          if (listed) sm.a.sel.cand[atomicAdd(&sm.cand_n, 1)] = selection_order_key(s[e], wave_p0 + q * (4 * kWave) + 4 * lane + e);
        }
      }
    });
    u64 thr;
    if (listed) {
      thr = rank_candidates<NT>(m, r, sm);
    } else {
      auto fn = [&](int i, u64& kk) -> bool {
        if (i < a.sink || i >= recent_from) return false;
        const float v = sc[i];
        if (bucket_of(v) != bin) return false;
        kk = selection_order_key(v, i);
        return true;
      };
      thr = block_kth_smallest<NT>(fn, n_valid, r, sm.generic, sm.a.sel.hist);
    }
    while (tied) {
      const int bit = __ffsll((unsigned long long)tied) - 1;
      tied &= tied - 1;
      const int p = wave_p0 + (bit >> 2) * (4 * kWave) + 4 * lane + (bit & 3);
      if (selection_order_key(sc[p], p) <= thr) take |= 1ull << bit;
    }
  }
  // output in ascending page order = (wave, quad, lane, element)
  int total;
  const int lane_pos = fast_scan<NT>((int)__popcll(take), sm, flip, total);
  int pos_q = __builtin_amdgcn_readfirstlane(lane_pos);
  int32_t* out = a.sel_pages + (size_t)u * k;
  for (int q = 0; q < nq; ++q) {
    u32 bits = (u32)(take >> (4 * q)) & 15u;
    const int cnt = __popc(bits), inc = wave_inclusive_scan(cnt);
    int pos = pos_q + inc - cnt;
    pos_q += __builtin_amdgcn_readlane(inc, kWave - 1);
    while (bits) {
      const int p = wave_p0 + q * (4 * kWave) + 4 * lane + __ffs((int)bits) - 1;
      bits &= bits - 1;
      if (pos < k) { sm.sel[pos] = (u32)p; out[pos] = p; }
      ++pos;
    }
  }
  for (int i = k_eff + tid; i < k; i += NT) {
    sm.sel[i] = FastSmem<NT, true>::kNoPage;
    out[i] = -1;
  }
}

// The same for units whose scores the registers hold (NP <= 32 NT), by quads of four consecutive pages: as many quads as pages
// are wanted have their best page at or before some bucket, so that the decisive bucket is no later; the quads that reach it,
// hardly more than pages are wanted, are listed and dealt out to the threads again, and only their pages are counted, compared and
// ranked.  Bound by instruction issue (16 waves on one CU: 100 instructions a thread are 0.7 us), of which the three passes of
// select_big need about 30 a page and this 3 a page and 20 a quad.  The selected pages are written from a map with four bits to
// a quad's byte, 32 pages a thread, in one block scan instead of a wave scan per load.  Where more quads than the list holds reach
// the bucket (many pages alike) the threads go through them where they are, in the registers.  (us per step, 8 units of 30000 pages of
// 4 tokens, k = 500, with select_big and so: 1200 pages alike 65.5 and 60.4, 2500 67.8 and 66.5, 9000 74.5 and 71.3, half
// of them 77.8 and 73.7 (83.7 with the pages of the last bucket counted one by one), all 100.0 and 79.3, none 38.6 and 35.1.)
template <int NT>
__device__ __forceinline__ void select_held_load(const FastArgs& a, int u, int seq, float4 (&s)[8]) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  int n_valid = (seq + a.P - 1) / a.P;
  n_valid = n_valid < a.NP ? n_valid : a.NP;
  const float* sc = a.scores + (size_t)u * a.NP;
  const int nq = (n_valid + 4 * NT - 1) / (4 * NT);
  const int p0 = w * (4 * kWave) * nq + 4 * lane;
  if ((a.NP & 3) == 0) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(sc), 0, a.NP * 4, 0x00020000);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, q < nq ? (p0 + q * (4 * kWave)) * 4 : 0, 0, 0);
      s[q] = make_float4(as_f32(v.x), as_f32(v.y), as_f32(v.z), as_f32(v.w));
    }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = p0 + q * (4 * kWave) + e;
        x[e] = sc[q < nq && p < a.NP ? p : a.NP - 1];
      }
      s[q] = make_float4(x[0], x[1], x[2], x[3]);
    }
  }
}
template <int NT>
__device__ __forceinline__ void select_held(const FastArgs& a, int u, int seq, const float4 (&s)[8], FastSmem<NT, true>& sm, int& flip) {
  typedef FastSmem<NT, true> Smem;
  constexpr int NW = NT / kWave, Q = 8, kQuads = 2 * NT;   // quads of a lane, quads of the list
  constexpr int kHeldPages = 4 * Q * NT;
  // the upper half of the page -> slot map is not in use: the list and the map of the selection
  struct Lists { float4 score[kQuads]; int quad[kQuads]; unsigned char picked[kHeldPages / 4]; };
  static_assert(sizeof(Lists) <= sizeof(uint16_t) * (Smem::kMaxPages - kHeldPages), "room behind the map of this many pages");
  Lists& ls = *reinterpret_cast<Lists*>(sm.p2s + kHeldPages);
  u32* hist_quads = sm.a.sel.hist;
  u32* hist_pages = sm.a.sel.hist + kRadixBins / 2;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave, k = a.k;
  int n_valid = (seq + a.P - 1) / a.P;
  n_valid = n_valid < a.NP ? n_valid : a.NP;
  const int k_eff = k < n_valid ? k : n_valid;
  const int recent_from = n_valid - a.recent;
  const int n_free = recent_from > a.sink ? recent_from - a.sink : 0;
  const int k_free = k_eff - (n_valid - n_free);
  const int free_quads = n_free > 0 ? (recent_from + 3) / 4 - a.sink / 4 : 0;   // with a free page
  const float* sc = a.scores + (size_t)u * a.NP;
  const int nq = (n_valid + 4 * NT - 1) / (4 * NT);
  const int wave_p0 = w * (4 * kWave) * nq;
  // bits of the four pages from p on below `bound`
  auto upto = [&](int p, int bound) -> u32 {
    const int n = bound - p;
    return (1u << (n < 0 ? 0 : (n > 4 ? 4 : n))) - 1u;
  };
  auto free_of = [&](int p) -> u32 { return upto(p, recent_from) & ~upto(p, a.sink); };
  auto page_of = [&](int q) -> int { return wave_p0 + q * (4 * kWave) + 4 * lane; };
  float best[Q], fmin = INFINITY, fmax = -INFINITY;
  u32 first = 0;                                         // bit q: in the first bucket
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u32 fr = q < nq ? free_of(page_of(q)) : 0u;
    const float x0 = fr & 1u ? s[q].x : -INFINITY, x1 = fr & 2u ? s[q].y : -INFINITY, x2 = fr & 4u ? s[q].z : -INFINITY,
                x3 = fr & 8u ? s[q].w : -INFINITY;
    best[q] = fmaxf(fmaxf(x0, x1), fmaxf(x2, x3));
    fmax = fmaxf(fmax, best[q]);
    fmin = fminf(fmin, best[q] > -INFINITY ? best[q] : INFINITY);
    // (a page that is no number is in the first bucket, and so is its quad.  The pages are looked at one by one: a sum of theirs may
    // be none where all are numbers, as of pairs that overflow to the two infinities, and a quad in an earlier bucket than any
    // of its pages would leave fewer pages than are wanted in the list)
    first |= __builtin_isunordered(x0, x1) || __builtin_isunordered(x2, x3) ? 1u << q : 0u;
    if (q < nq) ls.picked[page_of(q) >> 2] = (unsigned char)(upto(page_of(q), n_valid) & ~fr);   // the forced pages
  }
  fmin = wave_allreduce_min(fmin);
  fmax = wave_allreduce_max(fmax);
  if (lane == 0) sm.red[w] = make_float2(fmin, fmax);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    fmin = fminf(fmin, sm.red[i].x);
    fmax = fmaxf(fmax, sm.red[i].y);
  }
  if (k_free > 0) {
    const float range = fmax - fmin;
    const float inv = range > 0.f ? 2047.0f / range : 0.f;
    auto bucket_of = [&](float v) -> int { return (int)fminf(fmaxf((fmax - v) * inv, 0.f), 2047.f); };
    const bool one_bucket = inv == 0.f;                  // (one score for all, or infinities: nothing to count)
    int bk[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      bk[q] = q < nq && free_of(page_of(q)) ? ((first >> q) & 1u ? 0 : bucket_of(best[q])) : 2048;
      if (bk[q] < 2048 && !one_bucket) packed_bin_add<16>(hist_quads, bk[q]);
    }
    __syncthreads();
    int last = 2047, n_listed = free_quads;              // the quads up to bucket `last` are listed
    if (k_free <= free_quads && !one_bucket) {
      int before, in_last;
      packed_bin_find<16>(hist_quads, k_free, last, before, in_last);
      n_listed = before + in_last;
    }
    int bin, r;
    u64 thr = ~0ull;
    // the pages up to bucket `last` are counted: the decisive bucket, and which of its pages are in; found() is told that `bin` is
    // known, put_tied() puts the keys of this thread's pages there into the list
    auto decide = [&](auto put_tied, auto found) {
      __syncthreads();
      int below, m;
      bin = 0; below = 0; m = n_free;
      if (!one_bucket) packed_bin_find<16>(hist_pages, k_free, bin, below, m);
      r = k_free - below;                                // of the m pages of the decisive bucket r are in
      found();
      if (r == m) return;
      if (m <= kListCap) {
        put_tied();
        if (m <= kWave / 2) {
          __syncthreads();
          thr = kth_of_list(sm.a.sel.cand, m, r);
        } else {
          thr = rank_candidates<NT>(m, r, sm);
        }
      } else {
        auto fn = [&](int i, u64& kk) -> bool {
          if (i < a.sink || i >= recent_from) return false;
          const float x = sc[i];
          if (bucket_of(x) != bin) return false;
          kk = selection_order_key(x, i);
          return true;
        };
        thr = block_kth_smallest<NT>(fn, n_valid, r, sm.generic, sm.a.sel.hist);
      }
    };
    if (n_listed <= kQuads) {
      int mine = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) mine += bk[q] <= last ? 1 : 0;
      const int inc = wave_inclusive_scan(mine);
      int at = 0;
      if (lane == kWave - 1) at = atomicAdd(&sm.cand_n, inc);
      at = __builtin_amdgcn_readlane(at, kWave - 1) + inc - mine;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (bk[q] <= last) {
          ls.score[at] = s[q];
          ls.quad[at++] = page_of(q) >> 2;
        }
      __syncthreads();
      // the listed quads, up to two a thread
      float v[8];
      int quad[2], pb[8];                                // pages' buckets, 2048 = takes no part
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bool on = tid + i * NT < n_listed;
        quad[i] = on ? ls.quad[tid + i * NT] : -1;
        const float4 x = on ? ls.score[tid + i * NT] : make_float4(0.f, 0.f, 0.f, 0.f);
        const u32 fr = on ? free_of(4 * quad[i]) : 0u;
        v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = 4 * i + e, bj = (fr >> e) & 1u ? bucket_of(v[j]) : 2048;
          pb[j] = bj <= last ? bj : 2048;
          if (pb[j] < 2048) packed_bin_add<16>(hist_pages, pb[j]);
        }
      }
      auto key_of = [&](int j) -> u64 { return selection_order_key(v[j], 4 * quad[j >> 2] + (j & 3)); };
      decide([&]() {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (pb[j] == bin) sm.a.sel.cand[atomicAdd(&sm.tied_n, 1)] = key_of(j);
      }, NothingToDo());
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (quad[i] < 0) continue;
        u32 in = upto(4 * quad[i], n_valid) & ~free_of(4 * quad[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = 4 * i + e;
          in |= pb[j] < bin || (pb[j] == bin && key_of(j) <= thr) ? 1u << e : 0u;
        }
        ls.picked[quad[i]] = (unsigned char)in;
      }
    } else {
      // this thread's pages up to bucket `last`; those in it, which are most of them, are counted by the wave (one by one they wait for
      // each other at one word)
      int at_last = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (bk[q] > last) continue;
        const u32 fr = free_of(page_of(q));
        const float x[4] = {s[q].x, s[q].y, s[q].z, s[q].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int b = (fr >> e) & 1u ? bucket_of(x[e]) : 2048;
          at_last += b == last ? 1 : 0;
          if (b < last && !one_bucket) packed_bin_add<16>(hist_pages, b);
        }
      }
      at_last = wave_inclusive_scan(at_last);
      if (lane == kWave - 1 && at_last > 0 && !one_bucket) packed_bin_add<16>(hist_pages, last, (u32)at_last);
      u32 in = 0, tied = 0;                              // bit 4q + e: page_of(q) + e lies before the decisive bucket, or in it
      auto pages_of = [&](u32 bits, auto f) {            // (their scores come from memory again)
        while (bits) {
          const int bit = __ffs((int)bits) - 1;
          bits &= bits - 1;
          const int p = page_of(bit >> 2) + (bit & 3);
          f(bit, selection_order_key(sc[p], p));
        }
      };
      decide([&]() { pages_of(tied, [&](int, u64 key) { sm.a.sel.cand[atomicAdd(&sm.tied_n, 1)] = key; }); },
             [&]() {
#pragma unroll
               for (int q = 0; q < Q; ++q) {
                 const u32 fr = bk[q] <= last ? free_of(page_of(q)) : 0u;
                 const float x[4] = {s[q].x, s[q].y, s[q].z, s[q].w};
#pragma unroll
                 for (int e = 0; e < 4; ++e) {
                   const int b = (fr >> e) & 1u ? bucket_of(x[e]) : 2048;
                   in |= b < bin ? 1u << (4 * q + e) : 0u;
                   tied |= b == bin ? 1u << (4 * q + e) : 0u;
                 }
               }
             });
      if (thr == ~0ull) in |= tied;
      else pages_of(tied, [&](int bit, u64 key) { in |= key <= thr ? 1u << bit : 0u; });
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (bk[q] <= last) ls.picked[page_of(q) >> 2] |= (unsigned char)((in >> (4 * q)) & 15u);   // (beside its forced pages)
    }
  }
  __syncthreads();
  // output in ascending page order: 32 pages a thread
  static_assert(kHeldPages == 32 * NT, "a thread's 32 pages are eight bytes of the map");
  u64 bits = 32 * tid < n_valid ? reinterpret_cast<const u64*>(ls.picked)[tid] : 0ull;
  int total;
  int pos = fast_scan<NT>((int)__popcll(bits), sm, flip, total);
  int32_t* out = a.sel_pages + (size_t)u * k;
  while (bits) {
    const int bit = __ffsll((unsigned long long)bits) - 1;
    bits &= bits - 1;
    const int p = 32 * tid + 4 * (bit >> 3) + (bit & 7);
    if (pos < k) { sm.sel[pos] = (u32)p; out[pos] = p; }
    ++pos;
  }
  for (int i = k_eff + tid; i < k; i += NT) {
    sm.sel[i] = Smem::kNoPage;
    out[i] = -1;
  }
}

// All NT threads of a workgroup, for unit u.  DO_SELECT: scores -> sel_pages (Top-K, ties to the
// lower page, sink/recent pages forced, ascending page order, -1 padding).  DO_RESOLVE: sel_pages
// -> directory update, slots, hit mask, evicted list, counts, the (page, slot) miss list and,
// with do_gather, the copy of the missed pages into their slots.  HANDOFF: the scores were
// written by other workgroups of the same launch and are read with device-scope loads, and the
// selection is handed to the launch's attention workgroups through a.sel_entry: an entry that hits
// is published at once, an entry that missed when the fetched pages have been written through.
// Needs NP <= NT * IPT, Cmax <= KVD_FAST_MAX_CAPACITY, k <= KVD_MAX_TOPK.
// scores_ready() (HANDOFF only) is called by all threads once everything that does not depend on
// the scores has been done; it waits for them and returns false to give up: with DO_SELECT wave by wave, without a barrier
// inside (a wave loads its scores as soon as it has seen them complete), else as a workgroup.  Returns false then.
// scores_taken(): every wave has seen them complete (called by all threads).
// SEL_IN_LDS (with HANDOFF and without DO_SELECT): scores_ready() itself produces the selection —
// the hierarchical index's cluster selection, by the same workgroup — and leaves it in sm.sel
// (16-bit pages, kAbsent = padding) and in a.sel_pages; nothing is read back from global memory.
// BIG: more pages than the registers hold (NP <= KVD_BIG_MAX_PAGES whatever IPT, Cmax <= KVD_BIG_MAX_CAPACITY;
// without HANDOFF): select_big takes the pages, slots are read again where they are needed.  HELD: 1 the registers hold the
// scores (NP <= 32 NT), 2 and k <= NT: sequences of more than 12 NT pages are selected by quads.
struct ScoresAlreadyThere { __device__ bool operator()() const { return true; } };
template <int NT, int IPT, bool DO_SELECT, bool DO_RESOLVE, bool HANDOFF, class ScoresReady = ScoresAlreadyThere,
          bool SEL_IN_LDS = false, bool BIG = false, int HELD = 0, class ScoresTaken = NothingToDo, int SLOTS = -1, bool SLOT_QUADS = true>
__device__ __forceinline__ bool select_resolve_body(const FastArgs& a, int u, FastSmem<NT, BIG>& sm,
                                                    ScoresReady scores_ready = ScoresReady(), ScoresTaken scores_taken = ScoresTaken()) {
  static_assert(!(BIG && HANDOFF), "the big form is a kernel of its own");
  typedef typename FastSmem<NT, BIG>::page_t page_t;
  constexpr page_t kNoPage = FastSmem<NT, BIG>::kNoPage;
  constexpr int CPT = FastSmem<NT, BIG>::kMaxCapacity / NT;
  constexpr int UNROLL = BIG ? 1 : CPT;                 // (BIG: slots are read again where they are needed, not held in registers)
  constexpr int KPT = KVD_MAX_TOPK / NT;
  constexpr int NW = NT / kWave;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  const int b = u / a.Hkv;
  const int k = a.k;
  int flip = 0;

  // ---- every global load of the block, issued up front
  int32_t* spage = a.slot_page + (size_t)u * a.Cmax;
  int32_t* sstamp = a.slot_stamp + (size_t)u * a.Cmax;
  int sp[BIG ? 1 : CPT], ss[BIG ? 1 : CPT];           // page in slot (-1 free, -2 no such slot), stamp (BIG: read again where needed)
  int C = 0, R = 0;
  // consecutive slots per thread: as few as hold the window, or a small window would sit in one wave, which then goes through
  // the victim choice and the hand-out alone
  const int cpt = (a.Cmax + NT - 1) / NT;
  if (DO_RESOLVE) {
    if constexpr (!BIG) {
      // (slots beyond the window: -2 below.  As many slots as a thread holds come in loads of four, where every unit's start on 16 bytes: loads
      // of one word ask for the same 16 lines again each time.  us per step, all resident, 8 units of 4100 pages, windows of 3600
      // and 4000 slots 17.8 and 18.3 a word at a time, 17.1 and 17.1 so; lookahead eviction 19.9 and 18.6.  Not
      // in launches of several layers, which hide those loads and lose up to 0.7 % by the code: 6 layers of 16 units 61.5 and 61.9.)
      if (SLOT_QUADS && cpt == CPT && (a.Cmax & 3) == 0) {
#pragma unroll
        for (int j = 0; j < CPT; j += 4) {
          const int s = tid * CPT + j, at = s < a.Cmax ? s : a.Cmax - 4;
          const int4 p4 = *reinterpret_cast<const int4*>(spage + at), s4 = *reinterpret_cast<const int4*>(sstamp + at);
          sp[j] = p4.x; sp[j + 1] = p4.y; sp[j + 2] = p4.z; sp[j + 3] = p4.w;
          ss[j] = s4.x; ss[j + 1] = s4.y; ss[j + 2] = s4.z; ss[j + 3] = s4.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          const int s = tid * cpt + j;
          sp[j] = -2;
          ss[j] = 0;
          if (j >= cpt) continue;
          sp[j] = spage[s < a.Cmax ? s : a.Cmax - 1];
          ss[j] = sstamp[s < a.Cmax ? s : a.Cmax - 1];
        }
      }
    }
    C = a.capacity[u];
    R = a.resident[u];
  }
  // Page ownership: a wave owns 64 * IPT consecutive pages; its q-th 16-byte load covers 256 of
  // them (1 KiB contiguous), lane l taking four.  Item j of a lane is page_of(j).
  static_assert(IPT % 4 == 0, "four consecutive pages per load");
  const int wave_p0 = w * (kWave * IPT);
  auto page_of = [&](int j) -> int { return wave_p0 + (j >> 2) * (4 * kWave) + 4 * lane + (j & 3); };
  float s[BIG ? 4 : IPT];
  int seq = 0;
  bool by_quads = false;
  float4 held[HELD == 2 ? 8 : 1];
  auto load_scores = [&]() {
    const float* sc = a.scores + (size_t)u * a.NP;
    if ((a.NP & 3) == 0) {
      // bounds-checked by the buffer descriptor: pages beyond NP read as 0 and are never valid
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(sc), 0, a.NP * 4, 0x00020000);
#pragma unroll
      for (int q4 = 0; q4 < IPT / 4; ++q4) {
        const int off = page_of(4 * q4) * 4;
        // HANDOFF: device-scope load (the scores come from other workgroups of this launch)
        const u32x4_t v = HANDOFF ? __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 16)
                                  : __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        s[4 * q4] = as_f32(v.x); s[4 * q4 + 1] = as_f32(v.y); s[4 * q4 + 2] = as_f32(v.z); s[4 * q4 + 3] = as_f32(v.w);
      }
    } else {
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        const int p = page_of(j);
        s[j] = p < a.NP ? (HANDOFF ? load_agent(sc + p) : sc[p]) : 0.f;
      }
    }
  };
  if (DO_SELECT) {
    if (!HANDOFF && !BIG) load_scores();                       // (with HANDOFF the scores may not be complete yet)
    seq = a.seq_len[b];
    if constexpr (HELD == 2) {
      // (not where select_big's passes are few, nor for selections of which the list might not hold the quads: 16 units of 7500
      // pages 31.9 us a step with it and 33.3 with this, 2048 of 17500 pages 47.8 and 52.1.  Sequences that fill four loads of every
      // thread are not left to it beside a longer one, or the launch ends with them: one of 17000 pages and seven of 11000 pages
      // 34.6 either way, of 13000 35.6 with it and 34.7 with this, of 16300 35.8 and 34.7; all with the three passes alone 36.0.)
      by_quads = seq > 12 * NT * a.P;
      if (by_quads) select_held_load<NT>(a, u, seq, held);
    }
  } else if (!SEL_IN_LDS) {
    for (int i = tid; i < k; i += NT) {
      const int p = a.sel_pages[(size_t)u * k + i];
      sm.sel[i] = (p >= 0 && p < a.NP) ? (page_t)p : kNoPage;
    }
  }

  // ---- LDS set-up while the loads are in flight
  constexpr int kHistWords = BIG ? kRadixBins : kRadixBins / 2;   // (the ordinary form packs two buckets to a word)
  for (int i = tid; i < kHistWords; i += NT) sm.a.sel.hist[i] = 0;
  if (DO_RESOLVE) {
    u32* p2s32 = reinterpret_cast<u32*>(sm.p2s);
    for (int i = tid; i < (a.NP + 1) / 2; i += NT) p2s32[i] = 0xffffffffu;
    for (int i = tid; i < FastSmem<NT, BIG>::kMaxCapacity / 32; i += NT) sm.hit_bitmap[i] = 0;
    for (int i = tid; i < k; i += NT) sm.assign[i] = kAbsent;
  }
  if (tid == 0) { sm.cand_n = 0; sm.tied_n = 0; sm.n_ev = 0; sm.late = 0; }
  __syncthreads();
  float vs[BIG ? 1 : CPT];                             // lookahead eviction: this step's score of the page in each slot
  int vat[BIG ? 1 : CPT];                              // ... and which score that is (-1: none)
  if constexpr (DO_RESOLVE && BIG) {
    // (four loads on their way at a time)
    for (int sl0 = tid; sl0 < C; sl0 += 4 * NT) {
      int p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = spage[sl0 + i * NT < C ? sl0 + i * NT : C - 1];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (sl0 + i * NT < C && p[i] >= 0) sm.p2s[p[i]] = (uint16_t)(sl0 + i * NT);
    }
  } else if constexpr (DO_RESOLVE) {
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      if (j >= cpt) break;
      const int sl = tid * cpt + j;
      if (sl >= C) sp[j] = -2;                         // slots beyond this unit's capacity do not exist
      if (sp[j] >= 0) sm.p2s[sp[j]] = (uint16_t)sl;
    }
    // (without branches by lane, so that no load waits for the one before: a slot without a page reads some entry)
    if (a.lookahead) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        vat[j] = -1;
        if (j >= cpt) continue;
        vat[j] = sp[j] < 0 ? 0 : sp[j];
        if (a.page_cluster != nullptr) vat[j] = a.page_cluster[(size_t)u * a.NP + vat[j]];
      }
    }
  }
  int32_t* sslots = a.sel_slots + (size_t)u * k;
  int32_t* hmask = a.hit_mask + (size_t)u * k;
  int32_t* evout = a.evicted + (size_t)u * k;
  u64* entry = HANDOFF ? a.sel_entry + (size_t)u * k : nullptr;
  if (HANDOFF) {
    // everything that does not need the scores is done: now wait for them
    const bool there = scores_ready();
    if (DO_SELECT) {
      if (!there) sm.late = 1;                           // (the verdict is shared at the next barrier)
      load_scores();
    } else if (!there) {
      return false;
    }
  }
  if constexpr (DO_RESOLVE && !BIG) {
    if (a.lookahead) {
      const float* sc = a.scores + (size_t)u * a.score_stride;
      if constexpr (SLOTS == kLayoutNatural) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          vs[j] = 0.f;
          if (j >= cpt) continue;
          const int at = vat[j] < 0 ? 0 : vat[j];
          vs[j] = HANDOFF ? load_agent(sc + at) : sc[at];
        }
      } else {
        // No branch by the number of slots: what there is no score for lies outside the buffer.  (us per step without misses, 8 units of
        // 5625 pages of 16 tokens, a thread's 8 slots one by one, as many as it has with branches, and so: k = 200, window 3400,
        // 22.8, 23.0 and 22.9, k = 907 31.3, 31.6 and 31.3; of 4 tokens, k = 907, 23.8, 23.9 and 23.4.  In the launch over natural slots
        // this code costs steps with eviction by age 0.6 %: 32 units of 2084 pages of 24 23.9 and 24.0.)
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(sc), 0, a.score_stride * 4, 0x00020000);
#pragma unroll
        for (int j = 0; j < CPT; ++j)
          vs[j] = as_f32((u32)__builtin_amdgcn_raw_buffer_load_b32(rs, sp[j] >= 0 ? vat[j] * 4 : -4, 0, HANDOFF ? 16 : 0));
      }
    }
  }

  // ---- selection
  if constexpr (DO_SELECT && BIG) {
    if (HELD == 2 && by_quads) {
      if constexpr (HELD == 2) select_held<NT>(a, u, seq, held, sm, flip);
    } else {
      select_big<NT, HELD != 0>(a, u, seq, sm, flip);
    }
    if (!DO_RESOLVE) return true;
  } else if constexpr (DO_SELECT) {
    constexpr int kBinWords = IPT == 4 ? 8 : 16;       // 1024 or 2048 buckets
    constexpr float kBins = 128.0f * kBinWords;
    int n_valid = (seq + a.P - 1) / a.P;
    n_valid = n_valid < a.NP ? n_valid : a.NP;
    const int k_eff = k < n_valid ? k : n_valid;
    const int recent_from = n_valid - a.recent;
    // Which of this lane's pages are free to compete and which are forced, four consecutive pages
    // at a time: free = [sink, recent_from), forced = the other valid pages.
    u32 free_mask = 0, forced_mask = 0;               // bit j: page_of(j)
#pragma unroll
    for (int q4 = 0; q4 < IPT / 4; ++q4) {
      const int base = page_of(4 * q4);
      auto upto = [&](int bound) -> u32 {              // bits of the group's pages below `bound`
        const int n = bound - base;
        return (1u << (n < 0 ? 0 : (n > 4 ? 4 : n))) - 1u;
      };
      const u32 fr = upto(recent_from) & ~upto(a.sink);
      free_mask |= fr << (4 * q4);
      forced_mask |= (upto(n_valid) & ~fr) << (4 * q4);
    }
    float fmin = INFINITY, fmax = -INFINITY;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const bool fr = (free_mask >> j) & 1u;
      fmin = fminf(fmin, fr ? s[j] : INFINITY);
      fmax = fmaxf(fmax, fr ? s[j] : -INFINITY);
    }
    fmin = wave_allreduce_min(fmin);
    fmax = wave_allreduce_max(fmax);
    if (lane == 0) sm.red[w] = make_float2(fmin, fmax);
    __syncthreads();
    if (HANDOFF && sm.late) return false;
    scores_taken();
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      fmin = fminf(fmin, sm.red[i].x);
      fmax = fmaxf(fmax, sm.red[i].y);
    }
    const int n_free = recent_from > a.sink ? recent_from - a.sink : 0;
    const int k_free = k_eff - (n_valid - n_free);
    const float range = fmax - fmin;
    const float inv = range > 0.f ? (kBins - 1.0f) / range : 0.f;
    auto bucket_of = [&](float v) -> int { return (int)fminf(fmaxf((fmax - v) * inv, 0.f), kBins - 1.0f); };
    // every free page's bucket, computed once and kept, with many pages per lane two to a register; kNoBucket = not free
    constexpr int kNoBucket = 0x7fff;
    constexpr bool kPairs = IPT > 8;
    u32 bk[kPairs ? IPT / 2 : IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const u32 bj = ((free_mask >> j) & 1u) ? (u32)bucket_of(s[j]) : (u32)kNoBucket;
      if (!kPairs) bk[j] = bj;
      else if (j & 1) bk[j >> 1] |= bj << 16;
      else bk[j >> 1] = bj;
    }
    auto bucket_at = [&](int j) -> int { return kPairs ? (int)((bk[j >> 1] >> (16 * (j & 1))) & 0xffffu) : (int)bk[j]; };
    u32 take = forced_mask;                            // bit j: page_of(j) is selected
    if (k_free > 0) {
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if ((free_mask >> j) & 1u) packed_bin_add<kBinWords>(sm.a.sel.hist, bucket_at(j));
      __syncthreads();
      int bin, below, m;
      packed_bin_find<kBinWords>(sm.a.sel.hist, k_free, bin, below, m);
      const int r = k_free - below;                    // of the m pages of the decisive bucket r are in
      // a page in a bucket before the decisive one is in, one in a later bucket is out
      u32 tied = 0;
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        const int bb = bucket_at(j);
        take |= bb < bin ? (1u << j) : 0u;
        tied |= bb == bin ? (1u << j) : 0u;
      }
      if (r == m) {
        take |= tied;
      } else if (m <= kListCap) {
        // their keys go into one list, a wave's with one add to its length
        if (__any(tied != 0)) {
          const int mine = __popc(tied), inc = wave_inclusive_scan(mine);
          int at = 0;
          if (lane == kWave - 1) at = atomicAdd(&sm.cand_n, inc);
          at = __builtin_amdgcn_readlane(at, kWave - 1) + inc - mine;
#pragma unroll
          for (int j = 0; j < IPT; ++j)
            if ((tied >> j) & 1u) sm.a.sel.cand[at++] = selection_order_key(s[j], page_of(j));
        }
        // up to half a wave's lanes every wave ranks the list for itself, which saves a barrier and the broadcast of the key; a
        // longer one (many pages alike) is dealt out to the threads.  (us per token of 4 layers, 32 units of 1001 pages that grow by
        // pages that are all alike, with every wave ranking any list, up to 64 keys, and up to 32: after 2000 tokens 110.6, 110.6 and 107.9, after 2700 113.3, 109.4 and 109.9.)
        u64 thr;
        if (m <= kWave / 2) {
          __syncthreads();
          thr = kth_of_list(sm.a.sel.cand, m, r);
        } else {
          thr = rank_candidates<NT>(m, r, sm);
        }
#pragma unroll
        for (int j = 0; j < IPT; ++j)
          if (((tied >> j) & 1u) && selection_order_key(s[j], page_of(j)) <= thr) take |= 1u << j;
      } else {
        const float* sc = a.scores + (size_t)u * a.NP;
        auto fn = [&](int i, u64& kk) -> bool {
          if (i < a.sink || i >= recent_from) return false;
          const float v = HANDOFF ? load_agent(sc + i) : sc[i];
          if (bucket_of(v) != bin) return false;
          kk = selection_order_key(v, i);
          return true;
        };
        const u64 thr = block_kth_smallest<NT>(fn, n_valid, r, sm.generic, sm.a.sel.hist);
#pragma unroll
        for (int j = 0; j < IPT; ++j)
          if (((tied >> j) & 1u) && selection_order_key(s[j], page_of(j)) <= thr) take |= 1u << j;
      }
    }
    int32_t* out = a.sel_pages + (size_t)u * k;
    // output in ascending page order = (wave, load, lane, element): one block scan over the
    // lanes' totals gives the wave's first position, wave scans per load give the rest
    int total;
    const int lane_pos = fast_scan<NT>(__popc(take), sm, flip, total);
    if (IPT == 4) {
      // (a lane's pages follow each other; a page that is not selected goes to a place of the lane's own behind the others)
      int pos = lane_pos;
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        const bool in = (take >> j) & 1u;
        sm.sel[in ? pos : KVD_MAX_TOPK + lane] = (page_t)page_of(j);
        pos += in ? 1 : 0;
      }
    } else {
      int pos_q = __builtin_amdgcn_readfirstlane(lane_pos);   // lane 0: what the waves before this one selected
#pragma unroll
      for (int q4 = 0; q4 < IPT / 4; ++q4) {
        const u32 bits = (take >> (4 * q4)) & 15u;
        const int cnt = __popc(bits), inc = wave_inclusive_scan(cnt);
        int pos = pos_q + inc - cnt;
        pos_q += __builtin_amdgcn_readlane(inc, kWave - 1);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((bits >> e) & 1u) sm.sel[pos++] = (page_t)page_of(4 * q4 + e);
      }
    }
    for (int i = k_eff + tid; i < k; i += NT) sm.sel[i] = kNoPage;
    if (!DO_RESOLVE) {
      __syncthreads();
      for (int i = tid; i < k; i += NT) out[i] = i < k_eff ? (int)sm.sel[i] : -1;
      return true;
    }
  }

  // ---- resolve: lookup in the LDS map
  __syncthreads();                                     // the selection is in LDS
  const int per = (k + NT - 1) / NT;                   // consecutive selected entries per thread
  const int i0 = tid * per;
  int my_page[KPT];                                    // this thread's misses
  int my_misses = 0, my_hits = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    my_page[j] = -2;
    const int i = i0 + j;
    if (j < per && i < k) {
      const page_t entry_page = sm.sel[i];
      const bool none = entry_page == kNoPage;         // padding (or a page the caller made up)
      const int p = none ? -1 : (int)entry_page;
      const int sl = none ? -1 : (int)sm.p2s[p];
      const bool hit = !none && sl != kAbsent, miss = !none && sl == kAbsent;
      if (HANDOFF && !miss) store_agent(entry + i, pack_sel_entry(p, sl));
      if (hit) {
        sstamp[sl] = a.step;
        atomicOr(&sm.hit_bitmap[sl >> 5], 1u << (sl & 31));
      }
      if (!miss) sslots[i] = sl;
      hmask[i] = hit ? 1 : 0;
      if (DO_SELECT && !BIG) a.sel_pages[(size_t)u * k + i] = p;
      my_hits += hit ? 1 : 0;
      my_misses += miss ? 1 : 0;
      if (miss) my_page[j] = p;
    }
  }
  // one scan counts both: misses in the low half, hits in the high half (k <= 2048 each)
  int mh;
  const int ranks = fast_scan<NT>(my_misses | (my_hits << 16), sm, flip, mh);   // barrier inside: everyone is done with sm.sel
  int miss_rank = ranks & 0xffff;
  const int m = mh & 0xffff, n_hits = mh >> 16;
#pragma unroll
  for (int j = 0; j < KPT; ++j)
    if (my_page[j] >= 0) sm.miss[miss_rank++] = (u32)my_page[j] | ((u32)(i0 + j) << 16);
  const int e = (R + m - C) > 0 ? (R + m - C) : 0;
  if (m == 0) {
    // every selected page is resident: no slot to find, nothing leaves, nothing to fetch
    for (int j = tid; j < k; j += NT) evout[j] = -1;
    if (tid == 0) {
      a.miss_count[u] = 0;
      a.counts[u * 3 + 0] = n_hits;
      a.counts[u * 3 + 1] = 0;
      a.counts[u * 3 + 2] = 0;
      atomicAdd(&a.stats[0], (unsigned long long)n_hits);
    }
    return true;
  }
  // the histogram and the candidate counter serve the victim choice next
  if (DO_SELECT) {
    __syncthreads();                                   // (the candidates of the selection have been read)
    for (int i = tid; i < kHistWords; i += NT) sm.a.sel.hist[i] = 0;
    if (tid == 0) sm.cand_n = 0;
  }
  __syncthreads();                                     // ... and the hit bitmap and the misses are complete

  // ---- victims: the e smallest (stamp, page) among resident slots that were not hit
  // what this thread's j-th slot holds (the directory is written only after the slots have been handed out)
  auto page_at = [&](int j) -> int {
    if constexpr (BIG) return tid * cpt + j < C ? spage[tid * cpt + j] : -2;
    else return sp[j];
  };
  auto stamp_at = [&](int j) -> int {
    if constexpr (BIG) return sstamp[tid * cpt + j];
    else return ss[j];
  };
  auto score_at = [&](int j, int page) -> float {
    if constexpr (BIG) return a.lookahead ? victim_score<HANDOFF>(a, u, page) : 0.f;
    else return a.lookahead && vat[j] < 0 ? -INFINITY : vs[j];   // (a page of no cluster leaves first)
  };
  u32 cand_mask = 0;
#pragma unroll UNROLL
  for (int j = 0; j < CPT; ++j) {
    if (j >= cpt) break;
    const int sl = tid * cpt + j;
    const bool cand = page_at(j) >= 0 && !((sm.hit_bitmap[sl >> 5] >> (sl & 31)) & 1u);
    cand_mask |= cand ? (1u << j) : 0u;
  }
  // lookahead eviction buckets the candidates' scores linearly between their extremes
  float vmin = 0.f, vinv = 0.f;
  if (a.lookahead && e > 0) {
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll UNROLL
    for (int j = 0; j < CPT; ++j) {
      if (j >= cpt) break;
      if (!((cand_mask >> j) & 1u)) continue;
      const float v = score_at(j, page_at(j));
      if (v > -INFINITY) {                             // (a page of no cluster scores -inf: bucket 0 whatever the range)
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
      }
    }
    lo = wave_allreduce_min(lo);
    hi = wave_allreduce_max(hi);
    if (lane == 0) sm.red[w] = make_float2(lo, hi);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      lo = fminf(lo, sm.red[i].x);
      hi = fmaxf(hi, sm.red[i].y);
    }
    vmin = lo;
    vinv = hi > lo ? 2047.0f / (hi - lo) : 0.f;
  }
  const float page_scale = 32.f / (float)a.NP;
  auto la_bucket = [&](float v) -> int { return (int)fminf(fmaxf((v - vmin) * vinv, 0.f), 2047.f); };
  // A finite look-ahead pool: the key of the pool's last member in selection order (best page first)
  // over the unit's valid pages; a resident page is in the pool iff its key is not beyond it.
  bool pooled = false;
  u64 pool_thr = ~0ull;
  if (a.lookahead && a.la_pool > 0 && e > 0) {
    int n_valid = (a.seq_len[b] + a.P - 1) / a.P;
    n_valid = n_valid < a.NP ? n_valid : a.NP;
    if (a.la_pool < n_valid) {
      pooled = true;
      // Bound by the latency of the loads, of which a thread makes up to seven rounds.  (us per step with misses, a load at
      // a time with 1024 threads, with 512, and four at a time with 512: 8 units of 9000 pages 142, 149 and 133, 24 of 16384
      // 313, 338 and 302, 64 of 9000 583, 587 and 576, with clusters 16 of 9000 168, 186 and 171; eight at a time gain no
      // more, and 176 there.  Scores fetched once and kept in registers cost every step 20 % through the code they add.)
      // Without branches: a page of no cluster reads some score and has minus infinity.
      const float* sc = a.scores + (size_t)u * a.score_stride;
      const int32_t* cl = a.page_cluster != nullptr ? a.page_cluster + (size_t)u * a.NP : nullptr;
      auto score_of = [&](int at) -> float { return HANDOFF ? load_agent(sc + at) : sc[at]; };
      auto of_page = [&](int p, u64& kk) -> bool {
        kk = selection_order_key(score_of(p), p);
        return true;
      };
      auto of_cluster = [&](int p, u64& kk) -> bool {
        const int c = cl[p];
        const float v = score_of(c < 0 ? 0 : c);
        kk = selection_order_key(c < 0 ? -INFINITY : v, p);
        return true;
      };
      constexpr int kAhead = 4;
      pool_thr = cl == nullptr ? block_kth_smallest<NT, kAhead>(of_page, n_valid, a.la_pool, sm.generic, sm.a.sel.hist)
                               : block_kth_smallest<NT, kAhead>(of_cluster, n_valid, a.la_pool, sm.generic, sm.a.sel.hist);
      // (the histogram serves the victim choice next: it must start from zero again)
      __syncthreads();
      for (int i = tid; i < kHistWords; i += NT) sm.a.sel.hist[i] = 0;
      __syncthreads();
    }
  }
  auto in_pool = [&](float v, int page) -> bool { return selection_order_key(v, page) <= pool_thr; };
  auto la_key = [&](float v, int st, int page) -> u64 {
    return pooled ? pooled_victim_key(in_pool(v, page), v, st, page) : lookahead_victim_key(v, page);
  };
  auto la_bkt = [&](float v, int st, int page) -> int {
    if (!pooled) return la_bucket(v);
    // the halves of the bucket range: outside the pool by age, inside by score
    return in_pool(v, page) ? 1024 + (la_bucket(v) >> 1) : (victim_bucket(a.step, st, page, page_scale) >> 1);
  };
  auto vkey_of = [&](int j) -> u64 {
    const int st = stamp_at(j), p = page_at(j);
    return a.lookahead ? la_key(score_at(j, p), st, p) : ((u64)((u32)st ^ 0x80000000u) << 32) | (u32)p;
  };
  auto vbkt_of = [&](int j) -> int {
    if (!((cand_mask >> j) & 1u)) return -1;
    const int st = stamp_at(j), p = page_at(j);
    return a.lookahead ? la_bkt(score_at(j, p), st, p) : victim_bucket(a.step, st, p, page_scale);
  };
  u64 vthr = 0;
  if (e > 0) {
    auto refine = [&](int bin, int r) -> u64 {
      auto fn = [&](int sl, u64& kk) -> bool {
        const int p = spage[sl];
        if (p < 0 || ((sm.hit_bitmap[sl >> 5] >> (sl & 31)) & 1u)) return false;
        const int st = sstamp[sl];
        if (a.lookahead) {
          const float v = victim_score<HANDOFF>(a, u, p);
          if (la_bkt(v, st, p) != bin) return false;
          kk = la_key(v, st, p);
          return true;
        }
        if (victim_bucket(a.step, st, p, page_scale) != bin) return false;
        kk = ((u64)((u32)st ^ 0x80000000u) << 32) | (u32)p;
        return true;
      };
      return block_kth_smallest<NT>(fn, C, r, sm.generic, sm.a.sel.hist);
    };
    vthr = two_level_select<NT, CPT>(vkey_of, vbkt_of, cpt, e, sm, flip, refine);
  }

  // ---- hand out slots: free slots and victim slots in ascending slot order go to the misses in
  // ascending page order
  int avail = 0;
  u32 av_mask = 0, vic_mask = 0;
#pragma unroll UNROLL
  for (int j = 0; j < CPT; ++j) {
    if (j >= cpt) break;
    const bool vic = e > 0 && ((cand_mask >> j) & 1u) && vkey_of(j) <= vthr;
    const bool av = page_at(j) == -1 || vic;
    vic_mask |= vic ? (1u << j) : 0u;
    av_mask |= av ? (1u << j) : 0u;
    avail += av ? 1 : 0;
  }
  int total_avail;
  int rank = fast_scan<NT>(avail, sm, flip, total_avail);
#pragma unroll UNROLL
  for (int j = 0; j < CPT; ++j) {
    if (j >= cpt) break;
    if ((av_mask >> j) & 1u) {
      if (rank < m) {
        sm.assign[rank] = (uint16_t)(tid * cpt + j);
        if ((vic_mask >> j) & 1u) {
          const int at = atomicAdd(&sm.n_ev, 1);
          if (at < k) evout[at] = page_at(j);
        }
      }
      ++rank;
    }
  }
  __syncthreads();
  for (int i = tid; i < m; i += NT) {
    const int p = (int)(sm.miss[i] & 0xffffu), pos = (int)(sm.miss[i] >> 16);
    const int sl = sm.assign[i];
    const int slot = sl == kAbsent ? -1 : sl;         // always a slot while the directory is consistent
    sslots[pos] = slot;
    if (slot >= 0) {
      spage[slot] = p;
      sstamp[slot] = a.step;
    }
    a.miss_list[((size_t)u * k + i) * 2] = p;
    a.miss_list[((size_t)u * k + i) * 2 + 1] = slot;
  }
  for (int j = e + tid; j < k; j += NT) evout[j] = -1;
  if (tid == 0) {
    a.resident[u] = R + m - e;
    a.miss_count[u] = m;
    a.counts[u * 3 + 0] = n_hits;
    a.counts[u * 3 + 1] = m;
    a.counts[u * 3 + 2] = e;
    atomicAdd(&a.stats[0], (unsigned long long)n_hits);
    atomicAdd(&a.stats[1], (unsigned long long)m);
    atomicAdd(&a.stats[2], (unsigned long long)e);
  }
  // the misses' entries go out when every wave's copies have been acknowledged
  auto publish_misses = [&]() {
    if (!HANDOFF) return;
    wave_drain_memory();
    __syncthreads();
    for (int i = tid; i < m; i += NT)
      store_agent(entry + (sm.miss[i] >> 16), pack_sel_entry((int)(sm.miss[i] & 0xffffu), sm.assign[i] == kAbsent ? -1 : (int)sm.assign[i]));
  };
  if (!a.do_gather) {
    publish_misses();
    return true;
  }

  // ---- fetch the unit's missed pages, miss j being page sm.miss[j] for slot sm.assign[j].  Every wave for itself, without
  // barriers, a batch of pieces on its way at a time: four tokens' K and V a piece, or, in natural slots, 1 KiB.  Bound by the host
  // link, which takes 150 KB on their way to be busy (read by 8 workgroups 25 GB/s with 8 KiB of each on their way, 54 with
  // 32; 16 workgroups 56), and for few units by its latency.  (us per step with misses, with tiles of 256 threads, two
  // barriers and 16 KiB on their way, and so, the victim choice above included: 4 units of 1024 pages of 64 tokens 56.2 and 43.3,
  // 8 of 750 of 16 46.1 and 38.4, 8 of 4096 of 4 54.8 and 47.0, 32 of 8192 of 16 284.8 and 274.1.  The code is met cold, so less
  // of it is faster: with a second batch on its way while the first is stored, which is five copies of the unrolled loops instead of
  // two, these were 44.6, 41.0, 49.2 and 277.5.)
  __syncthreads();                                     // everyone is done with sm.a.sel
  const char* store_u = a.store + (size_t)u * a.NP * a.page_bytes;
  char* pool_u = a.pool + (size_t)u * a.Cmax * a.page_bytes;
  const int layout = SLOTS >= 0 ? SLOTS : a.tiled;
  const int pieces = layout == kLayoutNatural ? (a.P + 1) >> 1 : a.P >> 2, n_items = m * pieces;   // (a page is P half KiB)
  // Without branches: what is no item, or has no slot, is a buffer without bytes, whose loads and stores do nothing.  (A load
  // under a condition was waited for at once, where its register is joined with that of the other way.)
  // (at / pieces by the reciprocal rounded up: exact below 2^32 / pieces^2, and at most 2048 pages have 128 pieces each)
  const u32 recip = 0xffffffffu / (u32)pieces + 1u;    // (0 for one piece)
  const int w0 = __builtin_amdgcn_readfirstlane(w);      // (the compiler does not see that it is one number to a wave, and would load lane by lane)
  struct Piece { const char* src; char* dst; u32 bytes; int piece; };
  auto item = [&](int it, int end) -> Piece {
    const int at = it < n_items ? it : n_items - 1;
    const int jm = __builtin_amdgcn_readfirstlane(pieces == 1 ? at : (int)(((u64)(u32)at * recip) >> 32));
    const int slot = __builtin_amdgcn_readfirstlane((int)sm.assign[jm]);
    const u32 page = (u32)__builtin_amdgcn_readfirstlane((int)(sm.miss[jm] & 0xffffu));
    Piece x;
    x.bytes = it < end && slot != kAbsent ? a.page_bytes : 0u;
    x.src = store_u + (size_t)page * a.page_bytes;
    x.dst = pool_u + (size_t)slot * a.page_bytes;
    x.piece = at - jm * pieces;
    return x;
  };
  // 64 KiB of a workgroup are on their way at a time; with 48 units and more in a launch 16 (24 over natural slots).  So many
  // workgroups keep the link busy with less, and with more it is a queue of megabytes, at whose end they all come at once.  (us per step
  // with misses before the copies by waves, with 64 KiB, and so: 128 units of 175 pages of 32 tokens, k = 4, 154, 170 and 149,
  // k = 12 344, 354 and 337, 96 of 700 of 8 in two layers 238, 258 and 231, natural slots, 64 of 300 of 12 in two layers 350,
  // 326 and 316; as a chain 128 of 175, k = 12, of 16 192, 201 and 183, of 12 146, 163 and 143.  With 64 and 16 KiB 4 units of 175
  // of 32 33.5 and 34.9, 32 99.0 and 99.0, 64 178 and 176.)  With 512 threads every wave has fewer pieces, and those beyond are
  // asked for of a buffer without bytes and not stored (loops of their own cost the steps without misses 1 % through the code); with 1024
  // every fourth wave has all of its pieces, which is faster there (183 above with the other way 190).
  const int waves = NT > 512 && a.shallow_fetch ? NW / 4 : NW;
  if (layout == kLayoutNatural) {
    constexpr int kBatch = NT > 512 ? 4 : 8;
    const int depth = NT <= 512 && a.shallow_fetch ? 3 : kBatch;
    for (int it = w0 < waves ? w0 : n_items; it < n_items; it += depth * waves) {
      const int end = NT <= 512 && it + depth * NW < n_items ? it + depth * NW : n_items;
      uint4 v[kBatch];
      Piece of[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        of[i] = item(it + i * waves, end);
        v[i] = buffer_load16(of[i].src, of[i].bytes, (u32)of[i].piece * 1024u + (u32)lane * 16u);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (NT <= 512 && it + i * NW >= end) break;
        buffer_store16<HANDOFF>(of[i].dst, of[i].bytes, (u32)of[i].piece * 1024u + (u32)lane * 16u, v[i]);
      }
    }
  } else {
    constexpr int kBatch = NT > 512 ? 2 : 4;
    const int depth = NT <= 512 && a.shallow_fetch ? 1 : kBatch;
    const int tile_tokens = layout == kLayoutTiles ? kTileTokens : a.P;
    uint16_t* vt = &sm.a.vt[w][0];
    for (int it = w0 < waves ? w0 : n_items; it < n_items; it += depth * waves) {
      const int end = NT <= 512 && it + depth * NW < n_items ? it + depth * NW : n_items;
      PageGroup g[kBatch];
      Piece of[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        of[i] = item(it + i * waves, end);
        page_group_load(of[i].src, of[i].bytes, a.P, of[i].piece, g[i]);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (NT <= 512 && it + i * NW >= end) break;
        page_group_store<HANDOFF>(of[i].dst, of[i].bytes, tile_tokens, of[i].piece, vt, g[i]);
      }
    }
  }
  publish_misses();
  return true;
}

}  // namespace kvd
