// Host side of the one-launch step: its launch shape, where it can run, and the launch (the kernel: kvd_step_body.h).
#include "kvd_step_body.h"

// The splits that the rule leaves a launch with.  Where the library takes one layer as a chain of kernels and several in a
// launch, these have that chain's splits, for the same order of the sums.
static int rule_splits(const kvd_ctx* c, int multi_layer) {
  if (c->natural_launch) return c->S_natural;
  return multi_layer && !c->single_launch && kvd_layers_share_launch(c) ? c->S : c->S1;
}

// The launch shape of the one-launch step.  What kvd_set_step_shape / kvd_calibrate_step_shape fixed
// is taken; the rest follows the rule: one group; scoring workgroups = one round of resident
// workgroups (one per CU) minus 1/8 left to the selection workgroups that run beside them; passes
// such that the chunks of a group fill whole rounds of its scoring workgroups (time ~ rounds x
// passes; at equal cost the coarser chunk wins while every scoring workgroup still gets one: fewer
// reports and acknowledgement waits per byte); splits as kvd_create chose them.
//
// Units of more than 8192 pages make at most two passes: with more, few large chunks complete all units at once, and nothing
// overlaps their selection (us per step with the passes that the above would take and with this: 32 units of 16384 pages 5: 50.9
// and 49.2, 32 of 12500 4: 45.2 and 43.3, 64 of 9375 3: 61.1 and 59.8).
//
// Launches of several layers take scoring chunks of two passes as soon as those of one fill 3/4 of the CUs, over all layers,
// or, where the second chunk of a unit would be cut short, in one layer: the other layers cover what a coarser chunk leaves
// idle (us per layer-step with one pass and with two: 64 units of 2048 pages, 8 layers 19.1 and 18.8, 4 layers 21.2 and
// 20.8, 128 units of 538 pages 17.9 and 16.6, 128 of 2048 35.9 and 35.5; the fewer units lose a little: 8 of 4096 pages 6.4
// and 6.5, 16 of 1024 7.4 and 7.6, 32 of 2048, 3 layers 13.9 and 14.5).
kvd_shape kvd_step_shape(const kvd_ctx* c, int multi_layer, const kvd_shape* want, int n_layers) {
  kvd_shape w = want ? *want : c->shape[multi_layer ? 1 : 0];
  if (!multi_layer) n_layers = 1;
  else if (n_layers <= 0) n_layers = c->n_sets;         // (the most layers a launch of this context covers)
  const int score_np = c->Nc > 0 ? c->Nc : c->NP;
  const int chunk_pages = kvd::kStepThreads;
  const int slots = c->n_cus;
  kvd_shape e;
  e.groups = w.groups > 0 ? w.groups : 1;
  if (e.groups > c->U) e.groups = c->U;
  const int Ug = (c->U + e.groups - 1) / e.groups;      // units per group
  e.groups = (c->U + Ug - 1) / Ug;                      // (no empty group)
  int ns = w.n_score;
  if (ns <= 0) {
    int reserve = slots / 8;
    if (reserve > Ug) reserve = Ug;
    ns = slots - reserve;
  }
  if (ns < 1) ns = 1;
  int ps = w.passes;
  if (ps <= 0) {
    const int most = c->NP > 8192 ? 2 : 8;
    long long best_cost = -1;
    for (int cand = 1; cand <= most; ++cand) {
      const long long chunks = (score_np + (long long)chunk_pages * cand - 1) / ((long long)chunk_pages * cand);
      const long long rounds = (chunks * Ug + ns - 1) / ns;
      const long long cost = rounds * cand;
      if (best_cost < 0 || cost < best_cost || (cost == best_cost && chunks * Ug >= ns)) { best_cost = cost; ps = cand; }
    }
    const long long layer_chunks = (long long)c->U * ((score_np + chunk_pages - 1) / chunk_pages);
    if (ps == 1 && n_layers > 1 && (score_np >= 2 * chunk_pages ? n_layers * layer_chunks : score_np > chunk_pages ? layer_chunks : 0) >= 3LL * slots / 4)
      ps = 2;
  }
  const int chunks = (score_np + chunk_pages * ps - 1) / (chunk_pages * ps);
  if (ns > Ug * chunks) ns = Ug * chunks;
  e.passes = ps;
  e.n_score = ns;
  e.splits = w.splits > 0 ? w.splits : rule_splits(c, multi_layer);
  return e;
}

// Which shapes the context can run: passes 1..8; 1..(compute units) scoring workgroups; splits
// within what the partials were allocated for, with a split's entries fitting their LDS staging
// area; 1..8 groups.
bool kvd_step_shape_ok(const kvd_ctx* c, const kvd_shape& e) {
  if (e.passes < 1 || e.passes > 8 || e.n_score < 1 || e.n_score > c->n_cus) return false;
  if (e.splits < 1 || e.splits > kvd_most_splits(c) || e.splits > c->k) return false;
  if ((c->k + e.splits - 1) / e.splits > kvd::kAttnIdxCap) return false;
  if (e.groups < 1 || e.groups > 8) return false;
  return true;
}

// Slots are multiples of 512 bytes: where the pool starts on a cache line, none is shared by two of them.  Elsewhere an
// attention workgroup that reads a resident slot would leave the first or last line of its neighbour in its L2, and read
// old bytes there once the launch has filled that neighbour with another page.  (No pool yet: it may come to start on a line.)
static bool slots_have_own_lines(const kvd_ctx* c) { return (reinterpret_cast<uintptr_t>(c->pool) & 127u) == 0; }

// Over natural slots (pages of a size that is neither a multiple of 16 nor 4 or 8) the library's own choice of form runs a
// step as one launch too (kvd_step_form says 0; such a context takes no form -1).  Three
// launches were three chains of latencies (us per step as a chain and so: 32 units x 2084 pages of 24 tokens, G = 7, 26.4 and 23.0,
// 16 x 500 of 100 23.8 and 21.4, 112 x 250 of 20 35.8 and 32.5, 8 units of 10417 25.9 and 25.0; with misses 32 x 750 of 12 70.9 and
// 67.2, 8 x 1000 of 20 46.9 and 44.4, 8 x 2000 of 6 42.4 and 40.7; per launch of 8 layers of 16 x 375 of 24 127.6 and 77.3,
// of 4 layers of 2 x 10417 85.0 and 24.5).
bool kvd_natural_launch_ok(const kvd_ctx* c) {
  return c->tiled == kvd::kLayoutNatural && kvd_fast_path_ok(c) && !kvd_fast_path_big(c) && slots_have_own_lines(c);
}

bool kvd_single_launch_fits(const kvd_ctx* c) {
  return kvd_fast_path_ok(c) && !kvd_fast_path_big(c) && c->tiled &&
         (c->k + c->S1 - 1) / c->S1 <= kvd::kAttnIdxCap;   // a split's entries are staged in LDS
}

bool kvd_single_launch_ok(const kvd_ctx* c) { return kvd_single_launch_fits(c) && slots_have_own_lines(c); }

// Several layers share a launch wherever one can run, unless the caller has asked for another form (us per layer-step of
// the few units above, two chains of kernels in flight and one launch: 7 layers of 8 units of 10109 pages 19.3 and 11.2, 4
// layers of 4 units of 12500 20.0 and 9.3).
bool kvd_layers_share_launch(const kvd_ctx* c) {
  return c->single_launch || c->natural_launch ||
         (c->cfg.micro_batches == 0 && (kvd_single_launch_ok(c) || kvd_natural_launch_ok(c)) && (c->k + c->S - 1) / c->S <= kvd::kAttnIdxCap);
}

// How many of a unit's splits an attention workgroup of a launch of several layers takes.  The layers fill each other's gaps
// there, so fewer and longer workgroups are better as long as there is one for seven of eight CUs over all layers; the
// workgroups of a unit are to be about equally long, and what their waves leave of each split has to fit their LDS.  The splits themselves
// stay those of a single layer, and with them the order of the sums.  (us per layer-step with one and with this many: 8
// layers of 64 units x 4 splits 21.9 and 18.8, of 32 x 8 14.6 and 11.9, of 16 x 16 10.6 and 7.4, of 128 x 2 37.7 and
// 35.5; 3 layers of 32 x 8 16.8 and 13.9, but 14.7 with 4 instead of 2; 2 of 64 x 4 25.4 and 23.4, 26.1 with 4; 4 of 8 x 8
// 4.7 with one or two, 5.9 with 4; 6 of 40 x 5 and 4 of 56 x 4, with a workgroup for every CU and for seven of eight, 14.6 and 12.3, 17.1 and 16.5.
// Where one page in five is fetched, which the host does not know, it costs up to 6 %: a launch of 8 layers of 20 units 407
// and 430, of 8 of 28 575 and 572, 3 of 20 180 and 186, 3 of 56 440 and 450.)
static int kvd_step_take(const kvd_ctx* c, int splits, int n_layers) {
  const int per_split = (c->k + splits - 1) / splits, held = kvd::StepSmem<kvd::kStepThreads>::splits_held(c->G);
  const int room = held < kvd::kAttnIdxCap / per_split ? held : kvd::kAttnIdxCap / per_split;
  int wgs = (c->n_cus * 7 / 8 + n_layers * c->U - 1) / (n_layers * c->U);
  for (; wgs < splits; ++wgs) {
    const int take = (splits + wgs - 1) / wgs;
    if (take <= room && 8 * (take * wgs - splits) < splits) return take;
  }
  return 1;
}

// The last layer's splits have a workgroup each, where the others' workgroups take three or more: nothing runs beside them,
// least of all when the last pages have just come over the link, and that many splits one after the other take 20 us and
// more.  (us per launch with misses, in which one page in 30 to one in 7 is fetched, with a workgroup to each split in all
// layers, in none, and in the last one: 4 layers of 64 units 164.3, 175.0 and 164.8, 6 of 24 117.7, 119.3 and 113.2, 8 of 20
// 415.6, 436.7 and 432.0, 8 of 56 276.0, 280.5 and 265.9; without misses the same 80.8, 68.6 and 67.6, 75.3, 58.8 and 55.2,
// 90.8, 70.0 and 65.8, 147.3, 113.7 and 113.3.  But 4 layers of 16 units, of 16 splits, 47.6, 32.4 and 34.6, 3 of 20 41.2,
// 29.5 and 33.1; where a workgroup takes two, 8 of 100 224.0, 190.2 and 194.7.)
static int kvd_step_tail_layers(int splits, int take, int n_layers) {
  return take >= 3 && n_layers >= (splits > 8 ? 5 : 4) ? 1 : 0;
}

hipError_t kvd_launch_step(kvd_ctx* c, int layer, int n_layers, int step, const void* q, float* out, float* lse, hipStream_t s) {
  using namespace kvd;
  if (n_layers < 1 || n_layers > kStepMaxLayers || n_layers > c->n_sets || layer + n_layers > c->L) return hipErrorInvalidValue;
  StepArgs a;
  const int score_np = c->Nc > 0 ? c->Nc : c->NP;
  a.summ = reinterpret_cast<const uint16_t*>(c->Nc > 0 ? c->centroids : c->summaries) + (size_t)layer * c->U * score_np * kHeadDim;
  a.score_np = score_np;
  a.Nc = c->Nc;
  a.cluster_start = c->Nc > 0 ? c->cluster_start + (size_t)layer * c->U * (c->Nc + 1) : nullptr;
  a.cluster_pages = c->Nc > 0 ? c->cluster_pages + (size_t)layer * c->U * c->NP : nullptr;
  a.q = reinterpret_cast<const uint16_t*>(q);
  a.scores = c->d_scores;
  a.fa = kvd_fast_args(c, layer, step, true, c->d_scores, c->d_sel_pages, c->d_sel_slots, c->d_hit_mask, c->d_evicted,
                       c->d_counts, 0, n_layers);
  a.at = kvd_attn_args(c, layer, q, c->d_sel_pages, c->d_sel_slots, out, lse, 0);
  a.at.fuse_merge = 1;
  a.at.sel_entry = c->d_sel_entry;
  const bool natural = c->tiled == kLayoutNatural;
  const kvd_shape shape = kvd_step_shape(c, n_layers > 1, nullptr, n_layers);
  a.at.S = shape.splits;
  a.at.per_split = (c->k + shape.splits - 1) / shape.splits;
  // (the rule's number of splits, whether it was left to the rule or set: a shape that a context reports gives the same launch
  // when it is set; any other number that the caller has set stays as it is)
  a.at.take = n_layers > 1 && !natural && shape.splits == rule_splits(c, 1) ? kvd_step_take(c, shape.splits, n_layers) : 1;
  a.score_done = c->d_score_done;
  a.error = c->error_dev;
  a.timeline = nullptr;
  a.wait_limit = c->wait_limit_ticks;
  a.scale = c->scale;
  a.n_units = c->U;
  a.u0 = 0;
  // the layers of the launch: layer `layer + i` works in scratch set i
  a.n_layers = n_layers;
  a.layer0 = layer;
  a.Lp = c->Lp;
  a.store_base = c->store_dev;
  a.summ_stride = (long long)c->U * score_np * kHeadDim;
  a.q_stride = (long long)c->B * c->Hq * kHeadDim;
  a.out_stride = (long long)c->B * c->Hq * kHeadDim;
  a.lse_stride = (long long)c->B * c->Hq;
  a.cluster_start_stride = (long long)c->U * (c->Nc + 1);
  a.cluster_pages_stride = (long long)c->U * c->NP;
  a.pool_stride = (long long)c->U * c->Cmax * (long long)c->page_bytes;
  a.store_stride = (long long)c->U * c->NP * (long long)c->page_bytes;
  a.dir_unit_stride = c->U;
  a.dir_slot_stride = (long long)c->U * c->Cmax;
  a.dir_page_stride = (long long)c->U * c->NP;
  for (int i = 0; i < kStepMaxLayers; ++i) {
    const kvd_scratch x = kvd_scratch_set(c, i < n_layers ? i : 0);
    StepLayerSet& d = a.sets[i];
    d.scores = x.scores; d.sel_pages = x.sel_pages; d.sel_slots = x.sel_slots; d.hit_mask = x.hit_mask; d.evicted = x.evicted;
    d.counts = x.counts; d.miss_list = x.miss_list; d.miss_count = x.miss_count; d.part_acc = x.part_acc; d.part_ml = x.part_ml;
    d.attn_ticket = x.attn_ticket; d.score_done = x.score_done; d.sel_entry = x.sel_entry;
  }
  if (n_layers == 1) {
    // (a single layer works in the context's current set, whichever that is)
    StepLayerSet& d = a.sets[0];
    d.scores = c->d_scores; d.sel_pages = c->d_sel_pages; d.sel_slots = c->d_sel_slots; d.hit_mask = c->d_hit_mask;
    d.evicted = c->d_evicted; d.counts = c->d_counts; d.miss_list = c->d_miss_list; d.miss_count = c->d_miss_count;
    d.part_acc = c->d_part_acc; d.part_ml = c->d_part_ml; d.attn_ticket = c->d_attn_ticket; d.score_done = c->d_score_done;
    d.sel_entry = c->d_sel_entry;
  }
  const int chunk_pages = kStepThreads;                // a scoring chunk: every wave 64 pages x passes
  a.passes = shape.passes;
  a.n_score = shape.n_score;
  a.groups = shape.groups;
  a.group_units = (c->U + shape.groups - 1) / shape.groups;
  a.chunks = (score_np + chunk_pages * a.passes - 1) / (chunk_pages * a.passes);
  const int attn_wgs = (shape.splits + a.at.take - 1) / a.at.take, n_stages = n_layers * a.groups;
  a.tail_stages = kvd_step_tail_layers(shape.splits, a.at.take, n_layers) * a.groups;
  const int n_blocks = n_stages * (a.n_score + a.group_units) +
                       a.group_units * ((n_stages - a.tail_stages) * attn_wgs + a.tail_stages * shape.splits);
  c->tl_workgroups = n_blocks;
  if (c->profiling == 2 && n_blocks <= KVD_TIMELINE_MAX) a.timeline = c->d_timeline;
  const int ipt = (c->NP + chunk_pages - 1) / chunk_pages;
  auto launch = [&](auto bf16, auto layout) {
    if (n_layers > 1) launch_step<decltype(bf16)::value, decltype(layout)::value, true>(ipt, a, n_blocks, s);
    else launch_step<decltype(bf16)::value, decltype(layout)::value, false>(ipt, a, n_blocks, s);
  };
  auto by_layout = [&](auto bf16) {
    if (c->tiled == kLayoutPacked) launch(bf16, std::integral_constant<int, kLayoutPacked>());
    else if (c->tiled == kLayoutTiles) launch(bf16, std::integral_constant<int, kLayoutTiles>());
    else launch(bf16, std::integral_constant<int, kLayoutNatural>());
  };
  if (c->bf16) by_layout(std::true_type());
  else by_layout(std::false_type());
  return hipGetLastError();
}
