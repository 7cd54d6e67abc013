// The work split of a ragged batch: host arithmetic over its items' sizes, no
// device code.
#pragma once

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdint>
#include <vector>

#include "batch.h"

namespace aerl {

// Samples per lane of an item with nf features: the most of {4, 2, 1} whose
// 64-lane tile of all features fits the budget.
inline int batch_samples_per_lane(int32_t nf, size_t tile_budget) {
  int s = 4;
  while (s > 1 && (size_t)nf * 256 * s > tile_budget) s >>= 1;
  return s;
}

namespace {

struct ItemView {
  const DatasetRec *ds;
  const PopRec *pop;
  const aerl_batch_item *item;
};

int32_t sets_per_item(const DatasetRec &ds, int32_t n_sets, const BatchSplit &sp) {
  const int32_t Q = sp.Q;
  const size_t tile_bytes = (size_t)ds.nf * 64 * batch_samples_per_lane(ds.nf, sp.tile_budget) * 4;
  const int32_t q_fit =
      (int32_t)std::min<size_t>((kBatchLdsMax - tile_bytes - (size_t)ds.nf * 8 - 4) /
                                    ((size_t)std::max(hard_counters_per_set(ds.nc), 1) * 2),
                                1 << 20);
  return std::max(1, std::min({Q, n_sets, q_fit}));
}

// Estimated time (us) of a batch under a split.  A work item costs its pull,
// records and flush (10), and per wave tile the staging (KiB) and the walks of
// its 16 waves at two blocks per CU, whose length grows with the conditions of
// a rule set.  The list is pulled longest first, so it ends a part of a mean
// item after an even share of the work, or with its longest items.
double split_cost(const std::vector<ItemView> &v, const BatchSplit &sp, int n_cu) {
  double total = 0, longest = 0;
  int64_t n = 0;
  size_t lds = 0;
  for (const auto &e : v) {
    const DatasetRec &ds = *e.ds;
    const int32_t sets = e.pop->n_sets;
    if (sets <= 0 || ds.n_tiles == 0) continue;
    const int S = batch_samples_per_lane(ds.nf, sp.tile_budget);
    const int32_t q = sets_per_item(ds, sets, sp);
    lds = std::max(lds, hard_block_lds(ds.nf, S, q, ds.nc));
    const double stage = 0.077 * (ds.nf * 0.25 * S);
    const double visit = (S == 4 ? 2.49 : S == 2 ? 1.74 : 1.38) *
                         (0.673 + 0.327 / 60 * ((double)e.pop->n_conds / sets));
    const auto cost = [&](int32_t q1, int32_t tiles) {
      return 10 + tiles * (4 / S) * (stage + std::max(1.0, q1 / 16.0 + 0.73) * visit);
    };
    const auto add = [&](int64_t groups, int32_t tiles) {
      if (groups == 0 || tiles == 0) return;
      total += groups * (double)(sets / q) * cost(q, tiles);
      if (sets % q) total += groups * cost(sets % q, tiles);
      n += groups * ((sets + q - 1) / q);
      longest = std::max(longest, cost(q, tiles));
    };
    for (int c = 0; c < ds.nc; ++c) {
      add(ds.region_tiles[c] / sp.TG, sp.TG);
      add(1, ds.region_tiles[c] % sp.TG);
    }
  }
  const double slots = (double)n_cu * (2 * (lds + kStaticLds) <= kLdsPerCu ? 2 : 1);
  if ((double)n <= slots) return longest * ((double)n <= slots / 2 ? 0.86 : 1.0);  // alone on a CU
  const double share = total / slots;
  return std::max(share + 0.427 * total / n, std::pow(std::pow(share, 2.53) + std::pow(longest, 2.53), 1 / 2.53));
}

// The split that split_cost finds cheapest, of 32 to 512 rule sets by one or
// two tiles (these at 1.04 of their estimate), at the fields that are not given
// (> 0); unless that is below 0.92 of 512 sets by one tile, these, or by two
// where that is the cheaper one.  Fitted to 150 batches of 3 to 64 runs of 300 to
// 200 000 rows, each timed over its splits (profiles/batch_split_timings.txt):
// the choice is 1.1% slower than the best one on average and takes 0.76 of 512
// sets by one tile, at most 1.03 on any; over 110 others 1.6%, 0.78 and 1.08,
// beyond 1.02 on four.  Without the conditions and the margins those were up to
// 1.20, beyond 1.02 on ten (27 runs of 1000 to 30 000 rows with 8 to 128 sets 60
// us against 51).
std::array<int32_t, 3> default_split(const std::vector<ItemView> &v, int n_cu, const aerl_batch_cfg *cfg) {
  const int32_t kib = cfg && cfg->tile_kib > 0 ? cfg->tile_kib : 64;
  const int32_t sets = cfg && cfg->sets_per_task > 0 ? cfg->sets_per_task : 0;
  const int32_t tiles = cfg && cfg->tiles_per_task > 0 ? cfg->tiles_per_task : 0;
  std::array<int32_t, 3> best = {512, 1, kib};
  if (kib > (int32_t)(kBatchLdsMax / 1024)) return best;  // refused by the caller
  const auto cost = [&](int32_t q, int32_t tg) {
    BatchSplit sp;
    sp.Q = sets ? sets : q;
    sp.TG = tiles ? tiles : tg;
    sp.tile_budget = (size_t)kib * 1024;
    return split_cost(v, sp, n_cu);
  };
  const double plain = cost(512, 1), plain2 = cost(512, 2);
  double best_cost = 0.92 * plain;
  if (plain2 < plain) best[1] = 2;
  for (int32_t q = 512; q >= 32; q /= 2) {
    for (int32_t tg = 1; tg <= 2; ++tg) {
      const double c = (tg == 2 ? 1.04 : 1.0) * cost(q, tg);
      if (c < best_cost) {
        best_cost = c;
        best = {q, tg, kib};
      }
    }
  }
  if (sets) best[0] = sets;
  if (tiles) best[1] = tiles;
  return best;
}

}  // namespace

}  // namespace aerl
