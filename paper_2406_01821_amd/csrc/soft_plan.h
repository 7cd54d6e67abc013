// Launch plans of the relaxed path's kernels: host arithmetic over a table's
// and a population's sizes, no device code.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.h"

namespace aerl {

namespace {

constexpr int kSoftBlock = 512;  // threads of a forward block
// 16 waves of an adjoint block share its tile and accumulators in LDS, so the
// LDS limit still leaves 32 waves per CU.
constexpr int kBwdRegBlock = 1024;
// Waves per block of the LDS-state adjoint kernels: up to this many, fewer for
// rule sets whose per-wave state ([R][2][64] floats) would not fit.
constexpr int kBwdWaves = 8, kSmaxBwdWaves = 4;
constexpr int kProdMaxConds = 60;  // most conditions of a rule in product form
// Most rules whose state the adjoints keep in private memory, and the bound of
// the variants for shorter rule sets.  The runtime reserves a kernel's private
// memory for every wave that the GPU can hold, whatever the population: 32 rules
// take 1040 bytes per lane (540 MB) with four samples, 64 rules 2080 (1.1 GB),
// under the softmax head 1560 and 3100.  A launch that asks for less than one
// before it keeps the larger one's stride between waves, which makes it slower
// (53,348 x 26, 135 sets of 13 rules, after sets of 24: 454 us in a variant for
// 16 rules, 430 in this one, 420 before either): so the line is above the rules
// that populations usually have, and not below it.
constexpr int kRegRules = 64, kFewRules = 32;

struct SoftPlan {
  int S, Q, TG, n_groups;
  bool reg;   // backward: per-rule state in private memory, else in LDS
  bool cls;   // tiles classify the conditions
  int waves;  // LDS-state kernels: waves per block
  size_t lds;
};

// Tables of fewer tiles than this do not classify: a tile spans most of each
// column's range and little is decided (adjoint of 100 rule sets on 569 samples
// 46.0 us with and 45.0 us without it, on 4000 samples 47.5 and 46.8 us).
constexpr int64_t kClassifyTiles = 16;

// Feature tile and, where tiles classify, its extremes.
size_t tile_lds(int nf, int S, bool cls) {
  return (size_t)nf * 64 * S * sizeof(float) + (cls ? (size_t)nf * 2 * sizeof(float) : 0);
}

// Waves and rule-set chunk of an LDS-state adjoint kernel (tile xs bytes,
// per_set accumulator bytes, per_wave state bytes): the most waves (at most
// max_waves) that fit with one rule set per chunk, then the largest chunk
// (at most max_q sets) that fits.
void lds_state_plan(SoftPlan &p, size_t xs, size_t per_set, size_t per_wave, int max_waves,
                    int max_q, int n_sets) {
  p.waves = max_waves;
  while (p.waves > 1 && xs + per_set + p.waves * per_wave > kDynLdsMax) p.waves >>= 1;
  p.Q = std::max(1, std::min(n_sets, max_q));
  while (p.Q > 1 && xs + p.Q * per_set + p.waves * per_wave > kDynLdsMax) p.Q >>= 1;
  p.lds = xs + (size_t)p.Q * per_set + p.waves * per_wave;
}

int64_t count_groups(const DatasetRec &ds, int tg) {
  int64_t g = 0;
  for (int c = 0; c < ds.nc; ++c) g += (ds.region_tiles[c] + tg - 1) / tg;
  return g;
}

// Tiles per block group.  A launch has (set chunks) x (tile groups) blocks;
// the fewest groups that still give about `target` blocks (measured on the
// 262,144 x 32, 1024-set workload: a forward grid of one wave of blocks,
// 64 groups, runs 10.9 ms, 1024 groups 6.9 ms, as its blocks no longer stage
// their tiles in step; the adjoint runs 22.8 ms at 64 groups and 20.8 ms at
// 256), then fewer while the per-group partial sums (bytes_per_group each)
// exceed max_bytes.
int tiles_per_group(const DatasetRec &ds, int64_t chunks, int64_t target, size_t bytes_per_group,
                    size_t max_bytes) {
  int32_t widest = 1;
  for (int c = 0; c < ds.nc; ++c) widest = std::max(widest, ds.region_tiles[c]);
  const int64_t need = (target + std::max<int64_t>(chunks, 1) - 1) / std::max<int64_t>(chunks, 1);
  int tg = 1;
  while (tg < widest && count_groups(ds, 2 * tg) >= need) tg *= 2;
  while (tg < widest && (size_t)count_groups(ds, tg) * bytes_per_group > max_bytes) tg *= 2;
  return tg;
}
// Forward: 16 blocks per block slot (four 512-thread blocks per CU on 256
// CUs), fp64 partials of at most 8 MiB (half the no-allocation scratch).
constexpr int64_t kFwdTargetBlocks = 16384;
constexpr size_t kFwdPartMax = (size_t)8 << 20;
// Backward: 8 blocks per slot (two 1024-thread blocks per CU), partial
// gradients of at most 1 GiB.
constexpr int64_t kBwdTargetBlocks = 4096;
constexpr size_t kBwdPartMax = (size_t)1 << 30;

// Rule sets per block: 64, or fewer, down to one per wave (min_q), while
// the grid (set chunks x `groups` tile groups) stays under `target` blocks,
// so that a small workload spreads over more CUs instead of walking several
// rule sets per wave on a few of them.
int sets_per_block(int n_sets, int64_t groups, int64_t target, int min_q) {
  int q = std::max(1, std::min(n_sets, 64));
  while (q / 2 >= min_q && (int64_t)((n_sets + q - 1) / q) * groups < target) q /= 2;
  return q;
}

// Whether a forward pass classifies.  Per tile it costs the extremes (a pass
// over nf rows) and per rule set and 64 conditions a classification, and it
// saves a share of the sweep that grows with the conditions of a rule (one out
// of reach drops the rule).  Of 439 shapes timed both ways the line falls where
// a launch has 600,000 (tile, condition) pairs (60,000 x 32, 40 rule sets of 8
// x 4 conditions: 45 us, plain 55; 262,144 x 32 x 1024 of 16 x 4: 2.8 and 6.5
// ms), unless its rules hold one condition (253,611 x 53 x 1448 of 8 x 1: 4.1 and
// 3.9 ms) or, short of four, a block sweeps too few for the features that it looks
// over (96,217 x 32 x 533 of 2 x 2: 276 and 237 us); on wider tables, whose tiles
// are half or a quarter as long for the same extremes, only with enough rule sets
// per block (30,000 x 90 x 200 of 8-16 x 2-5: 190 and 180 us).  Smaller launches
// gain on narrow tables alone (40,000 x 60, 16 rule sets: 37 and 28 us; 20,011 x
// 45, 150 of 1-24 x 1-6: 98 and 104), by rules of more than two conditions or
// many of them per staged value (23,741 x 38, 32 of 24 x 2: 52 and 49 us; 32,803
// x 5, 3 of 50 x 1-2: 62 and 57).  Rules of more than 64 conditions are swept in
// full in any case.
bool forward_classifies(const DatasetRec &ds, const PopRec &pop, int sets_per_block) {
  if (ds.n_tiles < kClassifyTiles || pop.n_conds > 72LL * pop.n_rules) return false;
  const double per_block = (double)sets_per_block * pop.n_conds / std::max(pop.n_sets, 1);
  const double per_rule = (double)pop.n_conds / std::max(pop.n_rules, 1);
  if ((double)ds.n_tiles * pop.n_conds >= 6e5)
    return per_rule >= 1.3 && per_block >= (ds.nf > 64 ? 8.0 : per_rule < 4 ? 3.5 : 0.0) * ds.nf;
  return ds.n_tiles >= 24 && ds.nf <= 52 && per_block >= 200 &&
         (per_rule >= 2.5 || (per_rule >= 1.6 && per_block >= 12.0 * ds.nf));
}

SoftPlan plan_forward(const DatasetRec &ds, const PopRec &pop) {
  SoftPlan p{};
  p.Q = sets_per_block(pop.n_sets, count_groups(ds, 1), kFwdTargetBlocks, kSoftBlock / 64);
  p.cls = forward_classifies(ds, pop, p.Q);
  // four samples per lane; where tiles classify, while three blocks fit a CU
  // (60,000 x 60, where two would: 611 us, with two samples per lane 560 us)
  p.S = !p.cls || tile_lds(ds.nf, 4, true) <= kLdsPerCu / 3 ? 4 : 2;
  while (p.S > 1 && (size_t)ds.nf * 256 * p.S > 64 * 1024) p.S >>= 1;
  p.TG = tiles_per_group(ds, (pop.n_sets + p.Q - 1) / p.Q, kFwdTargetBlocks,
                         (size_t)std::max(pop.n_sets, 1) * sizeof(double), kFwdPartMax);
  p.n_groups = (int)count_groups(ds, p.TG);
  p.lds = tile_lds(ds.nf, p.S, p.cls) + (size_t)p.Q * 8;
  return p;
}

// (Tile, condition) pairs from which the first-firing adjoint classifies: below,
// its launch is a few waves' latency, which the extremes and the classification
// add to (40,000 x 60, 4 rule sets of 8 x 4 conditions, 20,000 pairs: 45.2 and
// 42.4 us; 3 to 10 thousand pairs 4% on average, 40 to 80 thousand -2%).  The
// softmax adjoint, whose reductions it spares as well, gains from the first.
constexpr double kBwdClassifyPairs = 4e4;

// Estimated time (us) of a private-memory adjoint with S samples per lane, Q
// rule sets per block and per_cu blocks on a CU, of LDS tiles of xs bytes.  A
// block stages its tile 4 / S times (latency, then KiB) and its 16 waves share
// its rule sets, the longest one last.  A visit of one rule set has a latency
// of its own and shares its SIMD with the waves beside it; two samples per lane
// take 0.66 and one 0.58 of its time with four.  Up to one round of blocks a
// launch lasts as long as its fullest CU, past it a part of a round more than
// an even share.  Fitted to 258 shapes of 8 to 510 features, 1 to 962 rule sets
// and 4 to 700 conditions per set on 300 to 262,144 rows, each timed under 16 to
// 20 plans: the choice is 0.9% slower than the best of them on average, and
// takes 0.65 times as long as samples fixed by the width and two blocks per CU
// whatever those left room for.
double adjoint_cost(const DatasetRec &ds, const PopRec &pop, int64_t groups, int TG, int S, int Q, int per_cu,
                    size_t xs) {
  constexpr int kCu = 256, kWaves = kBwdRegBlock / 64;
  const double sets = std::max(pop.n_sets, 1);
  const double blocks = std::ceil(sets / Q) * (double)groups;
  const double on_cu = std::min<double>(per_cu, std::max(1.0, std::ceil(blocks / kCu)));
  const double waves = on_cu * std::min(Q, kWaves) / 4;  // per SIMD
  const double conds = std::max(1.0, pop.n_conds / sets), rules = pop.n_rules / sets;
  const double visit = (0.16 * conds + 0.23 * rules) * (S == 4 ? 1.0 : S == 2 ? 0.66 : 0.58) * (6.7 + waves);
  const double turns = std::max(1.0, (double)Q / kWaves) + 0.26 * (pop.max_set_conds / conds - 1.0) + 0.085;
  const double block = TG * (4 / S) * (2.5 + 0.055 * ((double)xs / 1024) + turns * visit);
  const double rounds = blocks / (kCu * on_cu);
  return block * (rounds <= 1 ? 1.0 : rounds + 0.27);
}

// Plan of an LDS-state adjoint kernel (one sample per lane).
SoftPlan plan_lds_state(const DatasetRec &ds, const PopRec &pop, SoftPlan p, int max_waves) {
  p.reg = false;
  p.S = 1;
  lds_state_plan(p, (size_t)ds.nf * 64 * 4, (size_t)std::max(pop.max_set_conds, 1) * 2 * 4,
                 (size_t)std::max(pop.max_rules, 1) * 128 * 4, max_waves, 16, pop.n_sets);
  return p;
}

// Backward: per-rule state in private memory up to kRegRules rules, else in
// LDS.  Samples per lane (at most max_s) and rule sets per block (64, halved
// down to 4, or as many as the LDS has room for at one or two blocks per CU)
// are chosen together, by adjoint_cost: with the samples fixed first and the
// sets by what two blocks per CU left room for, blocks of wide tables or long
// rule sets held fewer rule sets than waves (16,000 x 310, 256 sets of 8 x 4
// conditions: one, 4354 us; now 64 in one block per CU, 0.4 ms).
SoftPlan plan_adjoint(const DatasetRec &ds, const PopRec &pop, int max_s, int lds_waves,
                      double classify_pairs) {
  SoftPlan p{};
  const size_t per_set = (size_t)std::max(pop.max_set_conds, 1) * 2 * 4;
  p.TG = tiles_per_group(ds, (pop.n_sets + 63) / 64, kBwdTargetBlocks,
                         (size_t)std::max(pop.n_conds, 1) * 2 * sizeof(float), kBwdPartMax);
  p.n_groups = (int)count_groups(ds, p.TG);
  if (pop.max_rules > kRegRules) return plan_lds_state(ds, pop, p, lds_waves);
  p.reg = true;
  p.cls = ds.n_tiles >= kClassifyTiles && (double)ds.n_tiles * pop.n_conds >= classify_pairs;
  const int most = std::max(1, std::min(pop.n_sets, 64));
  double best = 0;
  for (int S = max_s; S >= 1; S >>= 1) {
    const size_t xs = tile_lds(ds.nf, S, p.cls);
    for (size_t room : {kLdsPerCu / 2 - kStaticLds, kDynLdsMax}) {
      if (xs + per_set > room) continue;
      const int fit = (int)std::min<size_t>(most, (room - xs) / per_set);
      for (int q = 64; q >= 4; q >>= 1) {
        const int Q = std::min(q, fit);
        const size_t lds = xs + (size_t)Q * per_set;
        const int per_cu = 2 * (lds + kStaticLds) <= kLdsPerCu ? 2 : 1;
        const double cost = adjoint_cost(ds, pop, p.n_groups, p.TG, S, Q, per_cu, xs);
        if (p.Q == 0 || cost < best) {
          best = cost;
          p.S = S;
          p.Q = Q;
          p.lds = lds;
        }
      }
    }
  }
  if (p.Q == 0) p.lds = kDynLdsMax + 1;  // no plan fits: refused
  return p;
}
SoftPlan plan_backward(const DatasetRec &ds, const PopRec &pop) {
  return plan_adjoint(ds, pop, 4, kBwdWaves, kBwdClassifyPairs);
}

int smax_nc(int nc) { return nc <= 2 ? 2 : nc <= 4 ? 4 : nc <= 8 ? 8 : 16; }

// One or two rule sets of more than eight classes are a wave or two per block,
// which one sample per lane leaves waiting for their private memory: their state
// is kept in LDS where most wave tiles have samples (12 classes, one set of 33
// rules: 2081 samples 160 us against 205, 9000 169 and 198; 500 samples 1.0
// against 0.5, five sets 1.0 and 0.7 at any size).
SoftPlan plan_smax_backward(const DatasetRec &ds, const PopRec &pop) {
  const SoftPlan p = plan_adjoint(ds, pop, std::min(4, 16 / smax_nc(ds.nc)), kSmaxBwdWaves, 0);
  if (p.reg && smax_nc(ds.nc) > 8 && pop.n_sets <= 2 && ds.n >= 128LL * ds.nc) {
    SoftPlan own = p;
    own.cls = false;
    own = plan_lds_state(ds, pop, own, kSmaxBwdWaves);
    if (own.lds <= kDynLdsMax) return own;
  }
  return p;
}

// Same groups (and so the same workspace) as the first-firing forward.  Four
// samples per lane up to four classes and while three blocks fit a CU
// (20,011 x 45, 150 mixed rule sets: 94 us, with two samples 111 us; 60,000 x
// 60, where two would fit: 576 and 517 us), but not in a plain sweep of rules
// past the product form, whose registers would leave four waves per SIMD; else
// two, one where two do not fit.
SoftPlan plan_smax_forward(const DatasetRec &ds, const PopRec &pop) {
  SoftPlan p = plan_forward(ds, pop);
  const bool wide = p.cls || pop.max_rule_conds <= kProdMaxConds;
  p.S = smax_nc(ds.nc) <= 4 && wide && tile_lds(ds.nf, 4, p.cls) <= kLdsPerCu / 3 ? 4 : 2;
  if (tile_lds(ds.nf, p.S, p.cls) + (size_t)p.Q * 8 > kDynLdsMax) p.S = 1;
  p.lds = tile_lds(ds.nf, p.S, p.cls) + (size_t)p.Q * 8;
  return p;
}

// k_tune_sets takes tables of up to kTuneSetsTiles tiles, each wave tile with
// a wave of its own in a block, and populations whose blocks are resident at
// once, by LDS and by waves, with the fewest samples per lane that leave a
// block per CU (latency: 569 samples, 100 rule sets, 50 epochs: one 0.71, two
// 0.84, four 1.20 ms).  On more tiles a rule set outgrows one CU: 1500 samples
// 1.15 against 2.47 ms, but 4000 samples 2.40 against 2.18, 3000 x 60 with 400
// rule sets 5.2 against 4.1 ms.  Blocks past those resident start where the
// first ones end: up to half as many more still pay where rule sets differ in
// length, so that some end early (2048 x 30, 10 epochs: 520 rule sets of 1-8 x
// 1-4 conditions 0.51 ms against the adjoint kernel's 0.68, 1000 of them 0.79
// against 0.71; 2000 x 8, 700 rule sets of 8 x 4 0.91 against 0.87).
constexpr int64_t kTuneSetsTiles = 8;
constexpr int kTuneSetsWaves = 16;
struct TuneSetsPlan {
  bool use, x_lds;
  int S, n_wt, spb;
  size_t lds;
};
// Waves of k_tune_sets that one SIMD holds, by its registers (S = 4: up to 87
// VGPRs; all: 106 SGPRs).
int tune_sets_waves_per_simd(int S) { return S == 4 ? 5 : 7; }

TuneSetsPlan plan_tune_sets(const DatasetRec &ds, const PopRec &pop, int n_cu) {
  TuneSetsPlan best{};
  const bool uneven = 2LL * pop.max_set_conds * pop.n_sets >= 3LL * pop.n_conds;
  if (pop.max_rules > kRegRules || ds.n_tiles < 1 || ds.n_tiles > kTuneSetsTiles || pop.n_conds < 1)
    return best;
  for (int S = 4; S >= 1; S >>= 1) {
    if (S > 1 && (size_t)ds.nf * 256 * S > 64 * 1024) continue;  // the adjoint's bound
    TuneSetsPlan p{};
    const int64_t n_wt = ds.n_tiles * (AERL_TILE / (64 * S));
    if (n_wt > kTuneSetsWaves) break;
    p.S = S;
    p.n_wt = (int)n_wt;
    // rule sets per block: one, or more until there is a block per CU
    p.spb = 1;
    while ((p.spb + 1) * p.n_wt <= kTuneSetsWaves && (pop.n_sets + p.spb - 1) / p.spb > n_cu) ++p.spb;
    const size_t waves = (size_t)p.spb * p.n_wt;
    const size_t own = (waves + 1) / 2 * 2 * sizeof(double) +
                       (size_t)std::max(pop.max_set_conds, 1) * (p.spb * 32 + waves * 2 * sizeof(float));
    const size_t table = (size_t)ds.nf * (size_t)ds.n_pad * sizeof(float);
    p.x_lds = table + own <= kDynLdsMax;
    p.lds = own + (p.x_lds ? table : 0);
    const int64_t blocks = (pop.n_sets + p.spb - 1) / p.spb;
    const int64_t by_lds = (int64_t)(kLdsPerCu / (p.lds + kStaticLds));
    const int64_t by_waves = tune_sets_waves_per_simd(S) / (int64_t)((waves + 3) / 4);
    const int64_t resident = std::min<int64_t>({by_lds, by_waves, 2}) * n_cu;
    p.use = blocks <= resident || (uneven && 2 * blocks <= 3 * resident);
    if (p.use && (!best.use || blocks <= n_cu)) best = p;
  }
  return best;
}

// Where an update's parameter k (0 the coefficient, 1 the right-hand operand)
// of condition j has its moment: [2][n_conds], past 2^31 entries from 2^30
// conditions on.
__host__ __device__ inline int64_t moment_index(int k, int32_t n_conds, int32_t j) {
  return (int64_t)k * n_conds + j;
}

}  // namespace

}  // namespace aerl
