// Prints the launch plans of the relaxed path for shapes read from stdin, one
// per line: features, classes, samples, rule sets, rules per set, conditions
// per rule, conditions of the longest set.  Output: S Q blocks-per-CU groups LDS
// and classification of the first-firing adjoint, then of the fine-tuning kernel
// on 256 CUs whether it is used, S, blocks, waves per block and LDS.
#include <cstdio>

#include "soft_plan.h"

int main() {
  using namespace aerl;
  // the moments of a population past 2^30 conditions
  static_assert(sizeof(moment_index(1, 0, 0)) == 8, "64-bit index");
  if (moment_index(1, 1 << 30, (1 << 30) - 1) != (1LL << 31) - 1 ||
      moment_index(1, 0x7fffffff, 0x7ffffffe) != 2LL * 0x7fffffff - 1)
    return 1;
  long long n;
  int nf, nc, sets, rules, conds, longest;
  while (std::scanf("%d %d %lld %d %d %d %d", &nf, &nc, &n, &sets, &rules, &conds, &longest) == 7) {
    DatasetRec ds;
    ds.nf = nf;
    ds.nc = nc;
    ds.n = n;
    for (int c = 0; c < nc; ++c) {
      ds.class_count[c] = n / nc + (c < n % nc);
      ds.region_tile0[c] = (int32_t)ds.n_tiles;
      ds.region_tiles[c] = (int32_t)((ds.class_count[c] + AERL_TILE - 1) / AERL_TILE);
      ds.n_tiles += ds.region_tiles[c];
    }
    ds.n_pad = ds.n_tiles * AERL_TILE;
    PopRec pop;
    pop.nf = nf;
    pop.nc = nc;
    pop.n_sets = sets;
    pop.n_rules = sets * rules;
    pop.n_conds = pop.n_rules * conds;
    pop.max_rules = rules;
    pop.max_rule_conds = conds;
    pop.max_set_conds = longest;
    const SoftPlan p = plan_backward(ds, pop);
    const TuneSetsPlan t = plan_tune_sets(ds, pop, 256);
    std::printf("%d %d %d %d %zu %d %d %d %d %d %zu\n", p.S, p.Q,
                2 * (p.lds + kStaticLds) <= kLdsPerCu ? 2 : 1, p.n_groups, p.lds, (int)p.cls, (int)t.use,
                t.S, t.use ? (sets + t.spb - 1) / t.spb : 0, t.spb * t.n_wt, t.lds);
  }
}
