// Checks the batched paths' device tables (csrc/batch.h) at sizes that no
// test can allocate, and the split that a batch gets (csrc/batch_plan.h).
// Exits non-zero at the first violation.
#include <climits>
#include <cstdio>

#include "batch_plan.h"

using namespace aerl;

struct Run {
  int n, nf, nc, sets, conds;
};
static std::array<int32_t, 3> split_of(const std::vector<Run> &runs, const aerl_batch_cfg *cfg = nullptr) {
  std::vector<DatasetRec> ds(runs.size());
  std::vector<PopRec> pops(runs.size());
  std::vector<ItemView> v;
  for (size_t i = 0; i < runs.size(); ++i) {
    DatasetRec &d = ds[i];
    d.n = runs[i].n;
    d.nf = runs[i].nf;
    d.nc = runs[i].nc;
    for (int c = 0; c < d.nc; ++c) {
      d.region_tiles[c] = (runs[i].n / d.nc + AERL_TILE - 1) / AERL_TILE;
      d.n_tiles += d.region_tiles[c];
    }
    pops[i].n_sets = runs[i].sets;
    pops[i].n_conds = runs[i].conds;
    v.push_back({&d, &pops[i], nullptr});
  }
  return default_split(v, 256, cfg);
}

int main() {
  // A prediction task finds its population's heads behind 2^31 records and as
  // many soft words.
  PackedLayout L{};
  L.hconds_off = 4096;
  L.heads_off = L.hconds_off + ((size_t)20 << 31) + 256;
  PredictTask t{};
  t.heads = heads_from_conds(L);
  const size_t bytes = (size_t)((reinterpret_cast<uintptr_t>((const uint4 *)0 + t.heads)));
  if (bytes != L.heads_off - L.hconds_off) return std::puts("heads"), 1;
  // A batch is refused where its plain split has too many work items, as
  // before there was a planned one, and takes it where only the planned one has.
  const BatchSplit plain{512, 1, 65536}, planned{512, 2, 65536};
  BatchSplit sp = planned;
  if (settle_split(INT32_MAX / 2, plain, (int64_t)INT32_MAX + 1, &sp)) return std::puts("refusal"), 1;
  if (!settle_split((int64_t)INT32_MAX + 1, plain, INT32_MAX, &sp) || sp.TG != 1)
    return std::puts("plain"), 1;
  sp = planned;
  if (!settle_split(INT32_MAX, plain, INT32_MAX, &sp) || sp.TG != 2) return std::puts("planned"), 1;
  // Few runs of small populations that fill the GPU keep 512 sets by one tile
  // (58 us timed; 64 by two tiles 64, 32 by one 82), runs of few tiles split
  // their long populations (94 us; 32 by one tile 39), and given fields stay.
  const std::vector<Run> filled = {{111487, 47, 4, 77, 6128}, {3350, 118, 4, 21, 1323}, {15083, 99, 3, 16, 1116}};
  const std::vector<Run> few = {{2824, 215, 2, 297, 5919}, {433, 97, 3, 16, 218}, {699, 171, 3, 37, 722}};
  std::array<int32_t, 3> got = split_of(filled);
  if (got[0] != 512 || got[1] != 1 || got[2] != 64) return std::printf("filled %d x %d\n", got[0], got[1]), 1;
  got = split_of(few);
  if (got[0] > 64 || got[1] != 1) return std::printf("few %d x %d\n", got[0], got[1]), 1;
  const aerl_batch_cfg given{256, 2, 80};
  got = split_of(few, &given);
  if (got[0] != 256 || got[1] != 2 || got[2] != 80) return std::puts("given"), 1;
  return 0;
}
