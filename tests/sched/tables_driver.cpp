// Checks the batched paths' device tables (csrc/batch.h) at sizes that no
// test can allocate.  Exits non-zero at the first violation.
#include <cstdio>

#include "batch.h"

using namespace aerl;

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
  return 0;
}
