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
  return 0;
}
