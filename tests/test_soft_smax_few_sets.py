"""Where the softmax adjoint keeps a rule set's state in LDS
(paper_2406_01821_amd/csrc/soft_plan.h), on the host: few rule sets of many
classes, timed both ways."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include "soft_plan.h"
using namespace aerl;
int main() {
  int n, nf, nc, sets, rules, conds;
  while (std::scanf("%d %d %d %d %d %d", &n, &nf, &nc, &sets, &rules, &conds) == 6) {
    DatasetRec ds;
    ds.n = n;
    ds.nf = nf;
    ds.nc = nc;
    for (int c = 0; c < nc; ++c) ds.n_tiles += ds.region_tiles[c] = (n / nc + AERL_TILE - 1) / AERL_TILE;
    PopRec pop;
    pop.nf = nf;
    pop.n_sets = sets;
    pop.n_rules = sets * rules;
    pop.n_conds = sets * conds;
    pop.max_rules = rules;
    pop.max_rule_conds = 2;
    pop.max_set_conds = conds;
    const SoftPlan p = plan_smax_backward(ds, pop);
    std::printf("%d %d\n", (int)p.reg, p.lds <= kDynLdsMax);
  }
}
"""


@pytest.mark.parametrize("shape,private", [
    # samples, features, classes, rule sets, rules, conditions per set: us with private memory, with LDS
    ((2081, 20, 12, 1, 33, 50), False),    # 205, 160
    ((9000, 20, 12, 2, 12, 18), False),    # 88, 75
    ((500, 20, 12, 1, 33, 50), True),      # half
    ((2081, 20, 12, 5, 33, 50), True),     # 0.66
    ((2081, 20, 7, 1, 33, 50), True),      # 0.85
    ((20000, 512, 12, 1, 64, 200), True),  # no room in LDS
])
def test_state_of_few_sets(tmp_path, shape, private):
    src, exe = tmp_path / "few.cpp", str(tmp_path / "few")
    src.write_text(MAIN)
    r = subprocess.run(["g++", "-std=c++17", "-O0", "-D__HIP_PLATFORM_AMD__", "-I",
                        os.path.join(ROOT, "paper_2406_01821_amd", "csrc"), "-I",
                        os.path.join(ROOT, "include"), "-isystem", "/opt/rocm/include", str(src),
                        "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], input=" ".join(map(str, shape)), capture_output=True, text=True, timeout=60)
    assert r.stdout.split() == [str(int(private)), "1"]
