"""Launch plans of the relaxed path (paper_2406_01821_amd/csrc/
soft_plan.h), on the host: tests/sched/plan_driver.cpp prints them.  A grid
that fills the GPU keeps the waves of its blocks busy: samples per lane times
waves with a rule set times blocks per CU reaches most of what some
arrangement that fits the LDS reaches; and the fine-tuning kernel is used where
its blocks are resident at once, by LDS and by the waves that its registers
leave a SIMD, or half as many more with rule sets of uneven length."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2406_01821_amd", "csrc")
LDS, STATIC, WAVES = 160 * 1024, 64, 16


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                        os.path.join(ROOT, "include"), "-isystem", "/opt/rocm/include",
                        os.path.join(ROOT, "tests", "sched", "plan_driver.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(shapes):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, s)) for s in shapes),
                           capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    return run


def busiest(nf, cls, per_set, sets):
    best = 0
    for S in (4, 2, 1):
        xs = nf * 256 * S + (8 * nf if cls else 0)
        for per_cu in (1, 2):
            room = LDS // per_cu - STATIC
            if xs + per_set <= room:
                best = max(best, S * per_cu * min(WAVES, sets, (room - xs) // per_set))
    return best


def test_adjoint_blocks_keep_their_waves_busy(plans):
    shapes = [(nf, 2, 262_144, 1024, rules, conds, rules * conds)
              for nf in (8, 30, 64, 65, 90, 128, 129, 200, 250, 300, 310, 318, 319, 360, 450, 512)
              for rules, conds in ((2, 2), (8, 4), (16, 4), (24, 6), (32, 8), (48, 4), (60, 8), (64, 15))]
    for shape, (S, Q, per_cu, groups, lds, cls, *_) in zip(shapes, plans(shapes)):
        nf, _, _, sets, rules, conds, _ = shape
        assert Q >= 1 and lds <= LDS - STATIC, shape
        busy = S * per_cu * min(WAVES, Q)
        assert busy >= 0.45 * busiest(nf, cls, 8 * rules * conds, sets), (shape, S, Q, per_cu)


def test_small_grids_spread_over_the_gpu(plans):
    """Few tiles and rule sets: a block per CU before a second wave per SIMD."""
    for nf in (30, 64, 200, 310):
        (S, Q, per_cu, groups, *_), = plans([(nf, 2, 2500, 100, 24, 6, 144)])
        assert -(-100 // Q) * groups >= 100, (nf, S, Q)


def test_fine_tuning_blocks_are_resident(plans):
    shapes = [(nf, nc, n, sets, 8, 4, longest)
              for nf in (8, 30, 60, 200) for nc, n in ((1, 250), (2, 500), (2, 569), (1, 1000), (1, 2048))
              for sets in (1, 100, 257, 400, 512, 520, 700, 1000, 2000, 4000) for longest in (32, 60)]
    used = 0
    for shape, p in zip(shapes, plans(shapes)):
        use, S, blocks, waves, lds = p[6:]
        if not use:
            continue
        used += 1
        # registers: 85 VGPRs with four samples per lane leave a SIMD five waves,
        # 106 SGPRs seven
        resident = 256 * min(LDS // (lds + STATIC), (5 if S == 4 else 7) // -(-waves // 4), 2)
        uneven = 2 * shape[6] >= 3 * 8 * 4
        assert blocks <= resident * (1.5 if uneven else 1), shape
    assert used > len(shapes) // 3


def test_register_bounds_of_the_fine_tuning_plan():
    from test_kernel_resources import kernels
    found = {n: k for n, k in kernels().items() if "k_tune_sets" in n}
    assert found
    for n, k in found.items():
        waves = 5 if "ILi4E" in n else 7
        assert k[".vgpr_count"] <= 512 // waves // 8 * 8, n  # granules of 8
