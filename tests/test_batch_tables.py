"""Device tables of the batched paths at sizes past 32 bits and the split that
a batch gets, on the host: tests/sched/tables_driver.cpp checks the arithmetic
of csrc/batch.h and csrc/batch_plan.h."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tables_and_splits(tmp_path):
    exe = str(tmp_path / "tables_driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I",
                        os.path.join(ROOT, "paper_2406_01821_amd", "csrc"), "-I",
                        os.path.join(ROOT, "include"), "-isystem", "/opt/rocm/include",
                        os.path.join(ROOT, "tests", "sched", "tables_driver.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
