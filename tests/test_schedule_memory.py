"""CPU test of the schedule builder where device memory runs out (the host code of
schedule.hip with the HIP calls stubbed, tests/host/schedule_memory.cpp): a decode
that can do without the match-search tables is not refused for them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2202_13951_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_schedules_do_without_the_match_tables(tmp_path):
    flags = ["-O1", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    exe = str(tmp_path / "schedule_memory")
    objs = []
    for src, mode in ((os.path.join(CSRC, "schedule.hip"), ["--offload-arch=gfx950"]),
                      (os.path.join(ROOT, "tests", "host", "schedule_memory.cpp"), ["--cuda-host-only", "-x", "hip"])):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, *mode, *flags, "-c", src, "-o", obj], check=True, capture_output=True, timeout=300)
        objs.append(obj)
    subprocess.run([HIPCC, "--offload-arch=gfx950", *objs, "-o", exe], check=True, capture_output=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stderr
