"""The unit of the adjoint's 32-bit sums, on the host (tests/sum_unit_check.cpp):
no coarser, over many bricks and views, than the finest power of two that a
count of every pixel's contributions would allow (which the kernel took before
it bounded that count from the brick's corners), and never so fine that a sum
could overflow."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.parametrize("seed", [3, 20250704])
def test_unit_is_no_coarser_than_an_exact_count_allows(tmp_path, seed):
    exe = str(tmp_path / "sum_unit_check")
    cmd = [HIPCC, "-std=c++17", "-O2", "--offload-arch=gfx950", "--cuda-host-only",
           "-x", "hip", os.path.join(ROOT, "tests", "sum_unit_check.cpp"),
           "-x", "c++", os.path.join(ROOT, "paper_1909_02724_amd", "csrc", "tiles.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe, str(seed), "4000"], capture_output=True, text=True, check=True).stdout
    print(out)
    for line in out.splitlines():
        kind, *fields = line.split()
        s = {k: float(v) for k, v in (f.split("=") for f in fields)}
        assert s["views"] >= 5000 and s["over"] == 0, (kind, s)
        assert s["rms"] <= 100.0, (kind, s)
