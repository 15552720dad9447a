"""The back-projector's launch shapes, the rows its row walk reads, and the
adjoint's walk and fixed-point bounds.

A block of slices whose column drifts by less than a pixel against rows one
apart takes all its taps from consecutive staged rows at fixed offsets from
the block's first row, so a first row that is off by one, or a tile that is a
row short, would give wrong values without a fault. tests/row_walk_check.cpp
builds the kernels' brick setup, FP32 column arithmetic and launch rules for
the host and walks seeded random geometries: mirrored and plain runs, all
brick heights, one to four groups of threads a brick."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def walk_exe(tmp_path_factory):
    exe = tmp_path_factory.mktemp("walk") / "row_walk_check"
    cmd = [HIPCC, "-std=c++17", "-O2", "--offload-arch=gfx950", "--cuda-host-only",
           "-x", "hip", os.path.join(ROOT, "tests", "row_walk_check.cpp"),
           "-x", "c++", os.path.join(ROOT, "paper_1909_02724_amd", "csrc", "tiles.cpp"),
           "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("seed", [5, 20250311])
def test_row_walk_stays_inside_the_tile(walk_exe, seed):
    out = subprocess.run([str(walk_exe), str(seed), "4000"], capture_output=True, text=True,
                         check=True).stdout
    print(out)
    for line in out.splitlines():
        kind, *fields = line.split()
        s = {k: int(v) for k, v in (f.split("=") for f in fields)}
        # Every brick height, several groups and enough walked columns occur.
        assert s["walked"] >= 500 and s["columns"] >= 500_000, (kind, s)
        assert min(s["np16"], s["np8"], s["np4"], s["groups"]) >= 50, (kind, s)
        # The adjoint: walks in its tile, pixels within the bound, the bound not wide.
        assert s["adj_walked"] >= 1000 and s["adj_wide"] >= 20 and s["adj_slack"] <= 200, (kind, s)
        assert s["adj_low"] == s["adj_high"] == s["adj_over"] == 0, (kind, s)
        assert s["bad_shape"] == s["load"] == s["low"] == s["high"] == s["offset"] == 0, (kind, s)
