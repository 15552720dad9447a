"""The tile entries that the staged back-projector reads, on the host, in every
launch shape, with and without a row walk (tests/staged_rows_check.cpp), also
under the address and undefined-behaviour sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
SAN = [f for s in ("address", "undefined") for f in ("-Xarch_host", f"-fsanitize={s}")]


@pytest.mark.parametrize("seed, count, flags", [(11, 4000, []), (20250612, 4000, []), (7, 300, SAN)],
                         ids=["a", "b", "sanitized"])
def test_columns_stay_inside_the_tile(tmp_path, seed, count, flags):
    exe = str(tmp_path / "staged_rows_check")
    cmd = [HIPCC, "-std=c++17", "-O2", "--offload-arch=gfx950", "--cuda-host-only", *flags,
           "-x", "hip", os.path.join(ROOT, "tests", "staged_rows_check.cpp"),
           "-x", "c++", os.path.join(ROOT, "paper_1909_02724_amd", "csrc", "tiles.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, str(seed), str(count)], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stderr[-4000:]
    print(r.stdout)
    for line in r.stdout.splitlines():
        kind, *fields = line.split()
        s = {k: int(v) for k, v in (f.split("=") for f in fields)}
        assert min(s["walked"], s["single"], s["np16"], s["np8"], s["np4"]) >= count // 80, (kind, s)
        assert s["col"] == s["low"] == s["high"] == s["off"] == 0, (kind, s)
