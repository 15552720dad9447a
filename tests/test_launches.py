"""What the entry points launch: kernels, grids, workgroup sizes and LDS, planned
on the host with the HIP runtime replaced (tests/launch_recorder.cpp)."""
import os
import shutil
import subprocess
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    import paper_1909_02724_amd as fdk
    fdk.lib()  # fails where the library is not built
    exe = str(tmp_path_factory.mktemp("launches") / "launch_recorder")
    cmd = [HIPCC, "-std=c++17", "-O1", "--offload-arch=gfx950", "--cuda-host-only", "-x", "hip",
           os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-x", "none", fdk.LIB_PATH,
           "-Wl,-rpath," + os.path.dirname(fdk.LIB_PATH), "-rdynamic", "-ldl", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(*calls, cap=0):
        """Each call: (op, nx, ny, nz, nu, nv, sod, mag, pu, pv, off_v, views).
        cap: bytes of memory the calls may take beyond what is mapped before them."""
        r = subprocess.run([exe, "cap", str(cap), *(str(x) for c in calls for x in c)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        out = SimpleNamespace(launches=[], attrs=[], calls=[])
        for line in r.stdout.splitlines():
            kind, name, *rest = line.split()
            if kind == "attr":
                out.attrs.append((name, int(rest[0])))
                continue
            f = {k: [int(x) for x in v.split(",")] for k, v in (p.split("=") for p in rest)}
            f = {k: v[0] if len(v) == 1 else v for k, v in f.items()}
            (out.launches if kind == "launch" else out.calls).append(SimpleNamespace(name=name, **f))
        assert len(out.calls) == len(calls) and all(c.status == 0 for c in out.calls)
        return out

    run.capped = lambda cap, *calls: run(*calls, cap=cap)
    return run


def cube(op, n, pixels=1.0, cone=7.8, off_v=0.0, views=20, rows=None):
    """n^3 voxels, `pixels` a voxel along u and `rows` along v, sod of cone * n."""
    rows = pixels if rows is None else rows
    return (op, n, n, n, int(1.2 * n * pixels) + 4, int(1.2 * n * rows) + 4, cone * n, 2.0, 2.0 / pixels,
            2.0 / rows, off_v, views)


def test_wide_adjoint_tiles_hold_64_bit_sums(record):
    """Every tile of the adjoint's wide kernel has room for a view's 64-bit sums,
    16 bytes a pixel and its mirror or 8 a pixel."""
    calls = [cube("fp", 60, px, cone, ov) for px in (1.33, 1.6, 2.0, 2.3, 2.6, 3.0, 3.5, 4.0)
             for ov in (0.0, 0.27) for cone in (3.0, 7.8)]
    wide = [f for f in record(*calls).launches if f.name.startswith("fp_wide")]
    assert len(wide) >= 10
    for f in wide:
        view = (f.tu + 1) * f.tvp * (16 if f.mirror else 8)
        assert f.vc >= 1 and view <= f.lds <= 154 * 1024, f


@pytest.mark.parametrize("pixels, off_v, name", [
    (0.5, 0.0, "bp_tiled_kernel<float,_true>"), (0.5, 0.27, "bp_tiled_kernel<float,_false>"),
    (0.7, 0.27, "bp_tiled_kernel<float,_false>"), (0.75, 0.0, "bp_staged_kernel<float,_true,_4>"),
    (1.0, 0.0, "bp_staged_kernel<float,_true,_8>"), (1.0, 0.27, "bp_staged_kernel<float,_false,_8>")])
def test_small_tiles_without_a_walk_run_the_general_kernel(record, pixels, off_v, name):
    """Below the five-wave staged kernel's passes there is only its four-wave
    relative, slower there than the general one."""
    assert [f.name for f in record(cube("bp", 300, pixels, off_v=off_v, views=25)).launches] == [name]


def test_pitch_leaves_room_for_64_bit_sums(record):
    """A 32-bit tile of the adjoint is padded for the banks only where two views
    (the room of one view's 64-bit sums) still fit, if they fit without."""
    calls = [cube("fp", n, px, cone, ov, views=8) for n in (100, 160) for cone in (5.0, 9.1)
             for ov in (0.0, 0.27) for px in (0.9, 1.0, 1.1, 1.2, 1.9, 2.0, 2.05, 2.1, 2.12, 2.15, 2.2, 2.3)]
    tiled = [f for f in record(*calls).launches if f.name.startswith("fp_") and not f.wide and f.vc > 0]
    fit = [f for f in tiled if 2 * (f.tu + 1) * (f.tv | 1) * (8 if f.mirror else 4) <= 36352]
    assert len(tiled) >= 30 and len(fit) >= 20
    for f in fit:
        assert f.vc >= 2, f


@pytest.mark.parametrize("n, views, chunks", [(17, 1, 1), (17, 8, 8), (17, 96, 96), (30, 5, 5), (30, 61, 61), (48, 30, 15)])
def test_tiny_adjoint_launches_take_a_view_a_workgroup(record, n, views, chunks):
    """While that makes at most two workgroups a CU; else at least two views."""
    f, = [f for f in record(cube("fp", n, off_v=0.27, views=views)).launches if f.name.startswith("fp_")]
    assert f.grid[1] == chunks and (f.grid[0] * views <= 512) == (chunks == views)


def test_a_kernels_lds_limit_is_the_same_for_every_launch(record):
    """It belongs to the kernel: a smaller one set by another thread between a
    launch's setting and the launch would refuse it."""
    calls = [cube(op, n, px, cone, ov) for op in ("bp", "fp") for n in (20, 40, 64, 90, 128) for ov in (0.0, 0.27)
             for px in (0.9, 1.0, 1.1, 1.2, 1.7, 2.0) for cone in (3.0, 7.8)]
    calls += [("filter", 8, 8, 8, nu, 64, 90.0, 2.0, 1.0, 1.0, 0.0, 3) for nu in (3000, 4096, 4200, 6000)]
    out = record(*calls)
    limits = {}
    for name, value in out.attrs:
        limits.setdefault(name, set()).add(value)
    assert len(limits) >= 6 and len(out.attrs) >= 60
    assert all(len(v) == 1 for v in limits.values()), limits
    for f in out.launches:
        assert f.lds <= max({65536} | limits.get(f.name, set())), f


@pytest.mark.parametrize("nu, rows, kernel", [
    (64, 3072, "direct"), (64, 3073, "matrix"), (256, 16, "direct"), (256, 1023, "direct"), (256, 1024, "matrix"),
    (100, 1, "direct"), (1, 3072, "direct"), (1, 3073, "matrix"), (257, 1, "fft")])
def test_few_short_rows_are_filtered_directly(record, nu, rows, kernel):
    f, = record(("filter", 8, 8, 8, nu, 1, 90.0, 2.0, 1.0, 1.0, 0.0, rows)).launches
    assert f.name.startswith(f"filter_{kernel}_kernel<")


def test_a_forward_projection_evaluates_each_angle_once(record):
    """One sine and one cosine a view, whatever the launches and slice runs."""
    for n, off_v, views in ((17, 0.0, 400), (40, 0.27, 97), (41, 0.0, 96), (130, 0.0, 191)):
        assert record(cube("fp", n, off_v=off_v, views=views)).calls[0].trig == 2 * views


def test_a_forward_projection_allocates_no_memory_for_its_views(record):
    """No C++ exception may cross the C ABI: with 2^23 views and no memory to
    spare beyond their angles, the call plans every launch as with few."""
    out = record.capped(1 << 25, ("fp", 2, 2, 2, 4, 4, 90.0, 2.0, 1.0, 1.0, 0.0, 1 << 23))
    assert out.calls[0].trig == 2 << 23


@pytest.mark.parametrize("nx, ny, nz, pixels, halved", [
    (236, 109, 284, 1.9, False), (169, 164, 250, 1.9, False), (229, 118, 214, 1.8, False),
    (128, 160, 200, 1.9, True), (280, 100, 216, 1.42, True)])
def test_wide_tiles_halve_their_bricks_while_half_of_them_fit(record, nx, ny, nz, pixels, halved):
    """Beyond what the chip holds twice over, bricks of 8 slices are slower than
    the general kernel."""
    n = max(nx, ny, nz)
    call = ("bp", nx, ny, nz, int(1.3 * n * pixels), int(1.3 * n * pixels), 6.0 * n, 2.0, 2.0 / pixels,
            2.0 / pixels, 0.0, 20)
    f, = record(call).launches
    assert f.name == ("bp_groups_kernel<float,_true,_0,_8>" if halved else "bp_tiled_wide_kernel<float,_true>"), f
