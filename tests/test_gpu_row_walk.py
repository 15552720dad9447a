"""GPU parity of the back-projector's row walk, brick heights and view groups
against the FP64 CPU oracle: every launch shape the dispatch picks (bricks of
4, 8 and 16 slices, one to four groups of threads a brick, five- and four-wave
instances, row walks of 8 and 4 slices and the general loop), mirrored and
plain, with view counts below, at and off multiples of the groups.

Tolerance 1e-5 rel-L2 as for the other FP32 parity tests: FP32 coordinates of
a few 1e-6 pixel on random projections."""
import numpy as np
import pytest
import torch

import oracle
import synth

fdk = pytest.importorskip("paper_1909_02724_amd")

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def rel_l2(got, ref):
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


def host(t):
    return t.detach().cpu().double().numpy()


def geom(n, rows_per_slice, off_v, cone=8.0):
    """Volume n = (nx, ny, nz) and a detector that sees it, v advancing by
    about `rows_per_slice` a slice at the axis."""
    m = max(n)
    return synth.Geom(nx=n[0], ny=n[1], nz=n[2], nu=m + 21, nv=int(m * rows_per_slice) + 17,
                      sod=cone * m, sdd=2.0 * cone * m, du=2.0, dv=2.0 / rows_per_slice,
                      off_u=0.3, off_v=off_v)


SIZES = {  # by the number of 16 x 16 x 16 bricks (mirrored)
    "tiny": (33, 17, 40), "small": (97, 90, 95), "medium": (128, 126, 101),
    "pairs": (141, 144, 127), "large": (170, 176, 150),
}


@pytest.mark.parametrize("off_v", [0.0, 0.27], ids=["mirrored", "plain"])
@pytest.mark.parametrize("slope", [1.0, 1.12, 1.3], ids=["walk8", "walk4", "general"])
@pytest.mark.parametrize("size, views", [("tiny", 1), ("tiny", 7), ("small", 3), ("medium", 9),
                                         ("pairs", 5), ("large", 4)])
def test_launch_shapes_match_oracle(size, views, slope, off_v):
    g = geom(SIZES[size], slope, off_v)
    ang = synth.angles(views, start=0.37)
    print(f"row walk {size} views={views} slope={slope} off_v={off_v}", flush=True)
    q = synth.random_projections(views + 3, views, g)
    base = np.random.default_rng(2).standard_normal((g.nz, g.ny, g.nx)).astype(np.float32)
    ref = oracle.backproject(g, ang, q.astype(np.float64), scale=1.0e4)
    qt = torch.from_numpy(q).to(DEV)
    got = fdk.backproject(qt, g, ang, scale=1.0e4)
    assert rel_l2(host(got), ref) <= 1e-5
    assert torch.equal(got, fdk.backproject(qt, g, ang, scale=1.0e4))  # bitwise reproducible
    out = torch.from_numpy(base).to(DEV)
    fdk.backproject(qt, g, ang, scale=1.0e4, out=out, accumulate=True)
    assert rel_l2(host(out), base + ref) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_narrow_pitch_of_large_grids(dtype):
    """Mirrored grids beyond the resident bricks with tiles of which two fit a
    workgroup's share of LDS only at a column pitch of 3 or 13 mod 16."""
    g = geom((180, 225, 197), 1.0, 0.0, cone=1000.0 / 225)
    ang = synth.angles(3, start=0.37)
    qt = torch.from_numpy(synth.random_projections(8, 3, g)).to(DEV, dtype)
    assert rel_l2(host(fdk.backproject(qt, g, ang)), oracle.backproject(g, ang, host(qt))) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("size", ["tiny", "medium", "large"])
@pytest.mark.parametrize("off_v", [0.0, 0.27], ids=["mirrored", "plain"])
def test_16bit_storage_matches_oracle(dtype, size, off_v):
    g = geom(SIZES[size], 1.0, off_v)
    ang = synth.angles(6, start=0.1)
    qt = torch.from_numpy(synth.random_projections(4, 6, g)).to(DEV, dtype)
    ref = oracle.backproject(g, ang, host(qt))
    assert rel_l2(host(fdk.backproject(qt, g, ang)), ref) <= 1e-5


@pytest.mark.parametrize("size", ["tiny", "small", "medium", "large"])
@pytest.mark.parametrize("off_v", [0.0, 0.27], ids=["mirrored", "plain"])
def test_non_finite_pixels_reach_their_own_voxels_only(size, off_v):
    """A NaN or an infinity reaches exactly the voxels with a tap on it, as
    in the oracle, though the row walk reads one more row a voxel; all other
    voxels keep their values, and an accumulated slab is added to once."""
    g = geom(SIZES[size], 1.0, off_v)
    ang = synth.angles(5, start=0.2)
    q = synth.random_projections(9, 5, g)
    rng = np.random.default_rng(1)
    for s, value in [(0, np.nan), (2, np.inf), (4, -np.inf)]:
        q[s, rng.integers(3, g.nv - 3), rng.integers(3, g.nu - 3)] = value
    ref = oracle.backproject(g, ang, q.astype(np.float64), scale=1.0e4)
    out = torch.full((g.nz, g.ny, g.nx), 0.5, device=DEV)
    got = host(fdk.backproject(torch.from_numpy(q).to(DEV), g, ang, scale=1.0e4, out=out,
                               accumulate=True))
    fine = np.isfinite(ref)
    assert not fine.all()
    assert np.array_equal(fine, np.isfinite(got))
    assert rel_l2(got[fine], 0.5 + ref[fine]) <= 1e-5


@pytest.mark.parametrize("off_v", [0.0, 0.27], ids=["mirrored", "plain"])
@pytest.mark.parametrize("slope", [1.0, 1.12, 1.3], ids=["walk", "walk_edge", "single"])
@pytest.mark.parametrize("size, views, cone", [("tiny", 1, 8.0), ("tiny", 13, 3.0), ("small", 7, 8.0),
                                               ("medium", 97, 5.0), ("large", 3, 8.0)])
def test_adjoint_walk_matches_oracle(size, views, cone, slope, off_v):
    """The adjoint's row sums, in bricks that walk and bricks that take one
    slice at a time, for views along both axes, against the oracle; and on a
    volume of ones, where every pixel's sum comes closest to the fixed-point
    bound (an overflow would wrap), to 2e-6 of it: FP32 rounding of the
    coordinates and of the sums' few dozen adds."""
    g = geom(SIZES[size], slope, off_v, cone=cone)
    ang = synth.angles(views, start=0.6)
    print(f"adjoint walk {size} views={views} cone={cone} slope={slope} off_v={off_v}", flush=True)
    x = np.random.default_rng(views).standard_normal((g.nz, g.ny, g.nx)).astype(np.float32)
    for vol, tol in ((x, 1e-5), (np.ones_like(x), 2e-6)):
        ref = oracle.forward_project(g, ang, vol.astype(np.float64), scale=1.0e4)
        got = fdk.forward_project(torch.from_numpy(vol).to(DEV), g, ang, scale=1.0e4)
        err = rel_l2(host(got), ref)
        print(f"  {err:.2e}", flush=True)
        assert err <= tol
        fdk.forward_project(torch.from_numpy(vol).to(DEV), g, ang, scale=1.0e4, out=got,
                            accumulate=True)
        assert rel_l2(host(got), 2.0 * ref) <= tol


@pytest.mark.parametrize("off_v", [0.0, 0.27], ids=["mirrored", "plain"])
@pytest.mark.parametrize("views", [1, 2, 3, 5, 62, 63, 96, 97, 191])
def test_adjoint_short_chunks_match_oracle(views, off_v):
    """Few bricks: chunks of two views, up to 49 of them in a launch, the last
    of a direction shorter. Tolerance as above."""
    g = geom((17, 20, 18), 1.0, off_v)
    ang = synth.angles(views, start=0.2)
    x = np.random.default_rng(views).standard_normal((g.nz, g.ny, g.nx)).astype(np.float32)
    got = fdk.forward_project(torch.from_numpy(x).to(DEV), g, ang, scale=1.0e4)
    assert rel_l2(host(got), oracle.forward_project(g, ang, x.astype(np.float64), scale=1.0e4)) <= 1e-5


@pytest.mark.parametrize("pixels, cone, off_v", [
    (1.33, 3.0, 0.0), (2.0, 6.0, 0.0), (2.6, 6.0, 0.0), (2.0, 6.0, 0.27), (3.0, 6.0, 0.27),
    (5.0, 6.0, 0.0), (5.0, 6.0, 0.27)])
def test_adjoint_wide_tiles_match_oracle(pixels, cone, off_v):
    """Several pixels a voxel, wide cones: tiles of the wide kernel, of one and
    of two stages, and past it. Same tolerance; volumes with a non-finite voxel
    or with magnitudes too far apart for 64-bit sums give the direct kernel's
    non-finite pixels and its values."""
    nx, ny, nz = 33, 45, 38
    g = synth.Geom(nx=nx, ny=ny, nz=nz, nu=int(50 * pixels), nv=int(46 * pixels), sod=cone * ny,
                   sdd=2.0 * cone * ny, du=2.0 / pixels, dv=2.0 / pixels, off_u=0.3, off_v=off_v)
    ang = synth.angles(11, start=0.3)
    rng = np.random.default_rng(3)
    x = rng.standard_normal((nz, ny, nx)).astype(np.float32)
    far = (x * np.exp(rng.uniform(-30.0, 10.0, x.shape))).astype(np.float32)
    for vol in (x, far):
        ref = oracle.forward_project(g, ang, vol.astype(np.float64), scale=1.0e4)
        got = fdk.forward_project(torch.from_numpy(vol).to(DEV), g, ang, scale=1.0e4)
        err = rel_l2(host(got), ref)
        print(f"adjoint wide pixels={pixels} off_v={off_v} {err:.2e}", flush=True)
        assert err <= 1e-5
    for bad in (np.inf, np.nan):
        x[5, 7, 9] = bad
        v = torch.from_numpy(x).to(DEV)
        got = host(fdk.forward_project(v, g, ang))
        want = host(fdk.forward_project(v, g, ang, direct=True))
        fine = np.isfinite(want)
        assert not fine.all() and np.array_equal(fine, np.isfinite(got))
        assert rel_l2(got[fine], want[fine]) <= 1e-5


@pytest.mark.parametrize("magnitude", [1e-36, 1e-27, 1e36])
def test_adjoint_at_the_ends_of_the_float_range(magnitude):
    """The sums are scaled to the brick's largest voxel, so volumes near either
    end of FP32's range project as accurately as others."""
    g = geom((40, 33, 30), 1.0, 0.0)
    ang = synth.angles(4, start=0.2)
    x = np.random.default_rng(6).uniform(0.5, 1.0, (g.nz, g.ny, g.nx)).astype(np.float32)
    ref = oracle.forward_project(g, ang, x.astype(np.float64))
    got = fdk.forward_project(torch.from_numpy((x * np.float32(magnitude))).to(DEV), g, ang,
                              scale=1.0)
    # (projections of the smallest volumes are subnormal or zero in FP32)
    floor = 2.0 ** -149 * 200 / magnitude
    err = np.abs(host(got) / magnitude - ref).max()
    assert err <= 1e-5 * ref.max() + floor
