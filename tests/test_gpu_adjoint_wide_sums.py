"""The adjoint's wide tiles sum in 64 bits: one large voxel and fifteen of 2^-25
of it along a ray, in one brick. The large one's pixels hold all of the small
ones' sum, 3.75 units in their last place, which FP32 sums would lose.

|F(both) - F(large) - F(small)| stays below one such unit (the two projections'
own rounding), and below 1e-5 of the small part (FP32 coordinates)."""
import numpy as np
import pytest
import torch

import oracle
import synth

fdk = pytest.importorskip("paper_1909_02724_amd")

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("fixed_sums, far", [(False, 0.0), (True, 0.0), (True, 2.0 ** -45)],
                         ids=["default", "fixed", "fixed-far"])
@pytest.mark.parametrize("pixels, cone, off_v", [
    (2.0, 6.0, 0.0), (2.6, 6.0, 0.0), (2.6, 3.0, 0.0), (3.0, 6.0, 0.27), (2.6, 3.0, 0.27)])
def test_small_voxels_behind_a_large_one_are_kept(pixels, cone, off_v, fixed_sums, far):
    nx, ny, nz = 33, 45, 38
    g = synth.Geom(nx=nx, ny=ny, nz=nz, nu=int(50 * pixels), nv=int(46 * pixels), sod=cone * ny,
                   sdd=2.0 * cone * ny, du=2.0 / pixels, dv=2.0 / pixels, off_u=0.3, off_v=off_v)
    ang = np.array([0.0, np.pi])  # rays along y

    def project(x):
        v = torch.from_numpy(x.astype(np.float32)).to(DEV)
        return fdk.forward_project(v, g, ang, fixed_sums=fixed_sums).cpu().double().numpy()

    worst = 0.0
    for j in range(16, 32):  # one brick's columns at i = 16
        large, small = np.zeros((nz, ny, nx)), np.zeros((nz, ny, nx))
        large[nz // 2, j, 16] = 1.0
        small[nz // 2, 16:32, 16] = 2.0 ** -25
        small[nz // 2, j, 16] = 0.0
        if far:  # a brick spanning more than 2^40
            small[nz // 2, 16, 31] = far
        one = project(large)
        lost = np.abs(project(large + small) - one - oracle.forward_project(g, ang, small))
        hit = one > 0.1 * one.max()
        worst = max(worst, (lost[hit] / one[hit]).max() * 2.0 ** 23)
    print(f"wide sums pixels={pixels} cone={cone} off_v={off_v} {worst:.2f} units", flush=True)
    assert worst <= 1.0 + 3.75e-5
