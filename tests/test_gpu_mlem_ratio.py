"""MLEM's guarded ratio p / max(F x, 1e-3 max(F x)) against the same expression
in PyTorch, at projection counts about one full pass of the maximum's grid
(1024 blocks of 256 threads, eight loads each) and far below it.

F is deterministic, so the denominators are the same bits; the tolerance is two
units in the last place of the float32 quotient (2^-22)."""
import numpy as np
import pytest
import torch

fdk = pytest.importorskip("paper_1909_02724_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views,nv,nu", [(1, 2, 3), (1, 1024, 2047), (1, 1024, 2048), (1, 1024, 2049),
                                         (3, 1024, 2049)])
def test_ratio_at_the_edges_of_the_maximum(views, nv, nu):
    n, mag = 24, 1.5
    geom = fdk.Geometry(nx=n, ny=n, nz=n, nu=nu, nv=nv, sod=20.0 * n, sdd=20.0 * n * mag,
                        du=mag * (n + 1.0) / nu, dv=mag * (n + 1.0) / nv)
    ang = np.linspace(0.1, 0.4, views)
    gen = torch.Generator().manual_seed(nu)
    x = torch.rand((n, n, n), generator=gen)
    x[-1] *= 1e4  # the largest sums, on the detector's last rows, raise the floor
    x, p = x.cuda(), torch.rand((views, nv, nu), generator=gen).cuda()
    f = fdk.forward_project(x, geom, ang, fixed_sums=True)  # as the iteration does
    want = p / torch.maximum(f, 1e-3 * f.max())
    ratio = torch.empty_like(p)
    fdk.mlem_iteration(x.clone(), p, torch.ones_like(x), geom, ang, proj_tmp=ratio)
    assert float(f.max()) > 0.0
    torch.testing.assert_close(ratio, want, rtol=2.0 ** -22, atol=0.0)
