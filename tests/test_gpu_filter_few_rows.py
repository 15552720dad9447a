"""Short rows on both sides of the direct and the matrix filter (2^18
pixels, 3072 rows), at every remainder of the matrix kernel's tiles: the same bits, and the oracle's
values within FP32 rounding of them (2^-23, as for the other short rows)."""
import numpy as np
import pytest
import torch

import oracle
import synth

fdk = pytest.importorskip("paper_1909_02724_amd")

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("kind", ["ramlak", "shepp-logan"])
@pytest.mark.parametrize("nu", [2, 3, 5, 15, 16, 17, 63, 64, 65, 100, 127, 128, 129, 191, 192, 193, 255, 256])
def test_both_sides_of_the_line_agree(nu, kind):
    nv = 31
    views = -(-2 ** 18 // (nu * nv))
    g = synth.Geom(nx=32, ny=32, nz=32, nu=nu, nv=nv, sod=120.0, sdd=260.0, du=1.3, dv=0.9, off_u=-1.25,
                   off_v=0.4)
    gen = torch.Generator(device=DEV).manual_seed(nu)
    e = torch.randn((views, nv, nu), generator=gen, device=DEV)
    ang = synth.angles(views)
    q = fdk.filter(e, g, ang, kind=kind)
    adj = fdk.filter_adjoint(e, g, ang, kind=kind)
    for s in (0, views // 2, views - 1):
        one = e[s:s + 1].contiguous()
        assert torch.equal(q[s:s + 1], fdk.filter(one, g, ang, kind=kind, view0=s))
        assert torch.equal(adj[s:s + 1], fdk.filter_adjoint(one, g, ang, kind=kind, view0=s))
        host = one.cpu().double().numpy()
        for got, ref in ((q, oracle.filter(g, host, kind)), (adj, oracle.filter_adjoint(g, host, kind))):
            err = np.linalg.norm(got[s:s + 1].cpu().double().numpy() - ref) / np.linalg.norm(ref)
            assert err <= 2.0 ** -23
