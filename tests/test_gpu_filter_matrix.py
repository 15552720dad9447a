"""Rows of up to 256 pixels, filtered by FP64 matrix products: every remainder of
the 16-pixel tiles, 64-pixel parts and 4-tap steps, row counts off the 16 of a
workgroup and on both sides of the split of the columns (512 workgroups), row
bands, and the adjoint, against the FP64 oracle.

The sums are FP64, so a float32 result differs from the oracle's by its own
rounding, at most 2^-24 of it; 2^-23 leaves as much again for FP64 rounding at
cancelled outputs."""
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


def geom(nu, nv):
    return synth.Geom(nx=32, ny=32, nz=32, nu=nu, nv=nv, sod=120.0, sdd=260.0, du=1.3, dv=0.9,
                      off_u=-1.25, off_v=0.4)


@pytest.mark.parametrize("kind", ["ramlak", "shepp-logan"])
@pytest.mark.parametrize("nu", [1, 2, 3, 5, 15, 16, 17, 63, 64, 65, 100, 127, 128, 129, 191, 192, 193, 255, 256])
def test_short_rows_match_oracle(nu, kind):
    g = geom(nu, 7)
    e = np.random.default_rng(nu).standard_normal((3, 7, nu)).astype(np.float32)
    got = fdk.filter(torch.from_numpy(e).to(DEV), g, synth.angles(3), kind=kind)
    assert rel_l2(host(got), oracle.filter(g, e.astype(np.float64), kind)) <= 2.0 ** -23
    adj = fdk.filter_adjoint(torch.from_numpy(e).to(DEV), g, synth.angles(3), kind=kind)
    assert rel_l2(host(adj), oracle.filter_adjoint(g, e.astype(np.float64), kind)) <= 2.0 ** -23


@pytest.mark.parametrize("nu", [65, 130, 200, 256])
def test_many_rows_match_few(nu):
    """9000 rows (all columns in a workgroup) and the same rows 90 at a time
    (columns shared out) give the same bits; a band too."""
    g = geom(nu, 90)
    e = torch.from_numpy(np.random.default_rng(nu).standard_normal((100, 90, nu)).astype(np.float32)).to(DEV)
    ang = synth.angles(100)
    whole = fdk.filter(e, g, ang)
    ref = oracle.filter(g, host(e[41:42]))
    assert rel_l2(host(whole[41:42]), ref) <= 2.0 ** -23
    for s in (0, 41, 99):
        assert torch.equal(whole[s:s + 1], fdk.filter(e[s:s + 1], g, ang, view0=s))
    band = fdk.filter(e[:, 13:40].contiguous(), g, ang, rows=(13, 27))
    assert torch.equal(band, whole[:, 13:40])
