"""The packed C geometry holds each field as a ctypes constructor stores it,
integers that do not fit int32 included (the library then refuses or takes the
wrapped value as before)."""
import dataclasses

import numpy as np
import pytest

fdk = pytest.importorskip("paper_1909_02724_amd")

GOOD = fdk.Geometry(nx=64, ny=65, nz=66, nu=67, nv=68, sod=500.0, sdd=1000.0, dx=0.1, dy=0.2, dz=0.3,
                    du=0.4, dv=0.5, off_u=0.6, off_v=-0.7)


@pytest.mark.parametrize("change", [{}, {"nx": 2 ** 31}, {"ny": 2 ** 40 + 5}, {"nu": -3}, {"nz": "12"},
                                    {"nv": 3.7}, {"sod": float("nan")}, {"off_u": np.float32(0.1)}])
def test_fields_match_a_constructor(change):
    g = dataclasses.replace(GOOD, **change)
    ang = [0.25, 0.5, 4.0]
    cg, _keep = fdk._cgeom(g, ang)
    for name, kind in fdk._CGeometry._fields_:
        if name in ("np", "angles"):
            continue
        want = kind((float if kind is fdk.C.c_double else int)(getattr(g, name))).value
        got = getattr(cg, name)
        assert got == want or (got != got and want != want), name
    assert cg.np == 3 and [cg.angles[i] for i in range(3)] == ang


@pytest.mark.parametrize("change", [{"nx": "x"}, {"sdd": "y"}, {"nu": float("inf")}])
def test_values_that_are_no_numbers_raise_as_before(change):
    with pytest.raises((ValueError, OverflowError)):
        fdk._cgeom(dataclasses.replace(GOOD, **change), [0.0])
