"""A workgroup of the FFT filter sets up its twiddles and the ramp's spectrum
before its first rows: where it has few rows, that is most of its time. Timed
against the matrix filter on as many rows of 256 pixels, which does without:
0.55 of its time; 0.80 when the twiddles were gathered from one large table."""
import pytest
import torch

import synth

fdk = pytest.importorskip("paper_1909_02724_amd")

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _time(nu, rows):
    g = synth.Geom(nx=16, ny=16, nz=16, nu=nu, nv=rows, sod=500.0, sdd=1000.0)
    ang = synth.angles(1)
    e = torch.randn((1, rows, nu), device=DEV)
    out = torch.empty_like(e)
    fdk.filter(e, g, ang, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(50):
            fdk.filter(e, g, ang, out=out)
    best = float("inf")
    for _ in range(20):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_set_up_is_a_small_part_of_a_few_rows():
    assert _time(500, 4096) <= 0.68 * _time(256, 4096)
