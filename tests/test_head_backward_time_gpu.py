"""The output layer's backward over many rows: its values against float64 at the
edges of its 256 chains, and a time that a few blocks could not reach."""
import numpy as np
import pytest

from paper_2412_00802_amd import hthedl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    return t


def call(torch, Bn, Kd):
    g = torch.Generator(device="cuda").manual_seed(Bn + Kd)
    h = torch.randn((Bn, Kd), device="cuda", generator=g).relu().bfloat16()
    w, dz = torch.randn((Kd, 2), device="cuda", generator=g), torch.randn((Bn, 2), device="cuda", generator=g)
    dw, dh = torch.empty((Kd, 2), device="cuda"), torch.empty((Bn, Kd), dtype=torch.bfloat16, device="cuda")
    return h, w, dz, dw, dh


@pytest.mark.parametrize("Bn,Kd", [(1, 1), (255, 3), (256, 64), (257, 65), (513, 256)])
def test_chains(torch, Bn, Kd):
    h, w, dz, dw, dh = call(torch, Bn, Kd)
    hthedl.hth_head_backward(h, Bn, Kd, w, dz, dw, dh)
    hr, zr, wr = (v.double().cpu().numpy() for v in (h, dz, w))
    # a chain of ceil(Bn / 256) products, a tree of 8 levels
    lim = (-(-Bn // 256) + 9) * 2.0 ** -24 * 1.01 * (np.abs(hr.T) @ np.abs(zr)) + 1e-30
    assert (np.abs(dw.double().cpu().numpy() - hr.T @ zr) <= lim).all()
    want = (zr @ wr.T) * (hr > 0)
    lim = 2.0 ** -8 * np.abs(want) + 2.0 ** -22 * (np.abs(zr) @ np.abs(wr.T))
    assert (np.abs(dh.double().cpu().numpy() - want) <= lim).all()


def test_many_rows_fill_the_chip(torch):
    """65,536 rows of 256: 188 us with a block per column, 977 with four blocks."""
    Bn, Kd = 65536, 256
    args = call(torch, Bn, Kd)
    best = 1e9
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            hthedl.hth_head_backward(args[0], Bn, Kd, *args[1:])
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    assert best < 450, best
