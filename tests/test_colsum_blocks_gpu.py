"""Column sums at the edges of their blocks (64 columns, 256 from 65,536 columns on)
and of their chains' 32 loads in flight, and a time that 256 columns a block could
not reach."""
import numpy as np
import pytest

from paper_2412_00802_amd import hthedl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    return t


@pytest.mark.parametrize("M,N", [(0, 5), (1, 1), (3, 63), (4, 64), (127, 65), (128, 256), (129, 257), (515, 320),
                                 (130, 65535), (129, 65536), (9, 65793)])
@pytest.mark.parametrize("bf", [0, 1])
def test_block_edges(torch, M, N, bf):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    d = torch.randn((M, N), device="cuda", generator=g)
    d = d.bfloat16() if bf else d
    # four chains in a fixed order, added in a fixed order
    want = np.zeros((4, N), np.float32)
    v = d.float().cpu().numpy()
    for m in range(M):
        want[m % 4] += v[m]
    want = ((want[0] + want[1]) + want[2]) + want[3]
    out = torch.full((N,), 7.0, device="cuda")
    hthedl.hth_colsum(d if M else None, bf, M, N, out)
    np.testing.assert_array_equal(out.cpu().numpy(), want)


def test_a_training_batch_spreads_over_the_chip(torch):
    """8,192 rows of 1,024: 27 us, 63 in four blocks."""
    M, N = 8192, 1024
    d, out = torch.randn((M, N), device="cuda").bfloat16(), torch.empty(N, device="cuda")
    best = 1e9
    for _ in range(4):
        e, f = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e.record()
        for _ in range(20):
            hthedl.hth_colsum(d, 1, M, N, out)
        f.record()
        f.synchronize()
        best = min(best, e.elapsed_time(f) * 50)
    assert best < 45, best
