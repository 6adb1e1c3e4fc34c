"""Products over few k's that fill the chip: every tile form gives the bits of the
64 x 64 tiles, which a few rows at a time take, at the edges of a k-tile and of
the rule; and a time that one block a CU could not reach."""
import numpy as np
import pytest

from paper_2412_00802_amd import hthedl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    return t


def operands(torch, ta, tb, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=g).bfloat16()
    b = torch.randn((N, K) if tb else (K, N), device="cuda", generator=g).bfloat16()
    return a, b


# K = 1 and 129 only where neither operand is contiguous along k
@pytest.mark.parametrize("ta,tb,K", [(0, 1, 8), (0, 1, 64), (0, 1, 72), (0, 1, 512), (0, 1, 520), (0, 0, 8), (0, 0, 200),
                                     (0, 0, 512), (0, 0, 576), (1, 0, 1), (1, 0, 65), (1, 0, 128), (1, 0, 129)])
@pytest.mark.parametrize("M,N", [(2048, 2048), (4104, 1000)])
def test_forms_agree(torch, ta, tb, K, M, N):
    a, b = operands(torch, ta, tb, M, N, K)
    bias, mask = torch.randn(N, device="cuda"), torch.randn((M, N), device="cuda").bfloat16()
    c, cb = torch.empty((M, N), device="cuda"), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    G = hthedl.hth_gemm_bf16
    G(ta, tb, M, N, K, a, M if ta else K, b, K if tb else N, bias=bias, mask=mask, ldm=N, c32=c, ldc=N, cbf=cb, ldcb=N)
    d, db = torch.empty_like(c), torch.empty_like(cb)
    for m0 in range(0, M, 1024):
        m = min(1024, M - m0)
        G(ta, tb, m, N, K, a[:, m0:m0 + m].contiguous() if ta else a[m0:m0 + m], m if ta else K, b, K if tb else N,
          bias=bias, mask=mask[m0:m0 + m], ldm=N, c32=d[m0:m0 + m], ldc=N, cbf=db[m0:m0 + m], ldcb=N)
    assert torch.equal(c, d) and torch.equal(cb, db)
    af, bf = a.double(), b.double()
    af, bf = (af.T if ta else af), (bf.T if tb else bf)
    rows = np.r_[0:40, M - 40:M]
    want, size = af[rows] @ bf + bias.double(), af[rows].abs() @ bf.abs() + bias.abs().double()
    err = (c[rows].double() - want * (mask[rows] > 0)).abs()
    assert (err <= (K + 1) * 2.0 ** -23 * size).all()


def test_few_ks_share_a_cu(torch):
    """65,536 x 1024 over 64 k's: 55 us, 121 with one block a CU."""
    M, N, K = 65536, 1024, 64
    a, b = operands(torch, 0, 1, M, N, K)
    c = torch.empty((M, N), device="cuda")
    best = 1e9
    for _ in range(4):
        e, f = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e.record()
        for _ in range(20):
            hthedl.hth_gemm_bf16(0, 1, M, N, K, a, K, b, K, c32=c, ldc=N)
        f.record()
        f.synchronize()
        best = min(best, e.elapsed_time(f) * 50)
    assert best < 90, best
