"""Edges of the screener's kernels: GEMM tile choices, scoring straight from
feature lists, the feature hash's staged and unstaged walk, the output layer's
row and width remainders, training at odd batch sizes."""
import numpy as np
import pytest

from oracle import screener as S
from paper_2412_00802_amd import hthedl, screened, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    hthedl.lib()
    return t


# 128 x 128 tiles (256 of them and more) with ragged edges and k-tile remainders; 64 x 64 around one tile
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(2040, 2056, 72), (2048, 2048, 8), (64, 64, 136), (72, 56, 264)])
def test_gemm_tiles(torch, ta, tb, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), device="cuda", generator=g).bfloat16()
    b = torch.randn((K, N), device="cuda", generator=g).bfloat16()
    A, B = (a.T.contiguous() if ta else a), (b.T.contiguous() if tb else b)
    c = torch.full((M, N), float("nan"), device="cuda")
    hthedl.hth_gemm_bf16(ta, tb, M, N, K, A, M if ta else K, B, K if tb else N, c32=c, ldc=N)
    want = a.double() @ b.double()
    # fp32 accumulation of K products: 2^-23 a step of the running sum, bounded by the sum of magnitudes
    lim = K * 2.0 ** -23 * (a.double().abs() @ b.double().abs())
    assert bool(((c.double() - want).abs() <= lim + 1e-30).all())


def _rows(rng, n):
    """Hypotheses and their parents: ordinary ones, one whose rows overflow the wave (more than 64 features) and one
    that repeats a subtree more often than bf16 counts exactly (more than 256 times)."""
    cfg = synth.small_config(n=200, n_concepts=40, n_roles=5, n_data=3, seed_index=1300)
    kb = synth.make_kb(cfg)
    from paper_2412_00802_amd import search
    parents = synth.make_sized_hypotheses(cfg, kb, count=8)
    ref = search.Refiner(kb, rng)
    kids, pidx = [], []
    while len(kids) < n:
        p = int(rng.integers(0, len(parents)))
        for c in ref.refine(parents[p], 4):
            kids.append(c)
            pidx.append(p)
    kids, pidx = kids[:n], pidx[:n]
    if n > 2:
        kids[1] = ("or",) + tuple(("and", ("atom", i % 37), ("atom", i % 11)) for i in range(60))
        kids[2] = ("and",) + tuple(("atom", 3) for _ in range(301)) + (("atom", 4),)
    return parents, kids, pidx


@pytest.mark.parametrize("n,kind,mode", [(1, 0, "plain"), (63, 1, "delta"), (64, 0, "context"), (65, 1, "delta"),
                                         (200, 0, "delta")])
def test_scores_from_features(torch, n, kind, mode):
    from paper_2412_00802_amd.screener import FeatureBatch, Screener, init_params
    rng = np.random.default_rng(n + kind)
    parents, kids, pidx = _rows(rng, n)
    params = init_params(seed=n)
    params["b1"] = rng.standard_normal(1024).astype(np.float32) * 0.05
    params["b2"] = rng.standard_normal(256).astype(np.float32) * 0.05
    params["b3"] += np.float32(2.0)
    scr = Screener(params, batch=64, loss="mse")
    fb, pfb = FeatureBatch(*hthedl.encode_batch(kids)), FeatureBatch(*hthedl.encode_batch(parents))
    P = torch.from_numpy(np.asarray(pidx, dtype=np.int32)).cuda()
    base = rng.integers(0, 900, (n, 2)).astype(np.uint32)
    out = torch.full((n,), float("nan"), device="cuda")
    rel = mode != "plain"
    screened.score(scr, fb, n, 1000, 1200, out, base=torch.from_numpy(base.view(np.int32)).cuda(), kind=kind,
                   parents=pfb if rel else None, parent_index=P if rel else None, context=int(mode == "context"))
    x = S.delta_features(kids, parents, pidx, context=mode == "context") if rel else S.dense_features(kids)
    acts, _ = S.forward({k: v.astype(np.float64) for k, v in params.items()}, S.bf16(np.asarray(x, np.float32)),
                        rounding=True)
    want = S.predicted_f1(acts["z"], 1000, 1200, base, kind="log_removed" if kind else "share")
    # a bf16 activation may round the other way (2^-8 of one of 1,280 terms): z within 2^-8 relative, well inside
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=2.0 ** -8, atol=1e-5)
    with pytest.raises(hthedl.HthError):
        screened.score(scr, fb, n, 1000, 1200, out, kind=1, parents=pfb if rel else None, parent_index=P if rel else None)


def test_features_beyond_the_staged_range(torch):
    """More nodes in a block's hypotheses than its LDS area holds, next to blocks that fit, and the rest of a block."""
    from paper_2412_00802_amd.screener import FeatureBatch
    cfg = synth.small_config(n=200, n_concepts=40, n_roles=5, n_data=3, seed_index=1301)
    hyps = synth.make_sized_hypotheses(cfg, synth.make_kb(cfg), count=300)
    hyps[5] = ("and",) + tuple(("not", ("atom", i % 40)) for i in range(1200))
    fb = FeatureBatch(*hthedl.encode_batch(hyps))
    want = [v for h in hyps for v in S.subtree_features(h)]
    np.testing.assert_array_equal(fb.hash.cpu().numpy().view(np.uint64), np.array([w[0] for w in want], dtype=np.uint64))
    np.testing.assert_array_equal(fb.feat.cpu().numpy().view(np.uint16), np.array([w[1] for w in want], dtype=np.uint16))
    assert int(fb.bad.item()) == 0


@pytest.mark.parametrize("Bn,Kd", [(1, 8), (63, 256), (65, 264), (130, 37), (64, 600)])
def test_head_remainders(torch, Bn, Kd):
    rng = np.random.default_rng(Bn + Kd)
    h = np.maximum(rng.standard_normal((Bn, Kd)), 0).astype(np.float32)
    H = torch.from_numpy(h).cuda().bfloat16()
    hr = H.double().cpu().numpy()
    w, b = rng.standard_normal((Kd, 2)).astype(np.float32), rng.standard_normal(2).astype(np.float32)
    z = torch.empty((Bn, 2), device="cuda")
    W = torch.from_numpy(w).cuda()
    hthedl.hth_head_forward(H, Bn, Kd, W, torch.from_numpy(b).cuda(), z)
    lim = (Kd + 2) * 2.0 ** -23 * (np.abs(hr) @ np.abs(w) + np.abs(b))
    assert (np.abs(z.cpu().numpy() - (hr @ w.astype(np.float64) + b)) <= lim).all()
    dz = rng.standard_normal((Bn, 2)).astype(np.float32)
    dw, dh = torch.empty((Kd, 2), device="cuda"), torch.empty((Bn, Kd), dtype=torch.bfloat16, device="cuda")
    hthedl.hth_head_backward(H, Bn, Kd, W, torch.from_numpy(dz).cuda(), dw, dh)
    lim = (Bn + 2) * 2.0 ** -23 * (np.abs(hr.T) @ np.abs(dz)) + 1e-30
    assert (np.abs(dw.cpu().numpy() - hr.T @ dz.astype(np.float64)) <= lim).all()
    want = (dz.astype(np.float64) @ w.T.astype(np.float64)) * (hr > 0)
    np.testing.assert_allclose(dh.double().cpu().numpy(), want, rtol=2.0 ** -8, atol=1e-6)


@pytest.mark.parametrize("n,loss", [(1, "mse"), (67, "bce"), (1000, "mse")])
def test_training_step_odd_batches(torch, n, loss):
    """The one-call step against the single calls it stands for."""
    from paper_2412_00802_amd.screener import D_H1, D_H2, D_IN, Screener, init_params
    rng = np.random.default_rng(n)
    x = torch.from_numpy(((rng.random((n, D_IN)) < 0.004) * rng.integers(1, 3, (n, D_IN))).astype(np.float32)).cuda().bfloat16()
    y = torch.from_numpy(rng.random((n, 2)).astype(np.float32)).cuda()
    a, b = (Screener(init_params(seed=5), batch=n, lr=1e-3, loss=loss) for _ in range(2))
    for s in (a, b):
        for k in s.p:
            s.v[k].fill_(1e-8)
    a.train_step(n, y, x)
    G, kind = hthedl.hth_gemm_bf16, b.loss_kind
    b.forward(n, x)
    hthedl.hth_head_forward(b.h2, n, D_H2, b.p["w3"], b.p["b3"], b.z, y, b.dz, 1.0 / (2 * n), b.loss, loss_kind=kind)
    hthedl.hth_head_backward(b.h2, n, D_H2, b.p["w3"], b.dz, b.g["w3"], b.dh2)
    hthedl.hth_colsum(b.dz, 0, n, 2, b.g["b3"])
    G(1, 0, D_H1, D_H2, n, b.h1, D_H1, b.dh2, D_H2, c32=b.g["w2"], ldc=D_H2)
    hthedl.hth_colsum(b.dh2, 1, n, D_H2, b.g["b2"])
    G(0, 1, n, D_H1, D_H2, b.dh2, D_H2, b.w2b, D_H2, mask=b.h1, ldm=D_H1, cbf=b.dh1, ldcb=D_H1)
    hthedl.hth_colsum(b.dh1, 1, n, D_H1, b.g["b1"])
    G(1, 0, D_IN, D_H1, n, x, D_IN, b.dh1, D_H1, c32=b.g["w1"], ldc=D_H1)
    for k in ("w1", "b1", "w2", "b2", "w3", "b3"):
        pbf = b.w1b if k == "w1" else (b.w2b if k == "w2" else None)
        hthedl.hth_adamw(b.p[k], b.g[k], b.m[k], b.v[k], pbf, b.p[k].numel(), b.lr, b.b1, b.b2, b.eps,
                         b.wd if k[0] == "w" else 0.0, 1)
    b._transpose()
    assert a.step_no == 1
    for f in ("z", "dz", "dh2", "dh1", "w1b", "w2b", "w1t", "w2t"):
        assert torch.equal(getattr(a, f), getattr(b, f)), f
    for k in a.p:
        for f in ("g", "p", "m", "v"):
            assert torch.equal(getattr(a, f)[k], getattr(b, f)[k]), (f, k)


@pytest.mark.parametrize("n,k", [(1, 1), (255, 255), (4096, 1), (70_000, 1400)])
def test_topk_of_equal_leading_bits(torch, n, k):
    """Scores of one beam: all in a narrow range, with ties across the threshold, NaN and infinities."""
    rng = np.random.default_rng(n)
    s = (0.67 + rng.integers(0, 500, n) * 2.0 ** -24).astype(np.float32)
    if n > 300:
        s[:5] = [np.nan, np.inf, -np.inf, 0.0, -0.0]
    D = torch.from_numpy(s).cuda()
    idx, work = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(65538, dtype=torch.int32, device="cuda")
    hthedl.hth_topk(D, n, k, idx, work)
    got = idx.cpu().numpy()
    assert len(set(got.tolist())) == k and got.min() >= 0 and got.max() < n
    key = np.where(np.isnan(s), -np.inf, s)
    np.testing.assert_array_equal(np.sort(key[got]), np.sort(key)[n - k:])
