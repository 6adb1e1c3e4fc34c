"""Scoring of wide hypotheses: rows at the edge of the feature list (64 entries),
far longer ones next to short ones, batches that are wide on average, and the
time that one long row costs."""
import numpy as np
import pytest

from oracle import screener as S
from paper_2412_00802_amd import hthedl, screened
from paper_2412_00802_amd.screener import FeatureBatch, Screener, init_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    return t


def wide(k, seed):
    """k nodes, of which some are equal (k > 1)."""
    rng = np.random.default_rng(seed)
    return ("atom", seed % 900) if k == 1 else ("or",) + tuple(("atom", int(a)) for a in rng.integers(0, 900, k - 1))


# nodes of the rows and of the parents; context
@pytest.mark.parametrize("sizes,psizes,context", [
    ((1, 63, 64, 65, 66, 5, 700, 3, 64), None, 0),
    ((32, 33, 2, 60, 900, 4, 31), (32, 31, 62, 5, 800), 0),
    ((20, 22, 64, 9, 300), (22, 21, 300, 5), 1),
    ((1500, 1200), None, 0),                        # wide on average
    ((700, 40, 300), (500, 400), 1)])
@pytest.mark.parametrize("kind", [0, 1])
def test_scores_of_wide_rows(torch, sizes, psizes, context, kind):
    rng = np.random.default_rng(len(sizes) + context)
    kids = [wide(k, i) for i, k in enumerate(sizes)] * 5
    parents = [wide(k, i) for i, k in enumerate(psizes or (2,))]
    pidx = rng.integers(0, len(parents), len(kids))
    n = len(kids)
    params = init_params(seed=n)
    params["b1"] = rng.standard_normal(1024).astype(np.float32) * 0.05
    params["b3"] += np.float32(2.0)
    scr = Screener(params, batch=16, loss="mse")
    fb, pfb = FeatureBatch(*hthedl.encode_batch(kids)), FeatureBatch(*hthedl.encode_batch(parents))
    base = rng.integers(0, 900, (n, 2)).astype(np.uint32)
    out = torch.full((n,), float("nan"), device="cuda")
    rel = psizes is not None
    screened.score(scr, fb, n, 1000, 1200, out, base=torch.from_numpy(base.view(np.int32)).cuda(), kind=kind,
                   parents=pfb if rel else None, parent_index=torch.from_numpy(pidx.astype(np.int32)).cuda() if rel else None,
                   context=context)
    x = S.delta_features(kids, parents, pidx, context=bool(context)) if rel else S.dense_features(kids)
    acts, _ = S.forward({k: v.astype(np.float64) for k, v in params.items()}, S.bf16(np.asarray(x, np.float32)), rounding=True)
    want = S.predicted_f1(acts["z"], 1000, 1200, base, kind="log_removed" if kind else "share")
    # a bf16 activation may round the other way (2^-8 of one of 1,280 terms): z within 2^-8 relative
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=2.0 ** -8, atol=1e-5)


def test_one_long_row_costs_its_length(torch):
    """6,000 nodes in one of 256 rows: about 800 steps of a wave, not 560,000 (thousands of times the dense chain's)."""
    kids = [wide(6, i) for i in range(255)] + [wide(6000, 7)]
    fb, scr = FeatureBatch(*hthedl.encode_batch(kids)), Screener(init_params(seed=1), batch=256)
    out, base = torch.empty(256, device="cuda"), torch.ones((256, 2), dtype=torch.int32, device="cuda")

    def dense():
        fb.densify(0, 256, scr.x)
        hthedl.hth_head_score(scr.logits(256), 256, 10.0, 10.0, out, base=base)

    ms = []
    for f in (dense, lambda: screened.score(scr, fb, 256, 10, 10, out, base=base)):
        t = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        ms.append(float(np.median(t)))
    print("ms", ms)
    assert ms[1] < 10 * ms[0]
