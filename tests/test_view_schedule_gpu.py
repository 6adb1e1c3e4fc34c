"""The example view follows the schedule: no shared passes where the caller asked for none."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group_min", [0, 2])
def test_never_share(monkeypatch, group_min):
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")
    cfg = synth.small_config(n=5000, n_concepts=12, n_roles=3, n_pos=200, n_neg=150, seed_index=1900)
    kb = synth.make_kb(cfg)
    hyps = [("exists", i % 3, i // 3 % 2, ("atom", i % 12)) for i in range(40)]
    eng = hthedl.Engine(kb, max_hyps=64)
    hthedl.hth_kb_set_tuning(eng.handle, group_min=group_min)
    nodes, offs, ch = eng.upload_batch(hyps)
    eng.ensure_plan_scratch(nodes.shape[0] // 16)
    plan, _ = hthedl.hth_dplan_create(eng.handle, nodes, nodes.shape[0] // 16, offs, len(hyps), ch, ch.shape[0], eng.dp_scratch,
                                      eng.dp_scratch_bytes)
    assert (hthedl.hth_dplan_stats(plan)["shared_passes"] > 0) == (group_min > 0)
    hthedl.hth_dplan_destroy(plan)
    want = Oracle(kb).coverages(hyps)
    np.testing.assert_array_equal(eng.eval_batch_device(hyps), want)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    eng.close()


def test_many_directions(monkeypatch):
    """40,000 role directions in one view: the plan's time is that of as many passes without it, not of pairs of
    directions, and the copies' grids hold them."""
    import time
    import torch
    n, roles = 100, 20_000
    kb = synth.kb_from_edges(n, [np.arange(0, n, 2), np.arange(1, n, 5)], [[] for _ in range(roles)], pos=[0, 1, 2], neg=[3])
    kb.role_offsets = (np.arange(n + 1)[None] + n * np.arange(roles)[:, None]).astype(np.int64)
    kb.role_targets = ((np.arange(n)[None] + 1 + np.arange(roles)[:, None]) % n).astype(np.int32).ravel()
    hyps = [("exists", r, inv, ("atom", r % 2)) for r in range(roles) for inv in (0, 1)]
    enc, best, want = hthedl.encode_batch(hyps), {}, None
    for least in ("4294967295", "1"):
        monkeypatch.setenv("HTHEDL_VIEW_MIN", least)
        eng = hthedl.Engine(kb, max_nodes=1 << 17, max_hyps=len(hyps))
        times = []
        for _ in range(3):
            t = time.perf_counter()
            plan, nb = hthedl.hth_plan_create(eng.handle, *enc)
            times.append(time.perf_counter() - t)
            hthedl.hth_plan_destroy(plan)
        best[least] = min(times)
        got = eng.eval_batch_device(encoded=enc)
        want = got if want is None else want
        np.testing.assert_array_equal(got, want)
        eng.close()
    print("seconds", best)
    x = np.arange(3)
    for h in (0, 1, 777, 39_999):             # and by hand: the subject's one object, or the object's one subject
        r, inv = h // 2, h % 2
        y = (x - 1 - r) % n if inv else (x + 1 + r) % n
        assert want[h, 0] == (np.isin(y, np.arange(0, n, 2) if r % 2 == 0 else np.arange(1, n, 5))).sum()
    assert best["1"] < 4 * best["4294967295"]


@pytest.mark.parametrize("n,n_ex", [(65_536, 4000), (70_003, 17_500)])
def test_batches_below_the_view(n, n_ex):
    """Enough restrictions for shared passes, too few for the example view: one by one at the examples, as roots, above
    and under others, next to thresholds and rows that fillers read."""
    from tests.test_view_gpu import check, kb_with, zoo
    cfg, kb = kb_with(n, n_ex, seed=n)
    check(hthedl.Engine(kb, max_hyps=400), kb, zoo(kb))
