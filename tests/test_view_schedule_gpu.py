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
