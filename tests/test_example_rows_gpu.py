"""Example rows as a caller may hand them over after loading: bits past the last
individual are no examples (an index made of one would lie past every row)."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 9001, 131_071, 131_073])   # the last word's valid bits: 1, 41, 63, 1
def test_bits_past_the_last_individual(monkeypatch, n):
    import torch
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")
    cfg = synth.small_config(n=n, n_concepts=8, n_roles=2, cap=12, n_pos=n // 20 + 1, n_neg=n // 30 + 1, seed_index=1700)
    kb = synth.make_kb(cfg)
    hyps = [("exists", i % 2, i // 2 % 2, ("atom", i % 8)) for i in range(32)]
    hyps += [("and", ("not", h), ("dge", 0, float(kb.deciles[0, 3]))) for h in hyps[:8]]
    want = Oracle(kb).coverages(hyps)
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    rows = torch.zeros((2, eng.S), dtype=torch.int64, device="cuda")
    rows[:, :eng.W] = torch.from_numpy(np.stack([kb.pos_bits, kb.neg_bits]).view(np.int64)).cuda()
    rows[:, eng.W - 1] |= -1 << (n % 64)
    rows[:, eng.W:] = -1
    hthedl.hth_kb_set_examples(eng.handle, rows[0], rows[1])
    for name, got in (("device plan", eng.eval_batch_device(hyps)), ("host plan", eng.eval_batch(hyps)),
                      ("one by one", eng.eval_plain(hyps))):
        np.testing.assert_array_equal(got, want, err_msg=name)
    eng.close()
