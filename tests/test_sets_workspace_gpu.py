"""hth_eval_batch_sets in the workspace that hth_batch_workspace_bytes reports:
a root that a shared pass covers has a region of its own there."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


def test_covered_roots_fit():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    cfg = synth.small_config(n=500, n_concepts=40, n_roles=6, cap=12, n_pos=20, n_neg=20, seed_index=1500)
    kb = synth.make_kb(cfg)
    hyps = [(op, r, d, ("atom", c)) for op in ("exists", "forall") for r in range(6) for d in (0, 1) for c in range(40)]
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    nodes, offs, ch = hthedl.encode_batch(hyps)
    n = hthedl.hth_batch_workspace_bytes(eng.handle, nodes, offs, ch)
    ws = torch.empty(n, dtype=torch.uint8, device=eng.device)
    rows = torch.zeros((len(hyps), eng.S), dtype=torch.int64, device=eng.device)
    counts = torch.empty((len(hyps), 2), dtype=torch.int32, device=eng.device)
    hthedl.hth_eval_batch_sets(eng.handle, nodes, offs, ch, ws, n, rows, counts)
    assert (counts.cpu().numpy().view(np.uint32) == Oracle(kb).coverages(hyps)).all()
