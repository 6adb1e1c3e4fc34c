"""The rows that shared passes write, word by word against the oracle: every T
width, rows walked by a lane (with several words' counters in one register)
and rows cut into slices, empty words at the start, at the end and between, a
last word that is full and one that is not."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("empty", [[0], [39], [0, 1, 7, 20, 21, 22, 39], [13]])
@pytest.mark.parametrize("per_dir", [3, 12, 30, 70])
@pytest.mark.parametrize("n", [64 * 40, 64 * 40 - 54])
def test_instances(n, per_dir, empty):
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    rng = np.random.default_rng(per_dir + n + len(empty))
    subjects = [x for x in range(n) if x // 64 not in empty and rng.random() < 0.4]
    edges = [[(x, int(y)) for x in subjects for y in np.sort(rng.choice(n, size=k, replace=False))] for k in (2, 40)]
    atoms = [np.flatnonzero(rng.random(n) < p) for p in np.linspace(0.02, 0.9, 10)]
    kb = synth.kb_from_edges(n, atoms, edges, data=rng.standard_normal((1, n)), pos=list(range(0, n, 9)),
                             neg=list(range(4, n, 11)))
    o = Oracle(kb)
    hyps = []
    for r in (0, 1):
        forms = [("exists", r, 0, ("atom", a)) for a in range(10)] + [("forall", r, 0, ("atom", a)) for a in range(10)]
        forms += [(op, c, r, 0, ("atom", a)) for a in range(10) for op, c in
                  (("atleast", 2), ("atmost", 0), ("atmost", 1), ("exactly", 0), ("exactly", 2), ("atleast", 0))]
        hyps += [forms[i] for i in rng.permutation(len(forms))[:per_dir]]
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    nodes, offs, ch = hthedl.encode_batch(hyps)
    eng.ensure_workspace(hthedl.hth_batch_workspace_bytes(eng.handle, nodes, offs, ch))
    sets = torch.full((len(hyps), eng.S), -1, dtype=torch.int64, device="cuda")
    counts = torch.empty((len(hyps), 2), dtype=torch.int32, device="cuda")
    eng.ws.fill_(255)      # a word that nothing writes shows
    hthedl.hth_eval_batch_sets(eng.handle, nodes, offs, ch, eng.ws, eng.ws_bytes, sets, counts)
    np.testing.assert_array_equal(counts.cpu().numpy().view(np.uint32), o.coverages(hyps))
    got = sets.cpu().numpy().view(np.uint64)[:, :eng.W]
    for h, row in zip(hyps, got):
        np.testing.assert_array_equal(row, o.ext_bits(h), err_msg=str(h))
    np.testing.assert_array_equal(eng.eval_batch_device([("exists", 0, 1, h) for h in hyps]),
                                  o.coverages([("exists", 0, 1, h) for h in hyps]))
