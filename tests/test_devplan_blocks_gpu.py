"""Device plans at the edges of the count pass's blocks: 64 hypotheses, whose
nodes are kept in LDS up to 1,024 of them; wide nodes beyond the four children
that a key record holds; offsets that fall inside a block."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    cfg = synth.small_config(n=3001, n_concepts=20, n_roles=3, n_data=2, n_pos=300, n_neg=300, seed_index=1500)
    kb = synth.make_kb(cfg)
    return cfg, kb, Oracle(kb)


def wide(k, seed):
    """k children, most equal between seeds: the fifth and later decide."""
    kids = [("exists", i % 3, i % 2, ("atom", i % 20)) for i in range(k - 1)] + [("atom", seed % 20)]
    return ("and" if seed % 2 else "or",) + tuple(kids)


@pytest.mark.parametrize("count", [1, 63, 64, 65, 300])
@pytest.mark.parametrize("big", [0, 1100])
def test_blocks(case, count, big):
    cfg, kb, oracle = case
    hyps = synth.make_sized_hypotheses(cfg, kb, count=count)
    hyps += [("exists", 1, 0, wide(k, s)) for k in (4, 5, 6, 9) for s in range(4)] + [wide(5, s % 3) for s in range(6)]
    if big:      # one hypothesis with more nodes than a block's area
        hyps[count // 2] = ("or",) + tuple(("not", ("exists", i % 3, 0, ("atom", i % 20))) for i in range(big // 3))
    got = hthedl.Engine(kb, max_hyps=len(hyps)).eval_batch_device(hyps)
    np.testing.assert_array_equal(got, oracle.coverages(hyps))


def test_falling_offsets(case):
    cfg, kb, _ = case
    eng = hthedl.Engine(kb, max_hyps=64)
    nodes, offs, ch = hthedl.encode_batch(synth.make_sized_hypotheses(cfg, kb, count=70))
    bad = offs.copy()
    bad[30] = bad[28]
    with pytest.raises(hthedl.HthError) as e:
        eng.eval_batch_device(encoded=(nodes, bad, ch))
    assert e.value.status == -1 and "hypothesis 29" in str(e.value)
