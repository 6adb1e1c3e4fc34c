"""Device plans and the example view at the edges of their blocks: the count
pass's 32 hypotheses and 1,024 staged nodes, the example list's tiles of 2,048
words (131,072 individuals)."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    cfg = synth.small_config(n=3001, n_concepts=20, n_roles=3, n_data=2, n_pos=300, n_neg=300, seed_index=1501)
    kb = synth.make_kb(cfg)
    return cfg, kb, Oracle(kb)


def wide(k, seed):
    kids = [("exists", i % 3, i % 2, ("atom", i % 20)) for i in range(k - 1)] + [("atom", seed % 20)]
    return ("and" if seed % 2 else "or",) + tuple(kids)


@pytest.mark.parametrize("total", [31, 32, 33, 63, 64, 65])
def test_hypotheses_of_the_last_block(case, total):
    """One block short of full, full and one more; equal hypotheses on both sides of a block's end."""
    cfg, kb, oracle = case
    hyps = [wide(k, s) for k in (2, 4, 5, 9) for s in range(3)]
    hyps = (hyps + synth.make_sized_hypotheses(cfg, kb, count=total))[:total - 2] + hyps[:2]
    assert len(hyps) == total
    got = hthedl.Engine(kb, max_hyps=total).eval_batch_device(hyps)
    np.testing.assert_array_equal(got, oracle.coverages(hyps))


@pytest.mark.parametrize("nodes", [1023, 1024, 1025])
def test_nodes_of_a_block(case, nodes):
    """A block's nodes at the size of its LDS area, with a second block behind it."""
    cfg, kb, oracle = case
    hyps = [("exists", i % 3, 0, ("and", ("atom", i % 20), ("atom", (i + 7) % 20))) for i in range(31)]      # 4 nodes each
    left = nodes - 4 * 31
    pairs, odd = divmod(left - 1, 2)
    hyps.append(("or",) + tuple(("not", ("atom", i % 20)) for i in range(pairs)) + (("atom", 1),) * odd)
    assert hthedl.encode_batch(hyps)[0].shape[0] == nodes
    hyps += hyps[5:9] + [("and", hyps[3], ("atom", 2))]
    got = hthedl.Engine(kb, max_hyps=64).eval_batch_device(hyps)
    np.testing.assert_array_equal(got, oracle.coverages(hyps))


@pytest.mark.parametrize("n", [131_071, 131_072, 131_073, 262_209])
def test_example_list_of_several_tiles(monkeypatch, n):
    """Examples at both ends of every tile of the list, and a tile without any."""
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")
    cfg = synth.small_config(n=n, n_concepts=10, n_roles=2, cap=10, n_pos=1, n_neg=0, seed_index=1600)
    kb = synth.make_kb(cfg)
    edges = np.concatenate([np.arange(t - 70, t + 70) for t in (131_072, 262_144)] + [[0, 1, 63, 64, n - 65, n - 2, n - 1]])
    rng = np.random.default_rng(n)
    ex = np.unique(np.concatenate([edges, rng.integers(0, 131_072, 3000)]))     # the tile after: at its edges only
    ex = ex[(ex >= 0) & (ex < n)]
    kb.pos_bits, kb.neg_bits = synth.ids_to_bits(ex[::2], n), synth.ids_to_bits(ex[1::3], n)
    hyps = [("exists", i % 2, i // 2 % 2, ("atom", i % 10)) for i in range(20)]
    hyps += [("and", ("atom", i), ("not", hyps[i]), ("dge", 0, float(kb.deciles[0, i]))) for i in range(8)]
    hyps += [("exists", 0, 0, hyps[1]), ("not", ("atom", 4))]
    want = Oracle(kb).coverages(hyps)
    eng = hthedl.Engine(kb, max_hyps=64)
    np.testing.assert_array_equal(eng.eval_batch_device(hyps), want)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    eng.close()
