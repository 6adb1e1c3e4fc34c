"""The example view: batches whose coverage is evaluated over the examples only,
against the oracle, at the edges of its words and tiles, and with example rows
that change after the knowledge base was loaded (its size is counted on the
device at each launch)."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def view_everywhere(monkeypatch):
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")


def kb_with(n, n_ex, seed, **kw):
    cfg = synth.small_config(n=n, n_concepts=14, n_roles=4, cap=min(24, max(1, n // 2)), n_pos=1, n_neg=0, seed_index=1400 + seed, **kw)
    kb = synth.make_kb(cfg)
    rng = np.random.default_rng(seed)
    ex = rng.choice(n, size=n_ex, replace=False)
    kb.pos_bits, kb.neg_bits = synth.ids_to_bits(ex[:(n_ex + 1) // 2], n), synth.ids_to_bits(ex[n_ex // 3:], n)
    return cfg, kb


def zoo(kb):
    """Restrictions as roots, above and under others, shared between both places; counts a shared pass does not decide;
    thresholds and atoms at the root and in fillers; constants."""
    d = float(kb.deciles[0, 4])
    a, r = ("atom", 3), ("exists", 1, 0, ("atom", 2))
    under = ("atleast", 2, 0, 1, ("and", a, ("dge", 0, d)))
    out = [a, ("not", a), ("top",), ("bot",), r, ("not", r), under, ("exists", 2, 0, under), ("and", under, r, a),
           ("or", ("dge", 0, d), ("dle", 1, float(kb.deciles[1, 2])), ("not", ("dge", 0, d))),
           ("forall", 3, 1, ("or", r, under)), ("atmost", 12, 1, 0, a), ("and", ("atleast", 10, 0, 0, ("top",)), a),
           ("exactly", 1, 2, 1, ("not", a)), ("exists", 0, 0, ("top",)), ("forall", 0, 1, ("bot",)),
           ("exists", 1, 1, ("exists", 1, 0, ("exists", 3, 1, a)))]
    return out + out[3:9] + [("exists", i % 4, i % 2, ("atom", i % 14)) for i in range(70)]


def check(eng, kb, hyps):
    want = Oracle(kb).coverages(hyps)
    for name, got in (("device plan", eng.eval_batch_device(hyps)), ("host plan", eng.eval_batch(hyps))):
        bad = np.flatnonzero((got != want).any(axis=1))
        assert bad.size == 0, f"{name}: {hyps[bad[0]]} got {got[bad[0]]} want {want[bad[0]]}"


@pytest.mark.parametrize("n,n_ex", [(4, 1), (300, 63), (300, 64), (300, 65), (9001, 1023), (9001, 1025), (70_003, 4097)])
def test_example_counts(n, n_ex):
    cfg, kb = kb_with(n, n_ex, seed=n + n_ex)
    hyps = zoo(kb) + synth.make_hypotheses(cfg, kb, count=150, depth=5)
    check(hthedl.Engine(kb, max_hyps=len(hyps)), kb, hyps)


@pytest.mark.parametrize("edges", [300, 60_000])
def test_sparse_directions(edges):
    """Directions whose rows are mostly empty: short rows, compact T rows, examples without assertions."""
    cfg, kb = kb_with(90_001, 5000, seed=edges, total_edges=edges)
    check(hthedl.Engine(kb, max_hyps=400), kb, zoo(kb) + synth.make_hypotheses(cfg, kb, count=200, depth=4))


def test_heavy_and_long_rows(monkeypatch):
    """Rows of thousands of assertions among the examples."""
    monkeypatch.setenv("HTHEDL_HEAVY_MIN", "1024")
    n = 20_000
    rng = np.random.default_rng(5)
    rows = {int(x): np.sort(rng.choice(n, size=k, replace=False)) for x, k in zip(rng.choice(n, 300, replace=False), [5000] * 3 + [900] * 40 + [3] * 257)}
    edges = [[(x, int(y)) for x, ys in rows.items() for y in ys], [(int(y), x) for x, ys in rows.items() for y in ys[:50]],
             [(i, i + 1) for i in range(500)], []]
    atoms = [np.flatnonzero(rng.random(n) < p) for p in np.linspace(0.01, 0.9, 14)]
    kb = synth.kb_from_edges(n, atoms, edges, data=rng.standard_normal((2, n)), pos=sorted(rows)[:200],
                             neg=rng.choice(n, 700, replace=False))
    check(hthedl.Engine(kb, max_hyps=400), kb, zoo(kb))


def test_deep_regions():
    """Root programs beyond the register stack, and many leaves."""
    cfg, kb = kb_with(5000, 700, seed=9)
    deep = ("atom", 0)
    for i in range(12):
        deep = ("or", ("and", ("atom", i), ("exists", i % 4, 0, ("atom", 1))), ("and", ("atom", i + 1), deep))
    check(hthedl.Engine(kb, max_hyps=400), kb, [deep, ("not", deep), ("exists", 0, 0, deep)] + zoo(kb))


@pytest.mark.parametrize("now", ["none", "one", "all", "half"])
def test_examples_change_after_loading(now):
    """More, fewer or no examples than the plan's grids were sized for, by new rows and in place."""
    import torch
    n = 9001
    cfg, kb = kb_with(n, 200, seed=3)
    eng = hthedl.Engine(kb, max_hyps=400)
    hyps = zoo(kb) + synth.make_hypotheses(cfg, kb, count=100, depth=4)
    check(eng, kb, hyps)
    ids = {"none": [], "one": [n - 1], "all": np.arange(n), "half": np.arange(0, n, 2)}[now]
    kb.pos_bits, kb.neg_bits = synth.ids_to_bits(np.asarray(ids, np.int64), n), synth.ids_to_bits(np.asarray(ids, np.int64)[::3], n)
    rows = torch.zeros((2, eng.S), dtype=torch.int64, device="cuda")
    rows[:, :eng.W] = torch.from_numpy(np.stack([kb.pos_bits, kb.neg_bits]).view(np.int64)).cuda()
    hthedl.hth_kb_set_examples(eng.handle, rows[0], rows[1])
    check(eng, kb, hyps)
    kb.pos_bits = synth.ids_to_bits(np.arange(5, 800), n)
    rows[0, :eng.W] = torch.from_numpy(kb.pos_bits.view(np.int64)).cuda()
    check(eng, kb, hyps)


def test_set_rows_at_the_root_and_in_fillers():
    import torch
    cfg, kb = kb_with(9001, 900, seed=21)
    eng = hthedl.Engine(kb, max_hyps=64)
    o = Oracle(kb)
    parts = [("and", ("atom", 1), ("exists", 0, 0, ("atom", 2))), ("not", ("atom", 4))]
    table = torch.zeros((2, eng.S), dtype=torch.int64, device="cuda")
    for i, p in enumerate(parts):
        table[i, :eng.W] = torch.from_numpy(o.ext_bits(p).view(np.int64)).cuda()
    hthedl.hth_kb_set_sets(eng.handle, table, 2)
    forms = [lambda s: s, lambda s: ("not", s), lambda s: ("and", s, ("exists", 1, 1, ("atom", 5))),
             lambda s: ("exists", 2, 0, s), lambda s: ("or", ("forall", 1, 0, s), s)]
    hyps = [f(("set", i)) for i in (0, 1) for f in forms]
    want = o.coverages([f(parts[i]) for i in (0, 1) for f in forms])
    np.testing.assert_array_equal(eng.eval_batch_device(hyps), want)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)


def test_captured_launches_follow_the_examples():
    """A device plan's launch in a graph: replays read the example rows of the moment."""
    import torch
    cfg, kb = kb_with(9001, 400, seed=33)
    eng = hthedl.Engine(kb, max_hyps=400)
    hyps = zoo(kb)
    nodes, offs, ch = eng.upload_batch(hyps)
    n_nodes = nodes.shape[0] // 16
    eng.ensure_plan_scratch(n_nodes)
    plan, nb = hthedl.hth_dplan_create(eng.handle, nodes, n_nodes, offs, len(hyps), ch, ch.shape[0], eng.dp_scratch, eng.dp_scratch_bytes)
    eng.ensure_workspace(nb)
    out = torch.zeros((len(hyps), 2), dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        hthedl.hth_dplan_launch(plan, eng.ws, eng.ws_bytes, out, side)
    for k in (400, 2500, 7):
        ids = np.arange(0, k * 3, 3)
        kb.pos_bits = synth.ids_to_bits(ids, kb.n)
        eng.pos[:eng.W].copy_(torch.from_numpy(kb.pos_bits.view(np.int64)))
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), Oracle(kb).coverages(hyps))
        (torch.ones(1000, device="cuda") * k).sum().item()
    hthedl.hth_dplan_destroy(plan)
