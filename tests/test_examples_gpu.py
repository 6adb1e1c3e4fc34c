"""Restrictions evaluated at the examples alone (one hypothesis, counts only),
against the oracle: sizes around a tile of example words, rows around the
lengths where a lane, then a wave walks them, every count predicate, value
roles with and without rows that stay with the general passes."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth
from test_parity_gpu import numeric_kb, string_kb

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def examples_everywhere(monkeypatch):
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")


def check(kb, hyps):
    got, want = hthedl.Engine(kb).eval_plain(hyps), Oracle(kb).coverages(hyps)
    bad = np.flatnonzero((got != want).any(axis=1))
    assert bad.size == 0, f"{hyps[bad[0]]} got {got[bad[0]]} want {want[bad[0]]}"


@pytest.mark.parametrize("n", [70, 2047, 2048, 2049, 6200])
@pytest.mark.parametrize("heavy_min", [None, "1024"])
def test_role_restrictions(monkeypatch, n, heavy_min):
    if heavy_min:
        monkeypatch.setenv("HTHEDL_HEAVY_MIN", heavy_min)
    cfg = synth.small_config(n=n, n_concepts=10, n_roles=3, s=1.05, cap=min(n // 2, 1500), n_pos=n // 16, n_neg=n // 16,
                             seed_index=1700 + n)
    kb = synth.make_kb(cfg)
    a, tail = ("atom", 3), np.uint64(1) << np.uint64((n - 1) % 64)
    kb.pos_bits[-1] |= tail                  # the last individual is an example
    hyps = []
    for r in range(3):
        for d in (0, 1):
            hyps += [("exists", r, d, a), ("forall", r, d, ("not", a)), ("exists", r, d, ("top",)), ("forall", r, d, ("bot",))]
            for c in (1, 2, 7, 8, 9, 31, 33, 200):
                hyps += [(op, c, r, d, ("atom", 5)) for op in ("atleast", "atmost", "exactly")]
    r = ("exists", 0, 1, a)
    hyps += [("not", r), ("and", r, ("exists", 1, 0, r)), ("or", ("not", r), ("atmost", 2, 2, 0, ("or", r, a))), ("forall", 2, 1, r)]
    check(kb, hyps)


@pytest.mark.parametrize("heavy_min", [None, "1024"])
def test_value_roles(monkeypatch, heavy_min):
    """Roles with a row above the heavy-row threshold and roles without one."""
    if heavy_min:
        monkeypatch.setenv("HTHEDL_HEAVY_MIN", heavy_min)
    kb, _ = numeric_kb()
    check(kb, synth.make_numeric_hypotheses(kb, 120, seed=5) + [("neq", p, 7.5) for p in range(3)])
    kb = string_kb()
    check(kb, synth.make_string_hypotheses(kb, 120, seed=7) +
          [("scontains", 1, b""), ("not", ("sequal", 0, kb.strings[2])), ("exists", 0, 1, ("scontains", 0, b"a"))])


def batches(kb, hyps):
    """eval_batch over all of them and over a few (fewer role nodes than a view takes)."""
    eng, want = hthedl.Engine(kb, max_hyps=len(hyps)), Oracle(kb).coverages(hyps)
    for part in (slice(None), slice(0, 3), slice(5, 12)):
        np.testing.assert_array_equal(eng.eval_batch(hyps[part]), want[part])
    return eng, want


def test_value_roles_in_batches():
    kb, _ = numeric_kb()
    batches(kb, synth.make_numeric_hypotheses(kb, 200, seed=6) +
            [("exists", r % 3, r % 2, ("and", ("nge", 0, 1.0), ("atom", r))) for r in range(20)])
    kb = string_kb()
    batches(kb, synth.make_string_hypotheses(kb, 200, seed=8) +
            [("and", ("scontains", 0, b"a"), ("exists", r % 2, r % 2, ("and", ("scontains", 0, b"a"), ("atom", r % 8)))) for r in range(20)])


def test_saved_plan_and_short_workspace(monkeypatch):
    """A compiled plan reads the example rows of the moment, and a workspace of the size that a knowledge base without
    the example view asks for still serves the batch."""
    import torch
    n = 9001
    cfg = synth.small_config(n=n, n_concepts=14, n_roles=4, cap=24, n_pos=200, n_neg=200, seed_index=1760)
    kb = synth.make_kb(cfg)
    hyps = synth.make_hypotheses(cfg, kb, count=200, depth=4)
    eng, want = batches(kb, hyps)
    nodes, offs, ch = hthedl.encode_batch(hyps)
    counts = torch.empty((len(hyps), 2), dtype=torch.int32, device="cuda")
    full = hthedl.hth_batch_workspace_bytes(eng.handle, nodes, offs, ch)
    monkeypatch.setenv("HTHEDL_VIEW_MIN", str(2**31))
    plain = hthedl.Engine(kb, max_hyps=len(hyps))
    less = hthedl.hth_batch_workspace_bytes(plain.handle, nodes, offs, ch)
    assert less < full
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    hthedl.hth_eval_batch(eng.handle, nodes, offs, ch, ws, less, counts)
    np.testing.assert_array_equal(counts.cpu().numpy().view(np.uint32), want)
    plan, need = hthedl.hth_plan_create(eng.handle, nodes, offs, ch)
    assert need <= full
    hthedl.hth_plan_upload(plan, ws, full)
    for ids in (np.arange(n), np.arange(0, n, 97), np.array([n - 1])):
        kb.pos_bits, kb.neg_bits = synth.ids_to_bits(ids, n), synth.ids_to_bits(ids[::2], n)
        rows = torch.zeros((2, eng.S), dtype=torch.int64, device="cuda")
        rows[:, :eng.W] = torch.from_numpy(np.stack([kb.pos_bits, kb.neg_bits]).view(np.int64)).cuda()
        hthedl.hth_kb_set_examples(eng.handle, rows[0], rows[1])
        hthedl.hth_plan_launch(plan, ws, full, counts)
        np.testing.assert_array_equal(counts.cpu().numpy().view(np.uint32), Oracle(kb).coverages(hyps))
    hthedl.hth_plan_destroy(plan)
