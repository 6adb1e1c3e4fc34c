"""Value-role restrictions that share a walk of a role's values, from one to sixteen
a walk and with a remainder, against sets taken from the values
themselves; and a time that walks of sixteen over few individuals could not
reach."""
import numpy as np
import pytest

from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "the gpu tests need an MI355X"
    return t


def value_kb(n):
    """Subject x: 0 to 3 values, of numeric role 0 in 0 .. 99 and of string role 0 among 100 words."""
    rng = np.random.default_rng(n)
    kb = synth.kb_from_edges(n, [np.arange(0, n, 3)], [[]], pos=range(0, n, 2), neg=range(1, n, 2))
    off = np.zeros((1, n + 1), np.int64)
    off[0, 1:] = np.cumsum(rng.integers(0, 4, n))
    v = rng.integers(0, 100, int(off[0, -1]))
    kb = synth.with_numeric_roles(kb, off, v.astype(np.float32))
    return synth.with_string_roles(kb, off, v.astype(np.int32), [b"w%02d" % i for i in range(100)]), off[0], v


def want(n, off, ok):
    """Even and odd subjects with a value that passes."""
    x = np.unique(np.repeat(np.arange(n), np.diff(off))[ok])
    return [int((x % 2 == 0).sum()), int((x % 2 == 1).sum())]


@pytest.mark.parametrize("n,tasks", [(65, 1), (4097, 40), (20001, 100), (524289, 15), (524289, 16), (524289, 33), (524289, 100)])
def test_shared_walks(torch, n, tasks):
    kb, off, v = value_kb(n)
    eng = hthedl.Engine(kb, max_hyps=256)
    hyps = [("nge", 0, float(100 - i)) for i in range(tasks)]
    hyps += [("sequal", 0, b"w%02d" % (i % 100)) if i % 3 else ("scontains", 0, b"%02d" % (i % 100)) for i in range(tasks)]
    exp = [want(n, off, v >= 100 - i) for i in range(tasks)] + [want(n, off, v == i % 100) for i in range(tasks)]
    np.testing.assert_array_equal(eng.eval_batch(hyps), np.array(exp, np.uint32))
    eng.close()


def test_few_individuals_take_a_walk_each(torch):
    """40 restrictions on one role of 5,000 individuals: 10.6 us, 22 in walks of sixteen."""
    kb, _, _ = value_kb(5000)
    eng = hthedl.Engine(kb, max_hyps=64)
    enc = hthedl.encode_batch([("nge", 0, 2.5 * i) for i in range(40)])
    plan, nb = hthedl.hth_plan_create(eng.handle, *enc)
    ws, out = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda"), torch.empty((40, 2), dtype=torch.int32, device="cuda")
    hthedl.hth_plan_upload(plan, ws, ws.numel())
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            hthedl.hth_plan_launch(plan, ws, ws.numel(), out)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 50)
    hthedl.hth_plan_destroy(plan)
    eng.close()
    assert best < 20, best


@pytest.mark.parametrize("n,tasks,every", [(65537, 8, 16), (65537, 40, 16), (262145, 5, 8), (262145, 6, 8), (262145, 7, 7),
                                           (524287, 2, 9), (524288, 1, 8), (524289, 3, 7)])
def test_few_restrictions_at_the_examples_or_over_everyone(torch, n, tasks, every):
    """Both sides of the rule's lines (an eighth of the individuals, 2^19 of them, their
    product with the restrictions), also below a role restriction."""
    kb, off, v = value_kb(n)
    pos, neg = np.arange(0, n, 2 * every), np.arange(every, n, 2 * every)
    kb.pos_bits[:], kb.neg_bits[:] = synth.ids_to_bits(pos, n), synth.ids_to_bits(neg, n)
    eng = hthedl.Engine(kb, max_hyps=128)
    hyps = [("nge", 0, float(100 - i)) for i in range(tasks)] + [("sequal", 0, b"w%02d" % i) for i in range(tasks)]
    hyps += [("exists", 0, 0, ("nge", 0, 50.0)), ("not", ("exists", 0, 0, ("sequal", 0, b"w07")))]
    exp = []
    for ok in [v >= 100 - i for i in range(tasks)] + [v == i for i in range(tasks)]:
        x = np.unique(np.repeat(np.arange(n), np.diff(off))[ok])
        exp.append([np.isin(pos, x).sum(), np.isin(neg, x).sum()])
    exp += [[0, 0], [len(pos), len(neg)]]      # the role has no assertions
    np.testing.assert_array_equal(eng.eval_batch(hyps), np.array(exp, np.uint32))
    eng.close()


def test_few_strings_of_many_examples_take_one_launch(torch):
    """Eight string hypotheses, some below a role, where a quarter of 65,537 individuals
    are examples: 26 us, 40 with the others at the examples."""
    n = 65537
    kb = synth.make_kb(synth.small_config(seed_index=900, n=n, n_concepts=10, n_roles=4, cap=30, n_pos=n // 9, n_neg=n // 9))
    kb = synth.with_string_roles(kb, *synth.string_roles(n, 2, 6))
    eng = hthedl.Engine(kb, max_hyps=64)
    enc = hthedl.encode_batch([eng.intern(h) for h in synth.make_string_hypotheses(kb, 8, 3)])
    plan, nb = hthedl.hth_plan_create(eng.handle, *enc)
    ws, out = torch.empty(max(nb, 256), dtype=torch.uint8, device="cuda"), torch.empty((8, 2), dtype=torch.int32, device="cuda")
    hthedl.hth_plan_upload(plan, ws, ws.numel())
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            hthedl.hth_plan_launch(plan, ws, ws.numel(), out)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 50)
    hthedl.hth_plan_destroy(plan)
    eng.close()
    assert best < 33, best
