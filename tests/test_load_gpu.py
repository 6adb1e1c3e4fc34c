"""Loading: the transposed roles, word lists and object ranks at the edges of
the load's chunks (8,192 assertions) and buckets, checked through evaluations
and degrees against the assertions; validation at the same edges."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


def make(n, rows, n_atoms=3, seed=0):
    """rows: per role, {subject: sorted objects}."""
    rng = np.random.default_rng(seed)
    offs, tgs, base = np.zeros((len(rows), n + 1), np.int64), [], 0
    for i, role in enumerate(rows):
        deg = np.zeros(n, np.int64)
        for x, ys in role.items():
            deg[x] = len(ys)
        offs[i, 0] = base
        offs[i, 1:] = base + np.cumsum(deg)
        tgs += [np.asarray(role[x], np.int64) for x in sorted(role)]
        base += int(deg.sum())
    atoms = [np.flatnonzero(rng.random(n) < 0.4) for _ in range(n_atoms)]
    kb = synth.kb_from_edges(n, atoms, [[] for _ in rows], pos=range(0, n, 3), neg=range(1, n, 5))
    kb.role_offsets = offs
    kb.role_targets = (np.concatenate(tgs) if tgs else np.zeros(0)).astype(np.int32)
    return kb


def check(kb, hyps):
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    want = Oracle(kb).coverages(hyps)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    np.testing.assert_array_equal(eng.eval_plain(hyps), want)
    for r in range(kb.n_roles):
        o = kb.role_offsets[r]
        t = kb.role_targets[o[0]:o[-1]]
        assert hthedl.hth_kb_max_degree(eng.handle, r, 0) == int(np.diff(o).max())
        assert hthedl.hth_kb_max_degree(eng.handle, r, 1) == (int(np.bincount(t).max()) if t.size else 0)
    eng.close()


def hyps_for(n_roles):
    out = []
    for r in range(n_roles):
        for inv in (0, 1):
            out += [("exists", r, inv, ("atom", 0)), ("forall", r, inv, ("atom", 1)), ("atleast", 2, r, inv, ("atom", 2)),
                    ("atmost", 1, r, inv, ("top",)), ("exists", r, 1 - inv, ("exists", r, inv, ("atom", 0)))]
    return out


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 70_001])
def test_random_roles(n):
    """Dense, sparse and empty roles; objects over every bucket."""
    rng = np.random.default_rng(n)
    rows = []
    for p, cap in ((1.0, 12), (0.02, 40), (0.0, 1)):
        rows.append({int(x): np.sort(rng.choice(n, size=min(n, int(rng.integers(1, cap + 1))), replace=False))
                     for x in np.flatnonzero(rng.random(n) < p)})
    check(make(n, rows, seed=n), hyps_for(3))


@pytest.mark.parametrize("sizes", [[8191, 1], [8192], [8193], [1, 8191, 8192, 5], [20_000, 3, 8200]])
def test_rows_across_chunks(sizes):
    """Rows that end at, before and after a chunk's end, with empty rows between them."""
    n = 30_000
    rng = np.random.default_rng(sum(sizes))
    role = {100 * i + 7: np.sort(rng.choice(n, size=k, replace=False)) for i, k in enumerate(sizes)}
    check(make(n, [role], seed=1), hyps_for(1))


@pytest.mark.parametrize("n,hot", [(20_000, 19_000), (300, 300), (200_000, 40_000)])
def test_one_object_of_many_subjects(n, hot):
    """One object holds more assertions than a bucket's stage (or all of them)."""
    rng = np.random.default_rng(n)
    role = {int(x): np.unique([5 % n, int(rng.integers(0, n))]) for x in np.sort(rng.choice(n, size=hot, replace=False))}
    check(make(n, [role, {3: [5 % n]}], seed=2), hyps_for(2))


@pytest.mark.parametrize("at", [1, 8191, 8192, 8193, 16_384])
@pytest.mark.parametrize("fault", ["equal", "falling", "range", "negative"])
def test_faulty_targets_are_found(at, fault):
    """A fault at the edges of a chunk; the same value at a row's start is none."""
    n = 40_000
    role = {9: np.arange(20_000), 11: np.arange(5, 30)}
    kb = make(n, [role])
    kb.role_targets = kb.role_targets.copy()
    kb.role_targets[at] = {"equal": at - 1, "falling": 0, "range": n, "negative": -1}[fault]
    with pytest.raises(hthedl.HthError) as e:
        hthedl.Engine(kb)
    assert e.value.status == -1
    assert ("strictly increasing" if fault in ("equal", "falling") else "outside") in str(e.value)
    role = {9: np.arange(at), 11: np.arange(5, 30)}     # row 11 starts at `at`, below row 9's last object
    hthedl.Engine(make(n, [role])).close()


def test_faulty_offsets_are_found():
    kb = make(1000, [{1: [2, 3], 500: [7]}, {4: [1]}])
    kb.role_offsets = kb.role_offsets.copy()
    kb.role_offsets[0, 200] = 1                          # falls back inside the role
    with pytest.raises(hthedl.HthError) as e:
        hthedl.Engine(kb)
    assert e.value.status == -1 and "monotone" in str(e.value)
