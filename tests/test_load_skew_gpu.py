"""Loading roles that point into few objects: buckets of pairs at, below and
above the size that is counted and placed by slices (262,144 pairs, 65,536 a
slice), at the first, a middle and the last objects, next to ordinary ones."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth
from tests.test_load_gpu import hyps_for

pytestmark = pytest.mark.gpu


def kb_of(n, roles, seed):
    """roles: per role (subjects, [subjects][k] rising distinct objects)."""
    rng = np.random.default_rng(seed)
    kb = synth.kb_from_edges(n, [np.flatnonzero(rng.random(n) < 0.4) for _ in range(3)], [[] for _ in roles],
                             pos=range(0, n, 3), neg=range(1, n, 5))
    offs, tgs, base = np.zeros((len(roles), n + 1), np.int64), [], 0
    for i, (xs, ys) in enumerate(roles):
        deg = np.zeros(n, np.int64)
        deg[xs] = ys.shape[1]
        offs[i, 0], offs[i, 1:] = base, base + np.cumsum(deg)
        base += ys.size
        tgs.append(ys.ravel())
    kb.role_offsets, kb.role_targets = offs, np.concatenate(tgs).astype(np.int32)
    return kb


def objects(rng, count, k, lo, hi):
    return np.sort(rng.integers(lo, hi - k + 1, (count, k)), axis=1) + np.arange(k)


@pytest.mark.parametrize("pairs", [262_143, 262_144, 262_145, 330_001])
@pytest.mark.parametrize("lo", [0, 131_072, -1])
def test_bucket_sizes(pairs, lo):
    """`pairs` assertions to 40 objects (the last ones: lo -1), and 500 to any."""
    n = 300_007
    rng = np.random.default_rng(pairs + lo)
    lo = n - 40 if lo < 0 else lo
    xs = np.sort(rng.choice(n, size=pairs, replace=False)) if pairs < n else np.arange(n)
    ys = objects(rng, xs.size, 1, lo, lo + 40)
    if pairs >= n:               # two each for some of the subjects' worth
        xs, ys = np.arange(pairs // 2), objects(rng, pairs // 2, 2, lo, lo + 40)
    other = (np.sort(rng.choice(n, 250, replace=False)), objects(rng, 250, 2, 0, n))
    kb = kb_of(n, [(xs, ys), other, (np.arange(0), np.zeros((0, 1), np.int64))], seed=pairs)
    hyps = hyps_for(3)
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    np.testing.assert_array_equal(eng.eval_batch(hyps), Oracle(kb).coverages(hyps))
    for r in range(3):
        t = kb.role_targets[kb.role_offsets[r, 0]:kb.role_offsets[r, -1]]
        assert hthedl.hth_kb_max_degree(eng.handle, r, 1) == (int(np.bincount(t).max()) if t.size else 0)
    eng.close()


@pytest.mark.parametrize("roles,hot", [(1, 1), (1, 3000), (24, 5000)])
def test_several_buckets_and_widths(roles, hot):
    """Most of the assertions in one object, in a few buckets and in wide buckets (many roles); the others anywhere."""
    n = 200_000
    rng = np.random.default_rng(roles + hot)
    k = min(3, hot)
    parts = []
    for r in range(roles):
        xs = np.arange(0, n) if r % 8 == 0 else np.sort(rng.choice(n, 3000, replace=False))
        at = 77_777 if r % 16 == 0 else 3
        ys = objects(rng, xs.size, k, at, at + hot)
        ys[::7] = objects(rng, ys[::7].shape[0], k, 0, n)
        parts.append((xs, ys))
    if hot == 1:
        parts = [(np.arange(n), objects(rng, n, 1, 77_777, 77_778)), (np.arange(n), objects(rng, n, 2, 0, n)),
                 (np.arange(n), np.concatenate([np.full((n, 1), 5), objects(rng, n, 1, 9, n)], axis=1))]
    kb = kb_of(n, parts, seed=hot)
    hyps = hyps_for(min(len(parts), 3))
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    np.testing.assert_array_equal(eng.eval_batch(hyps), Oracle(kb).coverages(hyps))
    eng.close()
