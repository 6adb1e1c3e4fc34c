"""Assertions between one role's last row and the next role's first offset belong
to no subject: neither direction holds them, whatever they are."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl
from tests.test_load_gpu import hyps_for, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gap", [1, 5, 8192, 20_000])
@pytest.mark.parametrize("n,last", [(3000, 2999), (3000, 100), (70_000, 8)])
def test_gap_between_roles(gap, n, last):
    """Gaps shorter and longer than a chunk; the last subject with and without a row; an empty role before a gap."""
    rng = np.random.default_rng(gap + n)
    rows = [{int(x): np.sort(rng.choice(n, size=4, replace=False)) for x in (1, 7, last)}, {},
            {int(x): [int(x) // 2] for x in range(0, n, 9)}]
    kb = make(n, rows, seed=gap)
    hyps = hyps_for(3)
    want = Oracle(kb).coverages(hyps)
    o, t, cut = kb.role_offsets.copy(), kb.role_targets, kb.role_offsets[1:, 0].copy()
    for r in (1, 2):
        o[r] += r * gap
    extra = [rng.integers(0, n, size=gap).astype(np.int32) for _ in (1, 2)]
    extra[1][0] = n + 7                                   # not an individual
    kb.role_targets = np.concatenate([t[:cut[0]], extra[0], t[cut[0]:cut[1]], extra[1], t[cut[1]:]])
    kb.role_offsets = o
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    np.testing.assert_array_equal(eng.eval_batch_device(hyps), want)
    np.testing.assert_array_equal(eng.eval_plain(hyps), want)
    for r, role in enumerate(rows):
        assert hthedl.hth_kb_max_degree(eng.handle, r, 0) == max([len(y) for y in role.values()], default=0)
        objects = np.concatenate([np.asarray(y, np.int64) for y in role.values()]) if role else np.zeros(0, np.int64)
        assert hthedl.hth_kb_max_degree(eng.handle, r, 1) == (np.bincount(objects).max() if objects.size else 0)
    eng.close()
