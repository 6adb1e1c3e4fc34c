"""Example rows as a caller may hand them over after loading: bits past the last
individual are no examples (an index made of one would lie past every row)."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 9001, 131_071, 131_073])   # the last word's valid bits: 1, 41, 63, 1
def test_bits_past_the_last_individual(monkeypatch, n):
    import torch
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")
    cfg = synth.small_config(n=n, n_concepts=8, n_roles=2, cap=12, n_pos=n // 20 + 1, n_neg=n // 30 + 1, seed_index=1700)
    kb = synth.make_kb(cfg)
    hyps = [("exists", i % 2, i // 2 % 2, ("atom", i % 8)) for i in range(32)]
    hyps += [("and", ("not", h), ("dge", 0, float(kb.deciles[0, 3]))) for h in hyps[:8]]
    want = Oracle(kb).coverages(hyps)
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    rows = torch.zeros((2, eng.S), dtype=torch.int64, device="cuda")
    rows[:, :eng.W] = torch.from_numpy(np.stack([kb.pos_bits, kb.neg_bits]).view(np.int64)).cuda()
    rows[:, eng.W - 1] |= -1 << (n % 64)
    rows[:, eng.W:] = -1
    hthedl.hth_kb_set_examples(eng.handle, rows[0], rows[1])
    for name, got in (("device plan", eng.eval_batch_device(hyps)), ("host plan", eng.eval_batch(hyps)),
                      ("one by one", eng.eval_plain(hyps))):
        np.testing.assert_array_equal(got, want, err_msg=name)
    eng.close()


def test_speed_does_not_depend_on_the_examples_at_load():
    """Loaded with one example and given 25,000 of 400,000 later: the passes fill the chip as after loading with them
    (on one block a pass, as by the count at load, they take over four times as long)."""
    import torch
    n, roles, hyps_n = 400_000, 4, 64
    rng = np.random.default_rng(11)
    atoms = [np.flatnonzero(rng.random(n) < 0.3) for _ in range(8)]
    kb = synth.kb_from_edges(n, atoms, [[] for _ in range(roles)], pos=[5], neg=[])
    kb.role_offsets = (np.arange(roles)[:, None] * (8 * n) + np.arange(n + 1)[None] * 8).astype(np.int64)
    kb.role_targets = (np.sort(rng.integers(0, n - 8, (roles * n, 8)), axis=1) + np.arange(8)).astype(np.int32).ravel()
    late = hthedl.Engine(kb, max_hyps=hyps_n)
    ex = rng.choice(n, size=25_000, replace=False)
    kb.pos_bits, kb.neg_bits = synth.ids_to_bits(ex[:12_500], n), synth.ids_to_bits(ex[12_500:], n)
    known = hthedl.Engine(kb, max_hyps=hyps_n)
    hthedl.hth_kb_set_examples(late.handle, known.pos, known.neg)
    hyps = [("and", ("exists", i % roles, i // roles % 2, ("atom", i % 8)), ("not", ("forall", (i + 1) % roles, 0, ("atom", i // 8))))
            for i in range(hyps_n)]
    nodes, offs, ch = late.upload_batch(hyps)
    n_nodes, ms, out = nodes.shape[0] // 16, {}, {}
    for name, eng in (("late", late), ("known", known)):
        eng.ensure_plan_scratch(n_nodes)
        plan, nb = hthedl.hth_dplan_create(eng.handle, nodes, n_nodes, offs, hyps_n, ch, ch.shape[0], eng.dp_scratch, eng.dp_scratch_bytes)
        eng.ensure_workspace(nb)
        out[name] = torch.zeros((hyps_n, 2), dtype=torch.int32, device="cuda")
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            hthedl.hth_dplan_launch(plan, eng.ws, eng.ws_bytes, out[name])
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        ms[name] = float(np.median(times))
        hthedl.hth_dplan_destroy(plan)
    print("ms per launch", ms)
    assert torch.equal(out["late"], out["known"])
    assert ms["late"] < 2 * ms["known"]
