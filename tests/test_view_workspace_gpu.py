"""Workspaces with room for every row in full but not for the example view: the
plans run in them without it, next to workspaces that hold it."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2412_00802_amd import hthedl, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need an MI355X"
    cfg = synth.small_config(n=9001, n_concepts=14, n_roles=4, cap=24, n_pos=500, n_neg=400, seed_index=1800)
    kb = synth.make_kb(cfg)
    # many directions, few nodes on each: the view's offsets and targets outweigh the rows it saves
    hyps = [("exists", i % 4, i // 4 % 2, ("atom", i % 14)) for i in range(20)]
    hyps += [("and", ("atom", 3), ("not", h), ("dge", 0, float(kb.deciles[0, 3]))) for h in hyps[:6]]
    hyps += [("exists", 1, 1, ("and", ("atom", 2), hyps[0]))]
    return kb, hyps, Oracle(kb).coverages(hyps)


def sizes(monkeypatch, kb, hyps, create):
    """What the plan needs with the view and without it."""
    out = []
    for least in ("1", "4294967295"):
        monkeypatch.setenv("HTHEDL_VIEW_MIN", least)
        eng = hthedl.Engine(kb, max_hyps=64)
        plan, nb, destroy = create(eng)
        destroy(plan)
        eng.close()
        out.append(nb)
    monkeypatch.setenv("HTHEDL_VIEW_MIN", "1")
    assert out[0] > out[1]
    return out


def counts(torch, n):
    return torch.full((n, 2), 7, dtype=torch.int32, device="cuda")


def test_host_plan(monkeypatch, case):
    import torch
    kb, hyps, want = case
    enc = hthedl.encode_batch(hyps)
    full, least = sizes(monkeypatch, kb, hyps, lambda e: (*hthedl.hth_plan_create(e.handle, *enc), hthedl.hth_plan_destroy))
    eng = hthedl.Engine(kb, max_hyps=64)
    plan, nb = hthedl.hth_plan_create(eng.handle, *enc)
    assert nb == full
    spaces = [torch.empty(b, dtype=torch.uint8, device="cuda") for b in (full, least, full - 256)]
    with pytest.raises(hthedl.HthError) as e:
        hthedl.hth_plan_upload(plan, spaces[1], least - 256)
    assert e.value.status == -3
    for ws in spaces:
        hthedl.hth_plan_upload(plan, ws, ws.numel())
    for ws in spaces + spaces[::-1]:
        out = counts(torch, len(hyps))
        hthedl.hth_plan_launch(plan, ws, ws.numel(), out)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)
    # a workspace with the view's tables, named shorter: refused, as tables that do not fit
    with pytest.raises(hthedl.HthError) as e:
        hthedl.hth_plan_launch(plan, spaces[0], least, out)
    assert e.value.status == -3
    hthedl.hth_plan_destroy(plan)
    eng.close()


def test_device_plan(monkeypatch, case):
    import torch
    kb, hyps, want = case
    eng = hthedl.Engine(kb, max_hyps=64)
    nodes, offs, ch = eng.upload_batch(hyps)
    n_nodes = nodes.shape[0] // 16

    def create(e):
        e.ensure_plan_scratch(n_nodes)
        return *hthedl.hth_dplan_create(e.handle, nodes, n_nodes, offs, len(hyps), ch, ch.shape[0], e.dp_scratch,
                                        e.dp_scratch_bytes), hthedl.hth_dplan_destroy

    full, least = sizes(monkeypatch, kb, hyps, create)
    eng.close()
    eng = hthedl.Engine(kb, max_hyps=64)
    plan, nb, _ = create(eng)
    assert nb == full
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")

    def launch(size):
        out = counts(torch, len(hyps))
        hthedl.hth_dplan_launch(plan, ws, size, out)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)

    launch(full)
    for _ in range(2):                       # too short for either form: refused, and the plan is as it was
        with pytest.raises(hthedl.HthError) as e:
            launch(least - 256)
        assert e.value.status == -3
        launch(full)
    for size in (least, full, least):
        launch(size)
    hthedl.hth_dplan_destroy(plan)
    # a captured launch keeps its layout: a short workspace is refused from then on, and the graph's replays are right
    plan, _, _ = create(eng)
    out, side = counts(torch, len(hyps)), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        with pytest.raises(hthedl.HthError) as e:
            hthedl.hth_dplan_launch(plan, ws, least, out, side)
        assert e.value.status == -3
        hthedl.hth_dplan_launch(plan, ws, full, out, side)
    for _ in range(3):
        with pytest.raises(hthedl.HthError) as e:
            launch(least)
        assert e.value.status == -3
        out.fill_(7)
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)
    del g
    hthedl.hth_dplan_destroy(plan)
    eng.close()


def test_view_that_would_double_a_large_workspace(monkeypatch):
    """80 directions of 2M individuals: 1.3 GB of offsets for rows of 20 MB; the plan leaves the view out."""
    import torch
    n, roles = 2_000_003, 80
    kb = synth.kb_from_edges(n, [np.arange(0, n, 3), np.arange(0, n, 7)], [[] for _ in range(roles)], pos=range(0, 4000, 2), neg=range(1, 4000, 2))
    off = np.zeros((roles, n + 1), np.int64)
    off[:, 9:] = 2
    kb.role_offsets = off + 2 * np.arange(roles)[:, None]
    kb.role_targets = np.tile(np.array([3, 7], np.int32), roles)
    hyps = [("exists", r, inv, ("atom", 0)) for r in range(roles) for inv in (0, 1)]
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    want = np.zeros((len(hyps), 2), np.uint32)
    want[::2, 0] = 1                          # subject 8 (3 is of atom 0), an even number: positive
    nodes, offs, ch = eng.upload_batch(hyps)
    eng.ensure_plan_scratch(nodes.shape[0] // 16)
    plan, nb = hthedl.hth_dplan_create(eng.handle, nodes, nodes.shape[0] // 16, offs, len(hyps), ch, ch.shape[0], eng.dp_scratch,
                                       eng.dp_scratch_bytes)
    hthedl.hth_dplan_destroy(plan)
    host, hb = hthedl.hth_plan_create(eng.handle, *hthedl.encode_batch(hyps))
    hthedl.hth_plan_destroy(host)
    assert max(nb, hb, hthedl.hth_batch_workspace_bytes(eng.handle, *hthedl.encode_batch(hyps))) < 1 << 30
    np.testing.assert_array_equal(eng.eval_batch_device(hyps), want)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    eng.close()


def test_view_beside_a_small_plan_is_kept(monkeypatch):
    """The same directions under restrictions of their own, whose rows are a sixtieth of
    what the view adds: its room is asked for, and less is served without it."""
    import torch
    n, roles = 2_000_003, 80
    kb = synth.kb_from_edges(n, [np.arange(0, n, 3), np.arange(0, n, 7)], [[] for _ in range(roles)], pos=range(0, 4000, 2), neg=range(1, 4000, 2))
    off = np.zeros((roles, n + 1), np.int64)
    off[:, 9:] = 2
    kb.role_offsets = off + 2 * np.arange(roles)[:, None]
    kb.role_targets = np.tile(np.array([3, 8], np.int32), roles)      # subject 8 reaches itself
    hyps = [("exists", r, inv, ("exists", r, 0, ("atom", 0))) for r in range(roles) for inv in (0, 1)]
    eng = hthedl.Engine(kb, max_hyps=len(hyps))
    # 8 (positive) reaches 3, of atom 0, so it holds the inner restriction; then 8 itself, and 3 (negative) over the inverse
    want = np.zeros((len(hyps), 2), np.uint32)
    want[:, 0] = 1
    want[1::2, 1] = 1
    nodes, offs, ch = eng.upload_batch(hyps)
    eng.ensure_plan_scratch(nodes.shape[0] // 16)
    plan, nb = hthedl.hth_dplan_create(eng.handle, nodes, nodes.shape[0] // 16, offs, len(hyps), ch, ch.shape[0], eng.dp_scratch,
                                       eng.dp_scratch_bytes)
    assert nb > 1 << 30
    for room in (nb, 1 << 29):
        ws, out = torch.empty(room, dtype=torch.uint8, device="cuda"), counts(torch, len(hyps))
        hthedl.hth_dplan_launch(plan, ws, room, out)
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)
    hthedl.hth_dplan_destroy(plan)
    np.testing.assert_array_equal(eng.eval_batch(hyps), want)
    eng.close()
