"""Performance cases of the hypothesis-evaluation engine.

Each case is a piece of work that a program built on this package has it do,
through the public entry points of ``paper_2412_00802_amd``: hypotheses one at
a time, batches planned on the host and on the device, a refinement round,
instance sets for the set table, concrete roles, loading a knowledge base, a
screener training step and the scoring of refinement candidates.  Sizes come
from the workload descriptions of ``synth.CONFIGS`` and from the tests.

All inputs are drawn on the GPU (or vectorised on the host) from the seed, with
the distributions of ``synth``: concept trees whose children keep half of their
parent's members, Zipf out-degrees with distinct uniform targets, normal
property columns with missing values and decile thresholds, random trees of
DL operators with shared subtrees.

Counts, bit rows and specs are whole numbers and compared for equality, so
``exact`` has values for the screener's cases only.
"""
import math
import types

import numpy as np
import torch

from paper_2412_00802_amd import hthedl, screened
from paper_2412_00802_amd.screener import D_H1, D_H2, D_IN, FeatureBatch, Screener, init_params

DEV = "cuda"
MISSING = 0.1            # share of individuals without a value of a property
STRINGS, PATTERNS = 1000, 16
LEAVES_PER_STEP = 0.45   # random trees: share of pushes, then of one-child operators
UNARY = 0.35
MOST_EDGES = 60_000_000  # of a drawn knowledge base


# The knowledge bases.  edges = 0: every individual is a subject of every role.
TINY = {"n": 10_000, "concepts": 64, "roles": 8, "zipf": 2.0, "cap": 64, "edges": 0, "props": 4}
DENSE = {"n": 1_000_000, "concepts": 512, "roles": 32, "zipf": 1.8, "cap": 1024, "edges": 0, "props": 16}
SPARSE = {"n": 4_000_000, "concepts": 1024, "roles": 48, "zipf": 1.6, "cap": 8192, "edges": 40_000_000, "props": 32}
LARGE = {"n": 32_000_000, "concepts": 256, "roles": 16, "zipf": 1.5, "cap": 65_536, "edges": 125_000_000, "props": 32}
MEDIUM = {"n": 200_003, "concepts": 256, "roles": 12, "zipf": 1.6, "cap": 1024, "edges": 2_000_000, "props": 8}


def listed():
    return [
        # a service that answers single questions on a small knowledge base: launches and host planning count
        {"name": "plain_small", "kind": "plain", **TINY, "hyps": 8, "nodes": 6, "instances": True},
        # the same on a million individuals whose roles hold 8 assertions per subject: the single-node passes
        {"name": "plain_mid", "kind": "plain", **{**DENSE, "concepts": 128, "roles": 8, "props": 8}, "hyps": 16,
         "nodes": 8, "instances": False},
        # a small learner's batch, planned on the host
        {"name": "batch_small", "kind": "batch", **TINY, "hyps": 256, "nodes": 8},
        # the paper-scale batch over dense roles (266M assertions), planned on the host
        {"name": "batch_dense", "kind": "batch", **DENSE, "hyps": 4096, "nodes": 10},
        # an ordinary search step: a sparse KB of odd size, node arrays resident, planned on the device
        {"name": "device_medium", "kind": "device", **MEDIUM, "hyps": 8192, "nodes": 6.5},
        # the uneven batch of 65,536 hypotheses over 4M individuals, planned on the device
        {"name": "device_uneven", "kind": "device", **SPARSE, "hyps": 65_536, "nodes": 6.5},
        # a refinement round on the largest KB: 256 parents in the set table, candidates made on the device
        {"name": "round_large", "kind": "round", **LARGE, "parents": 256, "per": 64},
        # the instance sets of the hypotheses kept for the next round
        {"name": "sets_fill", "kind": "sets", **{**SPARSE, "n": 3_999_971, "concepts": 256, "roles": 16,
                                                 "edges": 13_000_000, "props": 8}, "hyps": 300, "nodes": 6.5},
        # multi-valued numeric roles and string roles (MIN/MAX/EXACT, EQUAL/CONTAIN) inside hypotheses
        {"name": "concrete_roles", "kind": "concrete", **{**MEDIUM, "n": 1_000_000, "edges": 10_000_000}, "nums": 4,
         "strs": 4, "hyps": 256, "nodes": 5},
        # a KB handed over by the caller: validated, its derived layouts built, the first questions answered
        {"name": "load_dense", "kind": "load", **{**DENSE, "concepts": 128, "roles": 16, "props": 4}, "hyps": 16,
         "nodes": 6},
        # one optimiser step of the screener on a minibatch of refinement pairs
        {"name": "train_step", "kind": "train", "rows": 1024, "parents": 256, "nodes": 8, "loss": "mse"},
        # screening refinement candidates: features, predicted F1, the best 2%
        {"name": "score_candidates", "kind": "score", "rows": 262_157, "parents": 2048, "nodes": 8, "batch": 8192},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a kind by its share of use, sizes over its whole range."""
    kind = rng.choice(["plain", "plain", "batch", "batch", "device", "device", "round", "sets", "concrete", "load",
                       "load", "train", "score"])
    if kind == "train":
        return {"kind": kind, "rows": _log(rng, 64, 8192), "parents": _log(rng, 16, 1024),
                "nodes": rng.choice([4, 6.5, 8, 12]), "loss": rng.choice(["mse", "bce"])}
    if kind == "score":
        return {"kind": kind, "rows": _log(rng, 2000, 400_000), "parents": _log(rng, 64, 4096),
                "nodes": rng.choice([4, 6.5, 8, 12]), "batch": rng.choice([4096, 8192, 16384])}
    n = _log(rng, 1000, 4_000_000)
    kb = {"n": n, "concepts": _log(rng, 16, 512), "roles": _log(rng, 2, 24), "zipf": rng.choice([1.5, 1.6, 1.8, 2.0]),
          "cap": min(_log(rng, 16, 8192), max(16, n // 20)), "edges": 0, "props": rng.randint(1, 16)}
    if rng.random() < 0.6:    # sparse roles: few individuals are subjects
        kb["edges"] = int(kb["roles"] * n * math.exp(rng.uniform(math.log(0.05), math.log(2.0))))
    if (kb["edges"] or kb["roles"] * n * _mean_degree(kb["zipf"], kb["cap"])) > MOST_EDGES:
        kb["edges"] = MOST_EDGES
    hyps = {"plain": _log(rng, 1, 24), "batch": _log(rng, 16, 4096), "device": _log(rng, 256, 16_384), "sets": _log(rng, 8, 400),
            "concrete": _log(rng, 8, 512), "load": _log(rng, 1, 64), "round": 0}[kind]
    case = {"kind": kind, **kb}
    if kind == "round":
        return {**case, "parents": _log(rng, 8, 256), "per": _log(rng, 8, 64)}
    case.update(hyps=hyps, nodes=rng.choice([4, 6.5, 8, 10]))
    if kind == "plain":
        case["instances"] = rng.random() < 0.5
    if kind == "concrete":
        case.update(nums=rng.randint(1, 4), strs=rng.randint(1, 4))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _words(gen, rows, words):
    """Random 64-bit words, int64 [rows][words]."""
    return torch.randint(-2**31, 2**31, (rows, 2 * words), dtype=torch.int32, device=DEV, generator=gen).view(torch.int64)


def _rows(bits, n, stride):
    """[rows][W] words as bit rows of the library: bits past n and padding words are zero."""
    out = torch.zeros((bits.shape[0], stride), dtype=torch.int64, device=DEV)
    out[:, :bits.shape[1]] = bits
    if n % 64:
        out[:, bits.shape[1] - 1] &= (1 << (n % 64)) - 1
    return out


def _csr(gen, n, cdf, p):
    """One role: degrees by the cdf over 1.., a subject with probability p, distinct targets in rising order."""
    deg = torch.searchsorted(cdf, torch.rand(n, dtype=torch.float64, device=DEV, generator=gen), right=True) + 1
    deg.clamp_(max=cdf.shape[0])
    if p < 1:
        deg *= torch.rand(n, device=DEV, generator=gen) < p
    src = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    key = src * n + torch.randint(0, n, (src.shape[0],), device=DEV, generator=gen)
    key = torch.unique_consecutive(torch.sort(key)[0])
    src = torch.div(key, n, rounding_mode="floor")
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=off[1:])
    return off, (key - src * n).to(torch.int32)


def _zipf(s, cap):
    d = torch.arange(1, cap + 1, dtype=torch.float64, device=DEV)
    p = d ** -s
    return torch.cumsum(p, 0) / p.sum(), float((d * p).sum() / p.sum())


def _chain(parts, offs):
    """Per-role arrays one after the other, offsets absolute: (offsets [R][N+1], values)."""
    base, rows = 0, []
    for o in offs:
        rows.append(o + base)
        base += int(o[-1])
    return torch.stack(rows), torch.cat(parts)


def _make_kb(case, gen):
    """The arrays that a program hands to hth_kb_create, on the GPU."""
    k = types.SimpleNamespace()
    n = k.n = case["n"]
    w, k.stride = (n + 63) // 64, hthedl.stride_for(n)
    levels, sizes = [], [len(a) for a in np.array_split(np.arange(case["concepts"]), 6)]
    for size in sizes:
        if not levels:
            bits = _words(gen, size, w) & (_words(gen, size, w) | (_words(gen, size, w) & _words(gen, size, w)))
        elif size:
            up = levels[-1]
            bits = up[torch.randint(0, up.shape[0], (size,), device=DEV, generator=gen)] & _words(gen, size, w)
        else:
            break
        levels.append(bits)
    k.concepts = _rows(torch.cat(levels), n, k.stride)
    some = [_words(gen, 1, w) & _words(gen, 1, w) & _words(gen, 1, w) & _words(gen, 1, w) for _ in range(2)]
    k.pos, k.neg = _rows(levels[0][:1] & some[0], n, k.stride)[0], _rows(~levels[0][:1] & some[1], n, k.stride)[0]
    del levels
    cdf, mean = _zipf(case["zipf"], case["cap"])
    p = min(1.0, case["edges"] / (case["roles"] * n * mean)) if case["edges"] else 1.0
    made = [_csr(gen, n, cdf, p) for _ in range(case["roles"])]
    k.offsets, k.targets = _chain([t for _, t in made], [o for o, _ in made])
    k.data = torch.randn((case["props"], n), device=DEV, generator=gen)
    for col in k.data:
        col[torch.rand(n, device=DEV, generator=gen) < MISSING] = math.nan
    some = k.data[:, :100_000].cpu().numpy()
    k.deciles = np.stack([np.sort(c[~np.isnan(c)])[[j * (int((~np.isnan(c)).sum()) - 1) // 10 for j in range(1, 10)]]
                          for c in some])
    d = k.desc = hthedl.KBDesc()
    d.n_individuals, d.stride_words, d.n_concepts, d.concept_bits = n, k.stride, case["concepts"], k.concepts.data_ptr()
    d.n_roles, d.n_edges = case["roles"], k.targets.shape[0]
    d.role_offsets, d.role_targets = k.offsets.data_ptr(), k.targets.data_ptr()
    d.n_data, d.data = case["props"], k.data.data_ptr()
    d.pos_bits, d.neg_bits = k.pos.data_ptr(), k.neg.data_ptr()
    k.derived_bytes = hthedl.hth_kb_derived_bytes(d)
    k.derived = torch.empty(k.derived_bytes, dtype=torch.uint8, device=DEV)
    return k


class _Handle:
    """A loaded KB; the handle goes with the object."""

    def __init__(self, k):
        self.kb, self.handle = k, hthedl.hth_kb_create(k.desc, k.derived, k.derived_bytes)

    def __del__(self):
        hthedl.hth_kb_destroy(self.handle)


def _hypotheses(rng, count, mean, concepts, roles, deciles, share=0.3, nums=None, strs=0, most=31):
    """Random hypotheses as node arrays (nodes, offsets, children, children offsets), drawn side by side.

    Node counts are geometric.  Each is grown in postfix order on a stack: a leaf, an operator on the top, or a
    conjunction/disjunction of the top two or three.  The first half of a share of them follows another
    hypothesis's draws, so that subtrees recur across the batch."""
    k = np.minimum(rng.geometric(1.0 / mean, count), most)
    most = int(k.max())
    u = rng.random((most, 6, count))
    other = np.where(rng.random(count) < share, rng.integers(0, count, count), np.arange(count))
    half = np.minimum(k, k[other]) // 2
    f = {name: np.zeros((count, most), np.int64) for name in ("op", "inv", "arity", "arg", "child", "q")}
    stack, depth = np.zeros((count, most + 1), np.int64), np.zeros(count, np.int64)
    kids, n_kids = np.zeros((count, most + 1), np.int64), np.zeros(count, np.int64)
    o = hthedl.OPS
    unary = np.array([o["not"], o["exists"], o["forall"], o["atleast"], o["atmost"]])
    bits = deciles.astype(np.float32).view(np.uint32).astype(np.int64)
    for t in range(most):
        a = np.flatnonzero(k > t)
        v = np.where(t < half[a], u[t][:, other[a]], u[t][:, a])
        d, left = depth[a], k[a] - t - 1
        push, one = left >= d, (d >= 1) & (left >= d - 1)
        act = np.where(v[0] < LEAVES_PER_STEP, 0, np.where(v[0] < LEAVES_PER_STEP + UNARY, 1, 2))
        act = np.where((act == 0) & ~push, 1, act)
        act = np.where((act == 2) & (d < 2), 1, act)
        act = np.where((act == 1) & ~one, np.where(d >= 2, 2, 0), act)
        # leaves
        i, x = a[act == 0], v[:, act == 0]
        leaf = np.select([x[1] < 0.75, x[1] < 0.95], [0, 1], 2)
        if nums is not None:      # concrete roles: two leaves of three read them
            leaf = np.where(x[5] < 0.33, leaf, np.where(x[5] < 0.66, 3, 4))
        prop = (x[2] * bits.shape[0]).astype(np.int64)
        f["op"][i, t] = np.choose(leaf, [o["atom"], np.where(x[4] < 0.5, o["dge"], o["dle"]), o["top"],
                                         np.choose((x[4] * 3).astype(int), [o["nge"], o["nle"], o["neq"]]),
                                         np.where(x[4] < 0.4, o["sequal"], o["scontains"])])
        f["arg"][i, t] = np.choose(leaf, [(x[2] * concepts).astype(np.int64), prop, 0,
                                          (x[2] * (len(nums) if nums is not None else 1)).astype(np.int64),
                                          (x[2] * max(1, strs)).astype(np.int64)])
        f["q"][i, t] = np.select([leaf == 1, leaf == 3, leaf == 4],
                                 [bits[prop, (x[3] * 9).astype(np.int64)],
                                  nums[(x[2] * len(nums)).astype(np.int64), (x[3] * nums.shape[1]).astype(np.int64)] if nums is not None else 0,
                                  np.where(x[4] < 0.4, (x[3] * STRINGS).astype(np.int64), (x[3] * PATTERNS).astype(np.int64))], 0)
        stack[i, depth[i]] = t
        depth[i] += 1
        # operators with one child
        i, x = a[act == 1], v[:, act == 1]
        op = unary[(x[1] * 5).astype(np.int64)]
        role = op != o["not"]
        f["op"][i, t], f["child"][i, t] = op, stack[i, depth[i] - 1]
        f["arg"][i, t] = np.where(role, (x[2] * roles).astype(np.int64), 0)
        f["inv"][i, t] = role & (x[3] < 0.5)
        f["q"][i, t] = np.where(op >= o["atleast"], 1 + (x[4] * 4).astype(np.int64), 0)
        stack[i, depth[i] - 1] = t
        # conjunctions and disjunctions
        i, x = a[act == 2], v[:, act == 2]
        arity = np.where((x[1] < 0.5) & (depth[i] >= 3), 3, 2)
        f["op"][i, t], f["arity"][i, t], f["child"][i, t] = np.where(x[2] < 0.5, o["and"], o["or"]), arity, n_kids[i]
        for j in range(3):
            g, s = i[j < arity], arity[j < arity]
            kids[g, n_kids[g] + j] = stack[g, depth[g] - s + j]
        n_kids[i] += arity
        depth[i] -= arity - 1
        stack[i, depth[i] - 1] = t
    coffs = np.concatenate([[0], np.cumsum(n_kids)])
    f["child"] += np.where(f["arity"] > 0, coffs[:-1, None], 0)
    at = np.arange(most) < k[:, None]
    nodes = np.zeros(int(k.sum()), hthedl.NODE_DTYPE)
    for name, v in f.items():
        nodes[name] = v[at]
    offs = np.concatenate([[0], np.cumsum(k)])
    return nodes, offs.astype(np.uint32), kids[np.arange(most + 1) < n_kids[:, None]].astype(np.uint32), coffs


def _alone(enc):
    """Each hypothesis as a (nodes, children) pair of its own."""
    nodes, offs, kids, coffs = enc
    out = []
    for h in range(offs.shape[0] - 1):
        own = nodes[offs[h]:offs[h + 1]].copy()
        own["child"][own["arity"] > 0] -= np.uint32(coffs[h])
        out.append((own, kids[coffs[h]:coffs[h + 1]].copy()))
    return out


def _concrete(case, gen, s):
    """Numeric and string concrete roles registered on the KB; -> sample values per numeric role, as float bits."""
    n, h = case["n"], s.load.handle
    cdf, _ = _zipf(1.6, 16)
    made = [_csr(gen, n, cdf, 0.5) for _ in range(case["nums"] + case["strs"])]
    s.num_off, flat = _chain([t for _, t in made[:case["nums"]]], [o for o, _ in made[:case["nums"]]])
    s.num_val = torch.round(torch.randn(flat.shape[0], device=DEV, generator=gen) * 16) / 16
    size = hthedl.hth_numeric_derived_bytes(h, case["nums"], flat.shape[0])
    s.num_der = torch.empty(max(256, size), dtype=torch.uint8, device=DEV)
    hthedl.hth_kb_set_numeric(h, case["nums"], s.num_off, s.num_val, flat.shape[0], s.num_der, size)
    s.str_off, flat = _chain([t for _, t in made[case["nums"]:]], [o for o, _ in made[case["nums"]:]])
    s.str_ids = torch.randint(0, STRINGS, (flat.shape[0],), dtype=torch.int32, device=DEV, generator=gen)
    lens = torch.randint(1, 13, (STRINGS,), device=DEV, generator=gen)
    s.dic_off = torch.zeros(STRINGS + 1, dtype=torch.int64, device=DEV)
    s.dic_off[1:] = torch.cumsum(lens, 0)
    s.dic = torch.randint(97, 103, (int(s.dic_off[-1]),), dtype=torch.uint8, device=DEV, generator=gen)
    size = hthedl.hth_string_derived_bytes(h, case["strs"], flat.shape[0])
    s.str_der = torch.empty(max(256, size), dtype=torch.uint8, device=DEV)
    hthedl.hth_kb_set_strings(h, case["strs"], s.str_off, s.str_ids, flat.shape[0], STRINGS, s.dic_off, s.dic, s.str_der, size)
    s.pat_off = torch.arange(PATTERNS + 1, device=DEV) * 2
    s.pat = torch.randint(97, 103, (2 * PATTERNS,), dtype=torch.uint8, device=DEV, generator=gen)
    hthedl.hth_kb_set_patterns(h, PATTERNS, s.pat_off, s.pat)
    return s.num_val[:64 * case["nums"]].reshape(case["nums"], -1).cpu().numpy().view(np.uint32).astype(np.int64)


def _refinements(rng, rows, parents, mean):
    """Parents and their one-step refinements as node arrays: a conjunct added (an atom, or an existential over
    one), or an atom inside replaced.  -> (parents, candidates, parent of each candidate)."""
    dec = np.sort(rng.standard_normal((32, 9)).astype(np.float32))
    p = _hypotheses(rng, parents, mean, 1024, 48, dec)
    pi = np.sort(rng.integers(0, parents, rows))
    p_len, p_kid = np.diff(p[1].astype(np.int64))[pi], np.diff(p[3])[pi]
    spot = (rng.random(rows) * p_len).astype(np.int64)
    swap = (rng.random(rows) < 0.3) & (p[0]["op"][p[1].astype(np.int64)[pi] + spot] == hthedl.OPS["atom"])
    deep = ~swap & (rng.random(rows) < 0.4)
    more = np.where(swap, 0, np.where(deep, 3, 2))
    offs = np.concatenate([[0], np.cumsum(p_len + more)])
    coffs = np.concatenate([[0], np.cumsum(p_kid + 2 * ~swap)])
    nodes = np.zeros(offs[-1], hthedl.NODE_DTYPE)
    kids = np.zeros(coffs[-1], np.uint32)
    shift = np.arange(int(p_len.sum())) - np.repeat(np.cumsum(p_len) - p_len, p_len)
    to = np.repeat(offs[:-1], p_len) + shift
    nodes[to] = p[0][np.repeat(p[1].astype(np.int64)[pi], p_len) + shift]
    joint = nodes["arity"][to] > 0
    nodes["child"][to[joint]] += np.repeat(coffs[:-1] - p[3][:-1][pi], p_len)[joint].astype(np.uint32)
    shift = np.arange(int(p_kid.sum())) - np.repeat(np.cumsum(p_kid) - p_kid, p_kid)
    kids[np.repeat(coffs[:-1], p_kid) + shift] = p[2][np.repeat(p[3][:-1][pi], p_kid) + shift]
    atom, o = rng.integers(0, 1024, rows), hthedl.OPS
    nodes["arg"][(offs[:-1] + spot)[swap]] = atom[swap]
    leaf = (offs[:-1] + p_len)[~swap]
    nodes["op"][leaf], nodes["arg"][leaf] = o["atom"], atom[~swap]
    at = (offs[:-1] + p_len + 1)[deep]
    nodes["op"][at], nodes["arg"][at], nodes["child"][at] = o["exists"], rng.integers(0, 48, at.shape[0]), p_len[deep]
    nodes["inv"][at] = rng.integers(0, 2, at.shape[0])
    top, c = (offs[1:] - 1)[~swap], (coffs[1:] - 2)[~swap]
    nodes["op"][top], nodes["arity"][top], nodes["child"][top] = o["and"], 2, c
    kids[c], kids[c + 1] = (p_len - 1)[~swap], (p_len + more - 2)[~swap]
    return p[:3], (nodes, offs.astype(np.uint32), kids), pi.astype(np.int32)


def _screener_inputs(case, seed):
    """What training and scoring share, as plain arrays: hypotheses, weights, targets or base coverage."""
    rng = np.random.default_rng([seed, 11])
    i = types.SimpleNamespace()
    i.parents, i.cands, i.pi = _refinements(rng, case["rows"], case["parents"], case["nodes"])
    i.params = init_params(int(rng.integers(1 << 30)))
    for name in ("b1", "b2"):
        i.params[name] += rng.standard_normal(i.params[name].shape).astype(np.float32) * 0.05
    i.params["b3"] += np.float32(3.0) + rng.random(2).astype(np.float32)
    i.y = rng.random((case["rows"], 2)).astype(np.float32) * np.float32(1 if case.get("loss") == "bce" else 8)
    i.moments = {k: (rng.standard_normal(v.shape, dtype=np.float32) * np.float32(1e-5),
                     (1 + rng.random(v.shape, dtype=np.float32)) * np.float32(1e-10)) for k, v in i.params.items()} if case["kind"] == "train" else {}
    i.base = rng.integers(1000, 100_000, (case["parents"], 2)).astype(np.int32)[i.pi]
    return i


STEP, N_POS, N_NEG = 200, 100_000, 100_000


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng([seed, 7])
    s = types.SimpleNamespace(case=case)
    kind = case["kind"]
    if kind in ("train", "score"):
        i = _screener_inputs(case, seed)
        s.scr = Screener(i.params, batch=case["rows"] if kind == "train" else case["batch"], device=DEV, lr=5e-4,
                         loss=case.get("loss", "mse"))
        s.fb, s.pfb = FeatureBatch(*i.cands, device=DEV), FeatureBatch(*i.parents, device=DEV)
        s.pi = torch.from_numpy(i.pi).to(DEV)
        if kind == "train":       # in the middle of training
            s.y, s.scr.step_no = torch.from_numpy(i.y).to(DEV), STEP
            for name, (m, v) in i.moments.items():
                s.scr.m[name].copy_(torch.from_numpy(m))
                s.scr.v[name].copy_(torch.from_numpy(v))
        else:
            s.base = torch.from_numpy(i.base).to(DEV)
            s.scores = torch.empty(case["rows"], device=DEV)
            s.sel = torch.empty(max(1, case["rows"] // 50), dtype=torch.int32, device=DEV)
            s.work = torch.empty(65538, dtype=torch.int32, device=DEV)
        return s
    s.kb = _make_kb(case, gen)
    args = (rng, case.get("hyps", 0), case.get("nodes", 1), case["concepts"], case["roles"], s.kb.deciles)
    if kind == "load":
        s.enc = _hypotheses(*args)[:3]
        load = _Handle(s.kb)      # what the first batch needs is asked for once
        size = hthedl.hth_batch_workspace_bytes(load.handle, *s.enc)
        del load
        s.ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        s.counts = torch.empty((case["hyps"], 2), dtype=torch.int32, device=DEV)
        return s
    s.load = _Handle(s.kb)
    h = s.load.handle
    if kind == "round":
        n_c, parents, cands = case["concepts"], case["parents"], case["parents"] * case["per"]
        i, j = (torch.randint(0, n_c, (parents,), device=DEV, generator=gen) for _ in range(2))
        s.sets = s.kb.concepts[i] & ~s.kb.concepts[j]
        hthedl.hth_kb_set_sets(h, s.sets, parents)
        s.rows = torch.arange(parents, dtype=torch.int32, device=DEV)
        s.dec = torch.from_numpy(s.kb.deciles.astype(np.float32)).to(DEV)
        s.draw_seed = seed + 1
        s.specs = torch.empty(cands * hthedl.CONJ_DTYPE.itemsize, dtype=torch.uint8, device=DEV)
        s.nodes = torch.empty(4 * cands * hthedl.NODE_DTYPE.itemsize, dtype=torch.uint8, device=DEV)
        s.offs = torch.empty(cands + 1, dtype=torch.int32, device=DEV)
        s.kids = torch.empty(2 * cands, dtype=torch.int32, device=DEV)
        s.n_nodes, s.count = 4 * cands, cands
        hthedl.hth_draw_conjuncts(h, s.draw_seed, s.rows, parents, case["per"], s.dec, s.specs)
        hthedl.hth_conjoin(s.specs, cands, s.nodes, s.offs, s.kids)
    else:
        nums = _concrete(case, gen, s) if kind == "concrete" else None
        enc = _hypotheses(*args, nums=nums, strs=case.get("strs", 0))
        s.count = case["hyps"]
        if kind == "plain":
            s.alone = _alone(enc)
            size = max(hthedl.hth_workspace_bytes(h, len(a), 1) for a, _ in s.alone)
            s.inst = torch.empty((s.count, s.kb.stride), dtype=torch.int64, device=DEV) if case["instances"] else None
        elif kind == "device":
            s.n_nodes = enc[0].shape[0]
            s.nodes = torch.from_numpy(enc[0].view(np.uint8)).to(DEV)
            s.offs = torch.from_numpy(enc[1].view(np.int32)).to(DEV)
            s.kids = torch.from_numpy(enc[2].view(np.int32)).to(DEV)
        else:
            s.enc = enc[:3]
            size = hthedl.hth_batch_workspace_bytes(h, *s.enc)
            if kind == "sets":
                s.sets = torch.empty((s.count, s.kb.stride), dtype=torch.int64, device=DEV)
    if kind in ("device", "round"):
        s.scratch_bytes = hthedl.hth_dplan_scratch_bytes(h, s.n_nodes)
        s.scratch = torch.empty(s.scratch_bytes, dtype=torch.uint8, device=DEV)
        plan, size = _plan(s)
        hthedl.hth_dplan_destroy(plan)
    s.ws = torch.empty(max(256, size), dtype=torch.uint8, device=DEV)
    s.counts = torch.empty((s.count, 2), dtype=torch.int32, device=DEV)
    return s


def _plan(s):
    return hthedl.hth_dplan_create(s.load.handle, s.nodes, s.n_nodes, s.offs, s.count, s.kids, s.kids.shape[0],
                                   s.scratch, s.scratch_bytes)


def run(s):
    kind, case = s.case["kind"], s.case
    if kind == "train":
        s.fb.densify(0, case["rows"], s.scr.x, s.pfb, s.pi)
        s.scr.train_step(case["rows"], s.y)
        return {"z": s.scr.z, "g": s.scr.g, "p": s.scr.p, "m": s.scr.m, "v": s.scr.v}
    if kind == "score":
        s.fb.recompute()
        s.pfb.recompute()
        screened.score(s.scr, s.fb, case["rows"], N_POS, N_NEG, s.scores, base=s.base, parents=s.pfb,
                       parent_index=s.pi, kind=1)
        hthedl.hth_topk(s.scores, case["rows"], s.sel.shape[0], s.sel, s.work)
        return {"scores": s.scores, "top": torch.sort(s.scores[s.sel.long()], descending=True)[0]}
    if kind == "load":
        load = _Handle(s.kb)
        hthedl.hth_eval_batch(load.handle, *s.enc, s.ws, s.ws.numel(), s.counts)
        return {"counts": s.counts, "degrees": [hthedl.hth_kb_max_degree(load.handle, r, d)
                                                for r in range(min(4, case["roles"])) for d in (0, 1)]}
    h = s.load.handle
    if kind == "plain":
        for i, (nodes, kids) in enumerate(s.alone):
            hthedl.hth_eval_one(h, nodes, kids, s.ws, s.ws.numel(), None if s.inst is None else s.inst[i], s.counts[i])
        return (s.counts,) if s.inst is None else (s.counts, s.inst)
    if kind in ("device", "round"):
        if kind == "round":
            hthedl.hth_draw_conjuncts(h, s.draw_seed, s.rows, case["parents"], case["per"], s.dec, s.specs)
            hthedl.hth_conjoin(s.specs, s.count, s.nodes, s.offs, s.kids)
        plan, size = _plan(s)
        hthedl.hth_dplan_launch(plan, s.ws, s.ws.numel(), s.counts)
        hthedl.hth_dplan_destroy(plan)
        return (s.counts, s.specs) if kind == "round" else s.counts
    if kind == "sets":
        hthedl.hth_eval_batch_sets(h, *s.enc, s.ws, s.ws.numel(), s.sets, s.counts)
        return s.counts, s.sets
    hthedl.hth_eval_batch(h, *s.enc, s.ws, s.ws.numel(), s.counts)
    return s.counts


def work(case):
    """The knowledge base read once (a role's offsets and targets in 32 bits, concept rows, columns, examples), the
    hypotheses and the results written; for the screener the products with the few features that a row holds."""
    kind = case["kind"]
    if kind in ("train", "score"):
        n = case["rows"]
        per = 2.0 * case["nodes"] + 4
        if kind == "train":       # x is a dense input of the layer; forward, both gradients, the optimiser's state
            pairs = D_IN * D_H1 + D_H1 * D_H2
            return {"bytes": 2.0 * n * D_IN + 30.0 * pairs, "flops": 2.0 * n * (2 * D_IN * D_H1 + 3 * D_H1 * D_H2)}
        return {"bytes": 16.0 * n * case["nodes"] + 16.0 * n + 2.0 * (D_IN * D_H1 + D_H1 * D_H2),
                "flops": 2.0 * n * (per * D_H1 + D_H1 * D_H2 + 2 * D_H2)}
    n, row = case["n"], 8.0 * ((case["n"] + 63) // 64)
    edges = case["edges"] or case["roles"] * n * _mean_degree(case["zipf"], case["cap"])
    hyps = case.get("hyps") or case["parents"] * case["per"]
    roles, concepts, props = case["roles"], case["concepts"], case["props"]
    if kind in ("plain", "sets"):     # the roles, concepts and columns that so few hypotheses name
        uses = hyps * case["nodes"]
        if kind == "plain":           # one after the other: each names its own
            edges, roles, concepts, props = edges / roles * 0.25 * uses, 0.25 * uses, 0.3 * uses, 0.08 * uses
        else:
            concepts, props = min(concepts, 0.3 * uses), min(props, 0.08 * uses)
    if kind == "load":
        got = roles * 8.0 * n + 4.0 * edges + concepts * row + roles * 8.0 * n + 4.0 * edges
        return {"bytes": got, "flops": 0.0}
    got = roles * 4.0 * n + 4.0 * edges + concepts * row + props * 4.0 * n + 2 * row + 8.0 * hyps
    if kind == "concrete":
        got += (case["nums"] + case["strs"]) * (4.0 * n + 4.0 * 0.5 * n * _mean_degree(1.6, 16))
    if kind == "round":
        got += case["parents"] * row
    if kind == "sets" or (kind == "plain" and case["instances"]):
        got += hyps * row
    return {"bytes": got, "flops": 0.0}


def _mean_degree(s, cap):
    d = np.arange(1, cap + 1, dtype=np.float64)
    return float((d ** (1 - s)).sum() / (d ** -s).sum())


# ---------------------------------------------------------------------------
# the screener in 64 bits
# ---------------------------------------------------------------------------


def _fnv(h, v, n):
    for i in range(n):
        h = (h ^ ((v >> np.uint64(8 * i)) & np.uint64(255))) * np.uint64(0x100000001B3)
    return h


def _features(nodes, offs, kids):
    """Feature index of every node: the subtree's FNV-1a hash (children of a conjunction or disjunction by the sum
    of their mixed hashes) mod 4096.  All hypotheses' j-th nodes at once."""
    u64, o = np.uint64, hthedl.OPS
    offs = offs.astype(np.int64)
    n_len = np.diff(offs)
    out = np.zeros(nodes.shape[0], u64)
    for j in range(int(n_len.max())):
        b = offs[:-1][n_len > j]
        n = nodes[b + j]
        op = n["op"].astype(u64)
        role = (op >= o["exists"]) & (op <= o["exactly"])
        value = (op == o["dge"]) | (op == o["dle"]) | ((op >= o["deq"]) & (op <= o["neq"]))
        many = (op == o["and"]) | (op == o["or"])
        h = _fnv(np.full(n.shape[0], 0xCBF29CE484222325, u64), op, 1)
        h = _fnv(h, np.where(role, n["inv"], 0).astype(u64), 1)
        h = _fnv(h, np.where(many, n["arity"], 0).astype(u64), 2)
        h = _fnv(h, np.where((op == o["atom"]) | role | value, n["arg"], 0).astype(u64), 4)
        h = _fnv(h, np.where((op >= o["atleast"]) & (op <= o["exactly"]) | value, n["q"], 0).astype(u64), 4)
        child = (op == o["not"]) | role
        got = out[b[child] + n["child"][child]]
        total = np.zeros(n.shape[0], u64)
        for c in range(int(n["arity"][many].max()) if many.any() else 0):
            g = many & (n["arity"] > c)
            z = out[b[g] + kids[n["child"][g].astype(np.int64) + c]] + u64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> u64(30))) * u64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> u64(27))) * u64(0x94D049BB133111EB)
            total[g] += z ^ (z >> u64(31))
        total[child] = got
        out[b + j] = np.where(child | many, _fnv(h, total, 8), h)
    return (out & u64(4095)).astype(np.int64)


def _dense(feats, offs, lo, hi, pfeats, poffs, pi):
    """Rows lo..hi: the features of each refinement minus its parent's, float64."""
    def put(f, o, rows, sign):
        n = np.diff(o)[rows]
        at = np.repeat(o[:-1][rows], n) + np.arange(int(n.sum())) - np.repeat(np.cumsum(n) - n, n)
        r = np.repeat(np.arange(rows.shape[0]), n)
        x.view(-1).index_add_(0, torch.from_numpy(r * D_IN + f[at]).to(DEV), torch.full((r.shape[0],), sign, dtype=torch.float64, device=DEV))
    x = torch.zeros((hi - lo, D_IN), dtype=torch.float64, device=DEV)
    put(feats, offs, np.arange(lo, hi), 1.0)
    put(pfeats, poffs, pi[lo:hi].astype(np.int64), -1.0)
    return x


def exact(case, seed):
    if case["kind"] not in ("train", "score"):
        return None
    i = _screener_inputs(case, seed)
    f, pf = _features(*i.cands), _features(*i.parents)
    offs, poffs = i.cands[1].astype(np.int64), i.parents[1].astype(np.int64)
    p = {k: torch.from_numpy(v).to(DEV).double() for k, v in i.params.items()}
    w1, w2 = (torch.from_numpy(i.params[k]).to(DEV).bfloat16().double() for k in ("w1", "w2"))

    def layers(x):
        h1 = torch.relu(x @ w1 + p["b1"])
        h2 = torch.relu(h1 @ w2 + p["b2"])
        return h1, h2, h2 @ p["w3"] + p["b3"]

    n = case["rows"]
    if case["kind"] == "score":
        scores = []
        for lo in range(0, n, 8192):
            hi = min(n, lo + 8192)
            z = layers(_dense(f, offs, lo, hi, pf, poffs, i.pi))[2]
            base = torch.from_numpy(i.base[lo:hi]).to(DEV).double()
            kept = torch.minimum((base - torch.expm1(z.clamp(min=0))).clamp(min=0), base)
            scores.append(2 * kept[:, 0] / (kept.sum(1) + N_POS))
        scores = torch.cat(scores)
        return {"scores": scores, "top": torch.topk(scores, max(1, n // 50))[0]}
    x, y = _dense(f, offs, 0, n, pf, poffs, i.pi), torch.from_numpy(i.y).to(DEV).double()
    h1, h2, z = layers(x)
    dz = ((torch.sigmoid(z) if case["loss"] == "bce" else z) - y) / (2 * n)
    dh2 = (dz @ p["w3"].T) * (h2 > 0)
    dh1 = (dh2 @ w2.T) * (h1 > 0)
    g = {"w1": x.T @ dh1, "b1": dh1.sum(0), "w2": h1.T @ dh2, "b2": dh2.sum(0), "w3": h2.T @ dz, "b3": dz.sum(0)}
    out = {"z": z, "g": g, "p": {}, "m": {}, "v": {}}
    t = STEP + 1
    for k, (m0, v0) in i.moments.items():
        m = 0.9 * torch.from_numpy(m0).to(DEV).double() + 0.1 * g[k]
        v = 0.999 * torch.from_numpy(v0).to(DEV).double() + 0.001 * g[k] ** 2
        decay = 1 - 5e-4 * (1e-4 if k[0] == "w" else 0.0)
        out["p"][k] = p[k] * decay - 5e-4 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        out["m"][k], out["v"][k] = m, v
    return out
