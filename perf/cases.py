"""Workloads of the join library whose speed is followed: what a program that
uses it has it do, through the public entry points of paper_2607_04489_amd.

Every pass starts from columns that lie in device memory and ends with results
whose order does not depend on the run: result pairs are put in probe-row order
with the library's own radix sort (what a late materialization that reads the
probe columns front to back does), groups in key order.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2607_04489_amd as eg
from paper_2607_04489_amd import selector as eg_selector

I32, I64 = torch.int32, torch.int64
DTYPES = {"int32": I32, "int64": I64}


# ---- cases -------------------------------------------------------------------------

def listed():
    return [
        # A small lookup: a thousand-row dimension against a micro-batch of facts. Latency and
        # the number of launches and copies decide.
        dict(name="join_small32", kind="join", key="int32", pay="int32", layout="dense", n_build=1000,
             n_probe=20011, match=0.8, result="pairs", selector="rule"),
        # The dense primary-key join of the benchmark (65,536 x 1,048,576 rows, int32).
        dict(name="join_dense32", kind="join", key="int32", pay="int32", layout="dense", n_build=65536,
             n_probe=1 << 20, match=0.8, result="pairs", selector="rule"),
        # An ordinary foreign-key join on 64-bit surrogate keys, odd sizes, row-id pairs out,
        # planned by the learned selector.
        dict(name="join_fk64", kind="join", key="int64", pay="int64", layout="sparse", n_build=1000003,
             n_probe=33554393, match=0.9, result="pairs", selector="learned"),
        # The benchmark's large sparse join (16.8M x 537M rows, int64) as the aggregate query
        # COUNT(*), SUM(r.p * s.p): the count-only mode of the join.
        dict(name="join_sum64", kind="join", key="int64", pay="int64", layout="sparse", n_build=1 << 24,
             n_probe=1 << 29, match=0.9, result="sum", selector="learned"),
        # A star query: a dimension with one attribute joined to facts with two measures, the
        # payload columns materialized, then summed per attribute value.
        dict(name="star_dim32", kind="star", key="int32", n_build=65536, n_probe=1 << 27, dup=1, zipf=0.0, match=0.9,
             groups=1000),
        # The same query over a many-to-many relation: each key repeated (mean 4), skewed probe
        # keys; the partitioned join with its payload columns.
        dict(name="star_skew32", kind="star", key="int32", n_build=1 << 24, n_probe=1 << 26, dup=4, zipf=0.5,
             match=1.0, groups=200000),
        # Group-by of 2^28 rows with two sums: a handful of groups (a status or region column).
        dict(name="groupby_few32", kind="groupby", key="int32", val="int32", n=1 << 28, groups=100, vals=2),
        # The same rows in a million groups (a customer column).
        dict(name="groupby_many32", kind="groupby", key="int32", val="int32", n=1 << 28, groups=1 << 20, vals=2),
        # A mid-size group-by on 64-bit keys with one 64-bit sum, odd row count.
        dict(name="groupby_mid64", kind="groupby", key="int64", val="int64", n=20000003, groups=50000, vals=1),
        # ORDER BY four int32 columns over 2^28 rows (the benchmark's multi-key sort): narrow
        # ranges and few-valued columns fused into one radix-sorted key.
        dict(name="sort_4keys32", kind="sort", key="int32", n=1 << 28, keys=4, ndv=256, descending=False),
        # A batch of independent joins of uneven sizes replayed as one captured graph.
        dict(name="batch_joins32", kind="batch", joins=256, log2_lo=8, log2_hi=18),
        # One full-batch training step of the variant selector on its 4,050 training instances.
        dict(name="selector_step", kind="train", batch=4050),
    ]


def _size(rng, lo, hi):
    """A size between lo and hi, even over its logarithm; as often odd as not."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["join", "join", "join", "star", "groupby", "groupby", "sort", "batch", "train"])
    if kind == "join":
        result = rng.choice(["pairs", "pairs", "sum"])
        key = rng.choice(["int32", "int64"])
        n_probe = _size(rng, 10000, (1 << 25) if result == "pairs" else (1 << 28))
        return dict(kind=kind, key=key, pay=rng.choice(["int32", "int64"]), layout=rng.choice(["dense", "sparse"]),
                    n_build=_size(rng, 500, min(1 << 24, n_probe)), n_probe=n_probe,
                    match=round(rng.uniform(0.1, 1.0), 3), result=result, selector=rng.choice(["rule", "learned"]))
    if kind == "star":
        dup = rng.choice([1, 1, 4])
        n_probe = _size(rng, 1 << 18, 1 << 26)
        n_build = _size(rng, 1000, min(1 << 24, n_probe))
        return dict(kind=kind, key=rng.choice(["int32", "int64"]), n_build=n_build,
                    n_probe=n_probe, dup=dup, zipf=rng.choice([0.0, 0.5]) if dup > 1 else 0.0,
                    match=round(rng.uniform(0.3, 1.0), 3), groups=_size(rng, 2, min(1 << 18, n_build // 64)))
    if kind == "groupby":
        n = _size(rng, 10000, 1 << 28)
        key = rng.choice(["int32", "int64"])
        return dict(kind=kind, key=key, val=rng.choice(["int32", "int64"]),
                    n=n if key == "int32" else min(n, (1 << 27) + 1), groups=_size(rng, 2, min(1 << 22, n // 64)),
                    vals=rng.choice([0, 1, 2]))
    if kind == "sort":
        key = rng.choice(["int32", "int64"])
        return dict(kind=kind, key=key, n=_size(rng, 5000, 1 << (28 if key == "int32" else 27)),
                    keys=rng.choice([2, 3, 4]), ndv=_size(rng, 16, 5000), descending=rng.choice([False, True]))
    if kind == "batch":
        lo = rng.choice([8, 10, 12])
        return dict(kind=kind, joins=_size(rng, 16, 300), log2_lo=lo, log2_hi=lo + rng.choice([4, 6]))
    return dict(kind=kind, batch=_size(rng, 500, 8000))


# ---- inputs ------------------------------------------------------------------------

_DEV = "cuda"


def _gen(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(seed)
    return g


def _ints(g, n, lo, hi, dtype):
    return torch.randint(lo, hi, (n,), generator=g, device=_DEV, dtype=dtype)


def _words(g, n, dtype):
    """Values over the type's whole range, but for its two ends."""
    info = torch.iinfo(dtype)
    return _ints(g, n, info.min + 1, info.max, dtype)


def _mix(x):
    """A bijection of 64-bit words (odd multiplies and xor-shifts): distinct in, distinct out."""
    for m, k in ((0x2545F4914F6CDD1D, 29), (0x369DEA0F31A53F85, 32)):
        x = x * m
        x = x ^ ((x >> k) & ((1 << (64 - k)) - 1))
    return x


def _mix31(x):
    """A bijection of [0, 2^31)."""
    m = (1 << 31) - 1
    for mul, k in ((0x2C1B3C6D, 15), (0x297A2D39, 13)):
        x = (x * mul) & m
        x = x ^ (x >> k)
    return x


def _distinct(g, n, extra, key, layout):
    """n distinct build keys in random order, and a function idx -> keys that no build row has."""
    i = torch.arange(n, device=_DEV, dtype=I64)
    off = int(_ints(g, 1, 0, 1 << 30, I64))
    if layout == "dense":  # a shuffled range, missing keys above it
        keys = i[torch.randperm(n, generator=g, device=_DEV)] + (off & 0xFFFF)
        miss = lambda j: (off & 0xFFFF) + n + j % max(1, n // 4)  # noqa: E731
        return keys, miss
    f = _mix31 if key == I32 else _mix
    if key == I32:
        assert n + extra < 1 << 31
    wrap = (lambda v: v & ((1 << 31) - 1)) if key == I32 else (lambda v: v)
    return f(wrap(i + off)), lambda j: f(wrap(j + (off + n)))


def _probe(g, n_probe, keys, match, miss, zipf, dtype, fixed=False):
    """Probe keys: with probability match a build key (uniform, or Zipf over them), else a missing one;
    fixed: exactly that share of the rows, in random places."""
    nd = keys.numel()
    if zipf > 0:
        w = torch.arange(1, nd + 1, device=_DEV, dtype=torch.float64).pow_(-zipf)
        cdf = torch.cumsum(w, 0)
        u = torch.rand(n_probe, generator=g, device=_DEV, dtype=torch.float64) * cdf[-1]
        src = torch.searchsorted(cdf, u).clamp_(max=nd - 1)
        del u, cdf, w
    else:
        src = _ints(g, n_probe, 0, nd, I64)
    pk = keys[src].to(dtype)
    del src
    if match < 1.0:
        if fixed:
            hit = torch.randperm(n_probe, generator=g, device=_DEV) < round(match * n_probe)
        else:
            hit = torch.rand(n_probe, generator=g, device=_DEV) < match
        pk = torch.where(hit, pk, miss(torch.arange(n_probe, device=_DEV, dtype=I64)).to(dtype))
    return pk


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "join":
        key, pay = DTYPES[case["key"]], DTYPES[case["pay"]]
        keys, miss = _distinct(g, case["n_build"], case["n_probe"], key, case["layout"])
        pk = _probe(g, case["n_probe"], keys, case["match"], miss, 0.0, key, fixed=case["result"] == "pairs")
        s = {"bk": keys.to(key), "pk": pk,
             "bp": _ints(g, case["n_build"], 0, 1000, pay), "pp": _ints(g, case["n_probe"], 0, 1000, pay)}
        s["selector"] = eg.SEL_LEARNED if case["selector"] == "learned" else eg.SEL_RULE
        if case["selector"] == "learned":
            eg_selector.load_model()
        s["sum"] = case["result"] == "sum"
        s["row_bits"] = max(1, (case["n_probe"] - 1).bit_length())
    elif kind == "star":
        key = DTYPES[case["key"]]
        nd = max(1, case["n_build"] // case["dup"])
        keys, miss = _distinct(g, nd, case["n_probe"], key, "sparse")
        bk = keys
        if case["dup"] > 1:  # geometric repeats of the mean asked for, rows shuffled
            p = 1.0 / case["dup"]
            u = torch.rand(nd, generator=g, device=_DEV, dtype=torch.float64).clamp_(min=1e-12)
            reps = (1 + torch.floor(torch.log(u) / math.log(1.0 - p))).to(I64).clamp_(max=64)
            bk = torch.repeat_interleave(keys, reps)
            bk = bk[torch.randperm(bk.numel(), generator=g, device=_DEV)]
        s = {"bk": bk.to(key), "pk": _probe(g, case["n_probe"], keys, case["match"], miss, case["zipf"], key),
             "attr": _ints(g, bk.numel(), 0, case["groups"], I32) * 3 + 11,
             "m1": _ints(g, case["n_probe"], 0, 1000, I32), "m2": _words(g, case["n_probe"], I32)}
    elif kind == "groupby":
        key, val = DTYPES[case["key"]], DTYPES[case["val"]]
        gid = _ints(g, case["n"], 0, case["groups"], I32)
        values = _mix31(torch.arange(case["groups"], device=_DEV, dtype=I64) + int(_ints(g, 1, 0, 1 << 20, I64)))
        if key == I64:
            values = values * 0x100000003  # spread beyond 32 bits, still distinct and positive
        s = {"keys": values.to(key)[gid], "vals": [_words(g, case["n"], val) for _ in range(case["vals"])]}
    elif kind == "sort":
        key = DTYPES[case["key"]]
        cols = []
        for c in range(case["keys"]):
            if c % 2 == 0:  # a narrow range
                base = int(_ints(g, 1, -(1 << 29), 1 << 29, I64))
                cols.append(base + _ints(g, case["n"], 0, 256, key))
            else:  # few values over the whole type
                cols.append(_words(g, case["ndv"], key)[_ints(g, case["n"], 0, case["ndv"], I32)])
        s = {"cols": cols, "descending": [case["descending"] and c % 2 == 0 for c in range(case["keys"])]}
    elif kind == "batch":
        r = random.Random(seed)
        joins = []
        for j in range(case["joins"]):
            nb = int(round(2.0 ** r.uniform(case["log2_lo"], case["log2_hi"])))
            npr = int(round(nb * r.uniform(4, 16)))
            keys, miss = _distinct(g, nb, npr, I32, "dense" if j % 2 == 0 else "sparse")
            joins.append((keys.to(I32), _ints(g, nb, 0, 1000, I32), _probe(g, npr, keys, r.uniform(0.1, 1.0), miss, 0.0, I32),
                          _ints(g, npr, 0, 1000, I32)))
        s = {"batch": eg.Batch(joins)}
    else:
        n = case["batch"]
        params = torch.zeros(eg.mlp_param_count(), device=_DEV)
        for (a, b), fan in zip(_WEIGHTS, (16, 64, 64)):
            params[a:b] = torch.randn(b - a, generator=g, device=_DEV) * math.sqrt(2.0 / fan)
        x = torch.randn(n, 16, generator=g, device=_DEV)
        target = torch.randn(n, 16, generator=g, device=_DEV) * 2.0 + x[:, :1]
        mask = (torch.rand(n, 16, generator=g, device=_DEV) < 0.8).float()
        s = {"trainer": eg.MlpTrainer(params, n), "x": x, "target": target, "mask": mask}
    s["kind"] = kind
    return s


# offsets of W1, W2, W3 (each followed by its bias) in the selector's parameter array
_WEIGHTS = ((0, 1024), (1088, 5184), (5248, 6272))
_BIASES = ((1024, 1088), (5184, 5248), (6272, 6288))


# ---- one pass ----------------------------------------------------------------------

def _in_key_order(g):
    """A group-by's result by ascending key."""
    keys, perm = eg.sort_pairs(g.keys, 8 * g.keys.element_size())
    perm = perm.long()
    return {"keys": keys, "counts": g.counts[perm], "sums": [t[perm] for t in g.sums]}


def run(s):
    kind = s["kind"]
    if kind == "join":
        plan = eg.join_plan(eg.stats(s["bk"]), eg.stats(s["pk"]), s["selector"])
        if s["sum"]:
            res = eg.join(s["bk"], s["bp"], s["pk"], s["pp"], plan, count_only=True)
            return {"count": res.count, "sum": res.checksum}
        res = eg.join(s["bk"], s["bp"], s["pk"], s["pp"], plan)
        probe, build = eg.sort_pairs(res.probe_rowid, s["row_bits"], vals=res.build_rowid)
        return {"count": res.count, "sum": res.checksum, "probe": probe, "build": build}
    if kind == "star":
        plan = eg.join_plan(eg.stats(s["bk"]), eg.stats(s["pk"]))
        res = eg.join_wide(s["bk"], [s["attr"]], s["pk"], [s["m1"], s["m2"]], plan)
        out = _in_key_order(eg.groupby(res.build_cols[0], res.probe_cols))
        out["rows"] = res.count
        return out
    if kind == "groupby":
        return _in_key_order(eg.groupby(s["keys"], s["vals"]))
    if kind == "sort":
        perm, keys, plan = eg.sort_multikey(s["cols"], s["descending"], with_sorted=True)
        return {"perm": perm, "keys": keys, "bits": int(plan.total_bits)}
    if kind == "batch":
        s["batch"].launch()
        counts, checksums, variants, flags = s["batch"].results()
        return {"counts": counts, "checksums": checksums, "variants": variants, "flags": flags}
    t = s["trainer"]
    t.step(s["x"], s["target"], s["mask"], 3e-3)
    return {"params": t.params, "m": t.m, "v": t.v, "grads": t.grads, "loss": t.loss}


# ---- what a pass cannot do without -------------------------------------------------

def _width(name):
    return 8 if name == "int64" else 4


def work(case):
    kind = case["kind"]
    if kind == "join":
        b = (case["n_build"] + case["n_probe"]) * (_width(case["key"]) + _width(case["pay"]))
        if case["result"] == "pairs":
            b += 8 * case["match"] * case["n_probe"]
    elif kind == "star":
        b = (case["n_build"] + case["n_probe"]) * _width(case["key"]) + 4 * case["n_build"] + 8 * case["n_probe"]
        b += 28 * min(case["groups"], case["n_build"])
    elif kind == "groupby":
        b = case["n"] * (_width(case["key"]) + case["vals"] * _width(case["val"]))
        b += min(case["groups"], case["n"]) * (_width(case["key"]) + 8 + 8 * case["vals"])
    elif kind == "sort":
        b = case["n"] * (case["keys"] * _width(case["key"]) + 4 + 4)
    elif kind == "batch":
        # mean of 2^U(lo, hi), ten probe rows to a build row, 55% of them matching
        mean = (2.0 ** case["log2_hi"] - 2.0 ** case["log2_lo"]) / (math.log(2.0) * (case["log2_hi"] - case["log2_lo"]))
        b = case["joins"] * mean * (11 * 8 + 10 * 0.55 * 8)
    else:
        macs = 16 * 64 + 64 * 64 + 64 * 16
        return {"bytes": 4.0 * (case["batch"] * 48 + 7 * 6288), "flops": 2.0 * case["batch"] * (3 * macs - 16 * 64)}
    return {"bytes": float(b), "flops": 0.0}


# ---- the same in 64 bits -----------------------------------------------------------

def exact(case, seed):
    """The training step's outputs in float64; the other kinds return whole numbers only."""
    if case["kind"] != "train":
        return None
    s = prepare(case, seed)
    x, target, mask = (s[k].double() for k in ("x", "target", "mask"))
    params = s["trainer"].params.double().requires_grad_(True)
    h = x
    for k, (wa, ba) in enumerate(zip(_WEIGHTS, _BIASES)):
        out = ba[1] - ba[0]
        h = h @ params[wa[0]:wa[1]].view(-1, out) + params[ba[0]:ba[1]]
        if k < 2:
            h = torch.relu(h)
    loss = (mask * (h - target) ** 2).sum() / mask.sum()
    (grad,) = torch.autograd.grad(loss, params)
    # as the step is called with 32-bit constants
    b1, b2, eps, lr = (float(torch.tensor(c, dtype=torch.float32)) for c in (0.9, 0.999, 1e-8, 3e-3))
    m, v = (1 - b1) * grad, (1 - b2) * grad ** 2
    new = params.detach() - lr * (m / (1 - b1)) / (torch.sqrt(v / (1 - b2)) + eps)
    return {"params": new, "m": m, "v": v, "grads": grad, "loss": loss.detach().reshape(1)}
