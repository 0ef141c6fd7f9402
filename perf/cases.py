"""The work that users of this framework have it do, as cases that can be timed.

A case is one pass through the public entry points of `paper_1901_01488_amd`
on inputs that a user's program has on the GPU beforehand: exact counts of
selections, counts followed by materializations, split selectivities,
micro-batches of arriving queries, training labels, star joins over filtered
build sides, and the estimator's inference and training.  Tables and
predicates are those of `datagen` (the star table, the Section 1 table, the
planning and learned-gate tables), at sizes from a few thousand rows to the
full 60M-row star table, odd and ragged ones among them.

`listed()` names the cases, `draw(rng)` gives others of the same ranges,
`prepare` makes what a program holds before the call, `run` is the call,
`work` the bytes and operations that no implementation can do without, and
`exact` the result from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_1901_01488_amd import datagen as dg
from paper_1901_01488_amd import esc, learned, planning

DEV = "cuda:0"
HUBER = 0.5


def listed():
    return [
        # one optimizer sub-query, the Section 1 selection with its udf on the 1M-row table:
        # launch and read-back latency
        {"name": "count_1m", "kind": "count", "table": "plain", "rows": 1_000_000, "preds": 1},
        # exact counts on the full fact table, two to five columns per selection: streaming rate
        {"name": "count_60m", "kind": "count", "table": "star", "rows": 60_000_000, "preds": 8},
        # count, decide, materialize on a mid-size fact table whose rows fill no whole tile
        {"name": "select_6m", "kind": "select", "rows": 6_000_007, "preds": 8},
        # the same on the full fact table: the framework's main path
        {"name": "select_60m", "kind": "select", "rows": 60_000_000, "preds": 8},
        # two weakly selective selections kept whole in turn, without counts before them
        {"name": "materialize_20m", "kind": "materialize", "rows": 20_000_003, "sel": 0.35, "proj": 3},
        # split selectivities of conjunctions for predicate ordering
        {"name": "conjuncts_10m", "kind": "conjuncts", "rows": 10_000_019, "preds": 4},
        # two full windows of three-table queries, every selection counted exactly
        {"name": "planning_100m", "kind": "planning", "rows": 100_000_000, "queries": 128, "probe": True},
        # exact training labels of the estimator
        {"name": "labels_10m", "kind": "labels", "rows": 10_000_000, "preds": 2048},
        # star join of a probe relation with two filtered dimensions (permutation keys): build and probe
        {"name": "join_star", "kind": "join", "rows": 200_000_000, "r": 2_000_000, "s": 20_000_000,
         "sel_r": 0.05, "sel_s": 0.15, "keys": "perm"},
        # the same with keys spread over all 32-bit integers
        {"name": "join_wide", "kind": "join", "rows": 20_000_003, "r": 50_021, "s": 2_000_003,
         "sel_r": 1.0, "sel_s": 1.0, "keys": "wide"},
        # the gate's estimates of one batch of predicates
        {"name": "predict_4096", "kind": "predict", "rows": 4096},
        # minibatch training steps of the estimator
        {"name": "train_256", "kind": "train", "batch": 256, "steps": 48, "samples": 20_000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count", "count", "select", "select", "materialize", "conjuncts", "planning", "labels",
                       "join", "join", "predict", "train", "gradients"])
    if kind == "count":
        return {"kind": kind, "table": rng.choice(["plain", "star", "star"]), "rows": _log(rng, 1_000, 60_000_000),
                "preds": rng.randint(1, 8)}
    if kind == "select":
        return {"kind": kind, "rows": _log(rng, 20_000, 60_000_000), "preds": rng.randint(1, 8)}
    if kind == "materialize":
        return {"kind": kind, "rows": _log(rng, 5_000, 40_000_000), "sel": round(10.0 ** rng.uniform(-4, -0.1), 6),
                "proj": rng.randint(1, 4)}
    if kind == "conjuncts":
        return {"kind": kind, "rows": _log(rng, 10_000, 40_000_000), "preds": rng.randint(1, 4)}
    if kind == "planning":
        return {"kind": kind, "rows": _log(rng, 1_000_000, 100_000_000), "queries": _log(rng, 4, 128),
                "probe": rng.random() < 0.5}
    if kind == "labels":
        return {"kind": kind, "rows": _log(rng, 50_000, 10_000_000), "preds": _log(rng, 32, 2048)}
    if kind == "join":
        r, s = _log(rng, 1_000, 2_000_000), _log(rng, 10_000, 20_000_000)
        return {"kind": kind, "rows": _log(rng, 50_000, 100_000_000), "r": r, "s": s,
                "sel_r": round(10.0 ** rng.uniform(-2, 0), 4), "sel_s": round(10.0 ** rng.uniform(-2, 0), 4),
                "keys": rng.choice(["perm", "perm", "wide", "dups"])}
    if kind == "predict":
        return {"kind": kind, "rows": _log(rng, 1, 262_144)}
    if kind == "train":
        return {"kind": kind, "batch": _log(rng, 16, 1024), "steps": rng.randint(8, 48), "samples": 20_000}
    return {"kind": kind, "rows": _log(rng, 1, 4096)}


# ---------------------------------------------------------------- selections on the star table

# Each selection is a list of leaves whose selectivity is known beforehand;
# constants come from the seed.  Columns: 0, 1 dates over 2,557 days,
# 2 quantity 1..50, 3 discount 0..10, 4 price (lognormal), 5 ten quantity
# steps each, 6 and 7 Zipf(1.2) foreign keys.
STAR_SELECTIONS = [
    [("date", 0, 60), ("qty", 2, 20)],
    [("disc", 3, 3), ("below", 4, 0.6)],
    [("after", 1, 500), ("fk", 7, 6), ("band", 4, 0.5)],
    [("fk", 6, 14), ("step", 5, 60)],
    [("date", 0, 365), ("disc", 3, 4), ("qty", 2, 25)],
    [("after", 0, 1200), ("after", 1, 1200), ("below", 4, 0.5), ("qty", 2, 30)],
    [("amount", 2, 5), ("fk", 7, 1), ("date", 0, 200), ("band", 4, 0.7)],
    [("date", 0, 900), ("after", 1, 800), ("qty", 2, 25), ("disc", 3, 5), ("below", 4, 0.8)],
]
STAR_PROJECTION = [6, 7, 4]
ZIPF_IDS = {6: 2_000_000, 7: 200_000}


def _normal_quantile(p):
    return math.sqrt(2.0) * float(torch.erfinv(torch.tensor(2.0 * p - 1.0, dtype=torch.float64)))


def _price(p):
    return np.float32(math.exp(8.0 + _normal_quantile(min(max(p, 1e-6), 1 - 1e-6))))


def _star_leaf(t, form, rng):
    what, c, x = form
    if what == "date":
        a = dg.DATE_LO + int(rng.integers(0, dg.DATE_SPAN - x + 1))
        return ("between", c, a, a + x - 1)
    if what == "after":
        return ("gt", c, dg.DATE_LO + dg.DATE_SPAN - 1 - x)
    if what == "qty":
        a = int(rng.integers(1, 51 - x + 1))
        return ("between", c, a, a + x - 1)
    if what == "amount":
        return ("in", c, [int(v) for v in rng.choice(np.arange(1, 51), x, replace=False)])
    if what == "disc":
        return ("in", c, [int(v) for v in rng.choice(np.arange(0, 11), x, replace=False)])
    if what == "below":
        return ("lt", c, _price(x))
    if what == "band":
        a = float(rng.uniform(0.0, 1.0 - x))
        return ("between", c, _price(a), _price(a + x))
    if what == "step":
        a = int(rng.integers(10, 510 - x + 1))
        return ("between", c, a, a + x - 1)
    rows = torch.from_numpy(rng.integers(0, t.nrows, x)).to(t.cols[c].device)
    vals = [int(v) for v in t.cols[c][rows].tolist()]
    return ("eq", c, vals[0]) if x == 1 else ("in", c, vals)


_MASS = {}


def _fk_mass(c, m):
    """Expected share of rows of an IN-list of the values of m sampled rows."""
    if (c, m) not in _MASS:
        p = np.arange(1, ZIPF_IDS[c] + 1, dtype=np.float64) ** -1.2
        p /= p.sum()
        _MASS[c, m] = float((p * (1.0 - (1.0 - p) ** m)).sum())
    return _MASS[c, m]


def _star_sel(sel):
    s = 1.0
    for what, c, x in sel:
        s *= {"date": x / dg.DATE_SPAN, "after": x / dg.DATE_SPAN, "qty": x / 50, "amount": x / 50, "disc": x / 11,
              "below": x, "band": x, "step": x / 500}[what] if what != "fk" else _fk_mass(c, x)
    return s


def _star_preds(t, count, seed):
    rng = np.random.default_rng(seed)
    return [("and", [_star_leaf(t, f, rng) for f in STAR_SELECTIONS[i % len(STAR_SELECTIONS)]]) for i in range(count)]


def _device_table(t):
    return esc.Table(t.nrows, t.dtypes, t.cols)


# ---------------------------------------------------------------- preparation


def prepare(case, seed):
    s = globals()["_prepare_" + case["kind"]](case, int(seed))
    s["kind"] = case["kind"]
    return s


def _star_inputs(case, seed):
    t = dg.table_star(case["rows"], seed=seed * 7 + 1, device=DEV)
    return t, _star_preds(t, case["preds"], seed * 7 + 2)


def _count_inputs(case, seed):
    if case["table"] == "star":
        return _star_inputs(case, seed)
    t = dg.table_plain(case["rows"], seed=seed * 7 + 1, device=DEV)
    return t, [dg.pred_plain(t, seed * 7 + 2 + i) for i in range(case["preds"])]


def _prepare_count(case, seed):
    t, specs = _count_inputs(case, seed)
    ctx, dt = esc.Context(0), _device_table(t)
    return {"ctx": ctx, "table": dt, "preds": [esc.Pred(dt, p) for p in specs],
            "ws": ctx.workspace(dt, esc.WS_COUNT), "stream": torch.cuda.current_stream()}


def _prepare_select(case, seed):
    t, specs = _star_inputs(case, seed)
    ctx, dt = esc.Context(0), _device_table(t)
    # temporary tables with room for what an estimate bounds (a foreign-key leaf could keep every row)
    room = [int(1.1 * t.nrows * _star_sel([f for f in STAR_SELECTIONS[i % len(STAR_SELECTIONS)] if f[0] != "fk"])) + 1000
            for i in range(len(specs))]
    # two workspaces in turn: a selection's count runs while the previous one is materialized
    return {"ctx": ctx, "table": dt, "preds": [esc.Pred(dt, p) for p in specs], "proj": STAR_PROJECTION,
            "ids": [torch.zeros(m, dtype=torch.int32, device=DEV) for m in room],
            "outs": [[torch.zeros(m, dtype=t.cols[j].dtype, device=DEV) for j in STAR_PROJECTION] for m in room],
            "ws": [ctx.workspace(dt, esc.WS_MATERIALIZE, key=("select", i)) for i in range(2)],
            "counts": torch.zeros(len(specs), dtype=torch.int64, device=DEV),
            "stream": torch.cuda.current_stream()}


def _materialize_inputs(case, seed):
    n = case["rows"]
    t = dg.table_plain(n, seed=seed * 7 + 1, device=DEV)
    # two ranges of the permutation key: exactly k rows each, evenly spread
    k = max(1, int(case["sel"] * n))
    rng = np.random.default_rng(seed * 7 + 2)
    specs = [("between", 0, int(a), int(a) + k - 1) for a in rng.integers(0, n - k + 1, 2)]
    return t, specs, k, [1, 2, 3, 0][:case["proj"]]


def _prepare_materialize(case, seed):
    t, specs, k, proj = _materialize_inputs(case, seed)
    ctx, dt = esc.Context(0), _device_table(t)
    room = k + k // 10 + 1   # as an estimate would give it: a tenth more than qualifies
    return {"ctx": ctx, "table": dt, "preds": [esc.Pred(dt, p) for p in specs], "proj": proj,
            "ids": [torch.zeros(room, dtype=torch.int32, device=DEV) for _ in specs],
            "outs": [[torch.zeros(room, dtype=torch.int32, device=DEV) for _ in proj] for _ in specs],
            "ws": ctx.workspace(dt, esc.WS_MATERIALIZE), "stream": torch.cuda.current_stream()}


def _prepare_conjuncts(case, seed):
    t, specs = _star_inputs(case, seed)
    ctx, dt = esc.Context(0), _device_table(t)
    return {"ctx": ctx, "table": dt, "preds": [esc.Pred(dt, p) for p in specs], "stream": torch.cuda.current_stream()}


def _planning_inputs(case, seed):
    sizes = [max(1000, case["rows"] // 100), max(1000, case["rows"] // 10), case["rows"]]
    tabs = [dg.table_mixed(n, 4, seed * 7 + i, DEV, kinds=list(dg.PLANNING_KINDS)) for i, n in enumerate(sizes)]
    qs = [dg.preds_anchored(t, case["queries"], seed=seed * 7 + 3 + i, min_conj=2, max_conj=4)
          for i, t in enumerate(tabs)]
    return tabs, list(zip(*qs))


def _prepare_planning(case, seed):
    tabs, queries = _planning_inputs(case, seed)
    ctx = esc.Context(0)
    # every query has arrived: the windows are full, as under load
    w = planning.Workload(ctx, [_device_table(t) for t in tabs], queries, np.zeros(len(queries)))
    return {"ctx": ctx, "work": w, "probe": case["probe"]}


def _labels_inputs(case, seed):
    t = dg.table_learned(case["rows"], seed=seed * 7 + 1, device=DEV)
    return t, dg.preds_anchored(t, case["preds"], seed=seed * 7 + 2)


def _prepare_labels(case, seed):
    t, specs = _labels_inputs(case, seed)
    ctx, dt = esc.Context(0), _device_table(t)
    return {"ctx": ctx, "table": dt, "preds": [esc.Pred(dt, p) for p in specs]}


def _join_inputs(case, seed):
    """Probe columns and the filtered build keys of both sides."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7 + 1)
    probe, build = [], []
    for n, sel in ((case["r"], case["sel_r"]), (case["s"], case["sel_s"])):
        k = max(1, int(n * sel))
        if case["keys"] == "perm":        # surrogate keys 0..n-1 in no order; a selection keeps k of them
            ids = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
            build.append(ids[:k].contiguous())
            probe.append(torch.randint(0, n, (case["rows"],), generator=g, device=DEV, dtype=torch.int32))
        elif case["keys"] == "wide":      # keys anywhere in the 32-bit integers; probe rows name any of the n
            ids = torch.randint(-2**31, 2**31, (n,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
            build.append(ids[:k].contiguous())
            probe.append(ids[torch.randint(0, n, (case["rows"],), generator=g, device=DEV)])
        else:                             # an attribute join: about four build rows per key
            d = max(1, n // 4)
            build.append(torch.randint(-(d // 2), d - d // 2, (k,), generator=g, device=DEV, dtype=torch.int32))
            probe.append(torch.randint(-(d // 2), d - d // 2, (case["rows"],), generator=g, device=DEV,
                                       dtype=torch.int32))
    # the exact counts order the lookups: the more selective side first
    if case["sel_s"] < case["sel_r"]:
        probe.reverse()
        build.reverse()
    return probe, build


def _prepare_join(case, seed):
    probe, build = _join_inputs(case, seed)
    ctx = esc.Context(0)
    return {"ctx": ctx, "build": build, "probe": esc.Table(case["rows"], [esc.INT32, esc.INT32], probe)}


def _mlp_inputs(n, seed):
    """Features in [0, 1] (many of them exactly 0 or 1) and ln-selectivity
    labels, with the estimator's initial parameters."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7 + 1)
    x = torch.rand((n, 64), generator=g, device=DEV)
    u = torch.rand((n, 64), generator=g, device=DEV)
    x = torch.where(u < 0.4, torch.zeros_like(x), torch.where(u < 0.55, torch.ones_like(x), x)).contiguous()
    y = -14.0 * torch.rand((n,), generator=g, device=DEV) ** 2 - 2.0 * x[:, 0]
    return x, y, dg.mlp_init(seed * 7 + 2)


def _prepare_predict(case, seed):
    x, _, params = _mlp_inputs(case["rows"], seed)
    ctx = esc.Context(0)
    return {"ctx": ctx, "mlp": esc.MLP(ctx, params), "x": x,
            "out": torch.zeros(case["rows"], dtype=torch.float32, device=DEV), "stream": torch.cuda.current_stream()}


def _order(case, seed):
    epochs = -(-case["steps"] * case["batch"] // (case["samples"] // case["batch"] * case["batch"]))
    return dg.minibatch_order(case["samples"], case["batch"], epochs, seed * 7 + 3)[:case["steps"] * case["batch"]]


def _prepare_train(case, seed):
    x, y, params = _mlp_inputs(case["samples"], seed)
    ctx = esc.Context(0)
    return {"ctx": ctx, "mlp": esc.MLP(ctx, params), "x": x, "y": y, "steps": case["steps"], "batch": case["batch"],
            "order": torch.from_numpy(_order(case, seed)).to(DEV)}


def _prepare_gradients(case, seed):
    x, y, params = _mlp_inputs(case["rows"], seed)
    ctx = esc.Context(0)
    return {"ctx": ctx, "mlp": esc.MLP(ctx, params), "x": x, "y": y}


# ---------------------------------------------------------------- the passes


def run(s):
    return globals()["_run_" + s["kind"]](s)


def _run_count(s):
    return [s["ctx"].count(s["table"], p, ws=s["ws"], stream=s["stream"]) for p in s["preds"]]


def _run_select(s):
    ctx, dt, preds, ws, st = s["ctx"], s["table"], s["preds"], s["ws"], s["stream"]
    out = []
    ctx.count_begin(dt, preds[0], ws[0], 0, stream=st)
    for i, p in enumerate(preds):
        if i + 1 < len(preds):
            ctx.count_begin(dt, preds[i + 1], ws[(i + 1) % 2], (i + 1) % 2, stream=st)
        c = ctx.count_end(i % 2)
        ids, cols = s["ids"][i], s["outs"][i]
        ctx.materialize_async(dt, p, s["proj"], ids, cols, ids.numel(), s["counts"][i:i + 1], ws[i % 2], stream=st)
        out.append([c, ids] + cols)
    return out


def _run_materialize(s):
    out = []
    for p, ids, cols in zip(s["preds"], s["ids"], s["outs"]):
        c = s["ctx"].materialize(s["table"], p, s["proj"], ids, cols, ids.numel(), ws=s["ws"], stream=s["stream"])
        out.append([c, ids[:c]] + [v[:c] for v in cols])
    return out


def _run_conjuncts(s):
    return [s["ctx"].count_conjuncts(s["table"], p, stream=s["stream"]) for p in s["preds"]]


def _run_planning(s):
    return s["work"].run_batched(exact_probe=s["probe"])["counts"].astype(np.int64)


def _run_labels(s):
    return learned.exact_counts(s["ctx"], s["table"], s["preds"]).astype(np.int64)


def _run_join(s):
    tabs = [s["ctx"].hash_table(k) for k in s["build"]]
    return s["ctx"].join_count(s["probe"], [0, 1], tabs)


def _run_predict(s):
    return s["mlp"].predict(s["x"], out=s["out"], stream=s["stream"])


def _run_train(s):
    loss = s["mlp"].train(s["x"], s["y"], s["order"], s["steps"], s["batch"])
    return {"loss": loss, "params": s["mlp"].get_params()}


def _run_gradients(s):
    return s["mlp"].gradients(s["x"], s["y"])


# ---------------------------------------------------------------- work


PARAMS = 64 * 256 + 2 * 256 * 256 + 256 + 3 * 256 + 1
FLOPS_ROW = 2 * (64 * 256 + 2 * 256 * 256 + 256)


def work(case):
    kind, n = case["kind"], case.get("rows", 0)
    if kind in ("count", "conjuncts", "select") and case.get("table") != "plain":
        sels = [STAR_SELECTIONS[i % len(STAR_SELECTIONS)] for i in range(case["preds"])]
        b = sum(4 * n * len(sel) for sel in sels)
        if kind == "select":   # per qualifying row: three values read, a row id and three values written
            b += sum(n * _star_sel(sel) * 4 * (2 * len(STAR_PROJECTION) + 1) for sel in sels)
        return {"bytes": b, "flops": 0}
    if kind == "count":
        return {"bytes": case["preds"] * 3 * 4 * n, "flops": 0}
    if kind == "materialize":
        return {"bytes": 2 * (4 * n + case["sel"] * n * 4 * (2 * case["proj"] + 1)), "flops": 0}
    if kind == "planning":
        rows = (max(1000, n // 100) + max(1000, n // 10) + (n if case["probe"] else 0))
        return {"bytes": -(-case["queries"] // 64) * rows * 16, "flops": 0}
    if kind == "labels":
        return {"bytes": 6 * 4 * n, "flops": 0}
    if kind == "join":
        return {"bytes": 8 * n + 4 * (case["r"] * case["sel_r"] + case["s"] * case["sel_s"]), "flops": 0}
    if kind == "predict":
        return {"bytes": n * 65 * 4 + PARAMS * 2, "flops": n * FLOPS_ROW}
    if kind == "train":
        return {"bytes": case["steps"] * case["batch"] * 65 * 4 + 6 * PARAMS * 4,
                "flops": 3 * case["steps"] * case["batch"] * FLOPS_ROW}
    return {"bytes": n * 65 * 4 + PARAMS * 4, "flops": 3 * n * FLOPS_ROW}


# ---------------------------------------------------------------- plain torch results


def _k(col, v):
    return torch.tensor(v, dtype=col.dtype, device=col.device)


def _cmp(x, test):
    if test[0] == "eq":
        return x == _k(x, test[1])
    if test[0] == "lt":
        return x < _k(x, test[1])
    if test[0] == "gt":
        return x > _k(x, test[1])
    if test[0] == "between":
        return (x >= _k(x, test[1])) & (x <= _k(x, test[2]))
    m = torch.zeros_like(x, dtype=torch.bool)
    for v in test[1]:
        m |= x == _k(x, v)
    return m


def _wrap(x):
    return ((x + 2**31) % 2**32) - 2**31


def _value(cols, e):
    if e[0] == "col":
        return cols[e[1]].to(torch.int64)
    if e[0] == "const":
        return e[1]
    a, b = _value(cols, e[1]), _value(cols, e[2])
    if e[0] == "mul":
        return _wrap(a * b)
    if e[0] == "add":
        return _wrap(a + b)
    return torch.fmod(a, b)   # mod: the truncated remainder


def _mask(cols, p):
    if p[0] in ("and", "or"):
        m = _mask(cols, p[1][0])
        for q in p[1][1:]:
            m = m & _mask(cols, q) if p[0] == "and" else m | _mask(cols, q)
        return m
    if p[0] == "udf":
        return _cmp(_value(cols, p[1]), p[2])
    return _cmp(cols[p[1]], (p[0],) + tuple(p[2:]))


def exact(case, seed):
    return globals()["_exact_" + case["kind"]](case, int(seed))


def _exact_count(case, seed):
    t, specs = _count_inputs(case, seed)
    return [int(_mask(t.cols, p).sum()) for p in specs]


def _kept(cols, p, proj):
    rows = _mask(cols, p).nonzero()[:, 0]
    return [rows.numel(), rows.to(torch.int32)] + [cols[j][rows] for j in proj]


def _exact_select(case, seed):
    t, specs = _star_inputs(case, seed)
    return [_kept(t.cols, p, STAR_PROJECTION) for p in specs]


def _exact_materialize(case, seed):
    t, specs, _, proj = _materialize_inputs(case, seed)
    return [_kept(t.cols, p, proj) for p in specs]


def _exact_conjuncts(case, seed):
    t, specs = _star_inputs(case, seed)
    out = []
    for p in specs:
        ms = [_mask(t.cols, q) for q in p[1]]
        pre = [ms[0]]
        for m in ms[1:]:
            pre.append(pre[-1] & m)
        out.append(([int(m.sum()) for m in ms], [int(m.sum()) for m in pre]))
    return out


def _exact_planning(case, seed):
    tabs, queries = _planning_inputs(case, seed)
    return np.array([[int(_mask(t.cols, p).sum()) if i < 2 or case["probe"] else 0
                      for i, (t, p) in enumerate(zip(tabs, q))] for q in queries], np.int64)


def _exact_labels(case, seed):
    t, specs = _labels_inputs(case, seed)
    return np.array([int(_mask(t.cols, p).sum()) for p in specs], np.int64)


def _exact_join(case, seed):
    probe, build = _join_inputs(case, seed)
    prod = None
    for p, b in zip(probe, build):
        keys, cnt = torch.unique(b, return_counts=True)
        at = torch.searchsorted(keys, p).clamp_(max=keys.numel() - 1)
        c = torch.where(keys[at] == p, cnt[at], torch.zeros_like(cnt[at]))
        prod = c if prod is None else prod * c
    return int(prod.sum())


def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _forward64(params, x):
    """Outputs and layer inputs; matrix operands are bfloat16, as the network is defined, sums are in 64 bits."""
    a = _bf16(x)
    acts = [a]
    for w, b in params[:-1]:
        a = _bf16(torch.relu(a @ _bf16(w) + b))
        acts.append(a)
    return (a @ _bf16(params[-1][0]) + params[-1][1])[:, 0], acts


def _params64(params):
    return [(torch.from_numpy(w).to(DEV).double(), torch.from_numpy(b).to(DEV).double()) for w, b in params]


def _gradients64(params, x, y):
    yhat, acts = _forward64(params, x)
    e = yhat - y.double()
    loss = torch.where(e.abs() <= HUBER, 0.5 * e * e, HUBER * (e.abs() - 0.5 * HUBER)).mean()
    d = e.clamp(-HUBER, HUBER) / len(y)
    grads = [(acts[-1].T @ d[:, None], d.sum().reshape(1))]
    dh = d[:, None] @ _bf16(params[-1][0]).T
    for i in range(len(params) - 2, -1, -1):
        dz = dh * (acts[i + 1] > 0)
        g = _bf16(dz)
        grads.insert(0, (acts[i].T @ g, dz.sum(0)))
        if i:
            dh = g @ _bf16(params[i][0]).T
    return grads, loss


def _flat(layers):
    return torch.cat([v.reshape(-1) for layer in layers for v in layer])


def _exact_predict(case, seed):
    x, _, params = _mlp_inputs(case["rows"], seed)
    return _forward64(_params64(params), x)[0]


def _exact_gradients(case, seed):
    x, y, params = _mlp_inputs(case["rows"], seed)
    return _flat(_gradients64(_params64(params), x, y)[0])


def _exact_train(case, seed):
    x, y, init = _mlp_inputs(case["samples"], seed)
    params = _params64(init)
    order = torch.from_numpy(_order(case, seed)).to(DEV).long().reshape(case["steps"], case["batch"])
    m = [[torch.zeros_like(v) for v in layer] for layer in params]
    v2 = [[torch.zeros_like(v) for v in layer] for layer in params]
    losses = []
    for t, rows in enumerate(order, 1):
        grads, loss = _gradients64(params, x[rows], y[rows])
        losses.append(loss)
        new = []
        for i, layer in enumerate(params):
            moved = []
            for j, p in enumerate(layer):
                g = grads[i][j].reshape(p.shape)
                m[i][j] = 0.9 * m[i][j] + 0.1 * g
                v2[i][j] = 0.999 * v2[i][j] + 0.001 * g * g
                moved.append(p - 1e-3 * (m[i][j] / (1 - 0.9 ** t)) / ((v2[i][j] / (1 - 0.999 ** t)).sqrt() + 1e-8))
            new.append(tuple(moved))
        params = new
    return {"loss": torch.stack(losses).cpu().numpy(), "params": _flat(params).cpu().numpy()}
