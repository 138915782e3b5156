"""The work that a program has this library do, as cases that can be timed.

A case is a dict of plain values. `listed()` are the ones that stand for real
use at fixed sizes, `draw(rng)` gives others of the same ranges, `prepare` makes
a case's inputs and keeps the handles that a program keeps, `run` is one pass
through the public entry points of `paper_2608_13696_amd.rel`, `work` the bytes
and operations that the pass cannot do without, and `exact` the same outputs in
plain torch.

The kinds of case:

* ``query``   -- `Context.filter_join_agg`: the whole filter, join and group-by, sized plainly.
* ``planned`` -- `Planner.plan`, then the query with the plan it gave.
* ``filter``  -- `Context.filter_compact`: a selection vector from one column.
* ``pred``    -- `Predicate.filter`: a conjunction over typed columns, compiled or interpreted.
* ``join``    -- `join_build`, `JoinTable.probe` and `join_gather`: the join operator by operator, a table built for each query.
* ``groupby`` -- `Context.groupby_agg` over 64-bit keys, with or without a selection vector.
* ``batch``   -- `Batch.run`: many independent queries in one launch.
* ``mlp``     -- forward, backward and Adam step of the planner's network.

Columns are those of the star join that the library's generators draw: fk
uniform or Zipf over the dim keys, price_cents in [90000, 10500000], qty in
[1, 50], day in [0, 2557), flag in {0, 1, 2}; pk a permutation, prio in
{0..4}, grp uniform in [0, groups).
"""
from __future__ import annotations

import math

import torch

from paper_2608_13696_amd import autotune, planner_train, rel

DAYS = 2557
PRICE_LO, PRICE_HI = 90_000, 10_500_000
SAMPLE = 256  # rows of each table that the planner's sketch looks at


def listed() -> list[dict]:
    return [
        # The smallest query of the library's benchmark: six short kernels, where launches and latency are the cost.
        dict(name="query_60k_prio_flag", kind="query", n=60_000, m=15_000, by="prio_flag", zipf=0.0, stride=1, groups=0,
             day_lt=1800, stats=False),
        # A reporting query at scale factor 1: few groups, a join index that fits L2.
        dict(name="query_6m_prio_flag", kind="query", n=6_000_000, m=1_500_000, by="prio_flag", zipf=0.0, stride=1,
             groups=0, day_lt=1800, stats=False),
        # The headline workload: scale factor 10, skewed foreign keys, one group per key that has rows.
        dict(name="query_60m_fk", kind="query", n=60_000_000, m=15_000_000, by="fk", zipf=0.8, stride=1, groups=0,
             day_lt=1200, stats=False),
        # A query whose group count nobody knows beforehand: sketch, network and the sized run.
        dict(name="planned_60m_dim_grp", kind="planned", n=60_000_000, m=15_000_000, by="dim_grp", zipf=1.2, stride=1,
             groups=100_000, day_lt=1200, stats=False),
        # A stand-alone selection over a whole column, of a size that no tile divides.
        dict(name="filter_60m", kind="filter", n=59_999_999, op="lt", day_lt=1200),
        # A WHERE clause that is prepared once and run often.
        dict(name="pred_compiled_60m", kind="pred", n=60_000_000, mode="compiled", terms="day,qty,price,flag", width=0.0),
        # The same clause run ad hoc, where compiling it first would cost more than it saves.
        dict(name="pred_interpreted_60m", kind="pred", n=60_000_000, mode="interpreted", terms="day,qty,price,flag",
             width=0.0),
        # The join as separate operators, for programs that want the joined rows and not their sums.
        dict(name="join_60m", kind="join", n=60_000_000, m=15_000_000, zipf=0.8, stride=1, day_lt=1200, payload=False),
        # Grouping a selection by a few codes: every row lands on one of a handful of groups.
        dict(name="groupby_6m_15", kind="groupby", n=6_000_000, groups=15, spread=1, selected=0.7, hint=True),
        # Grouping by a wide key: more groups than any on-chip table holds (customers, sessions), of an odd size.
        dict(name="groupby_20m_2m", kind="groupby", n=19_999_999, groups=2_000_000, spread=1009, selected=1.0, hint=True),
        # Thousands of small queries at once, of very different sizes: the batched benchmark.
        dict(name="batch_4096", kind="batch", k=4096, lo=1000, hi=1_000_000, table_seed=4),
        # One training step of the planner's network at its batch size.
        dict(name="mlp_step_256", kind="mlp", rows=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["query", "query", "query", "planned", "filter", "pred", "pred", "join", "groupby", "groupby", "batch",
                       "mlp"])
    if kind in ("query", "planned"):
        n = _log(rng, 1_000, 60_000_000)
        m = max(16, min(15_000_000, int(n / 4 * math.exp(rng.uniform(math.log(0.25), math.log(4.0))))))
        by = "dim_grp" if kind == "planned" else rng.choice(["prio_flag", "fk", "dim_grp"])
        return dict(kind=kind, n=n, m=m, by=by, zipf=rng.choice([0.0, 0.5, 0.8, 1.2]), stride=rng.choice([1, 1, 1, 3, 40]),
                    groups=_log(rng, 1, m) if by == "dim_grp" else 0, day_lt=rng.randrange(128, 2430),
                    stats=kind == "query" and rng.random() < 0.3)
    if kind == "filter":
        return dict(kind=kind, n=_log(rng, 1_000, 60_000_000), op=rng.choice(["lt", "le", "gt", "ge", "eq", "ne"]),
                    day_lt=rng.randrange(25, 2530))
    if kind == "pred":
        names = rng.sample(list(TERMS), rng.randrange(1, 6))
        return dict(kind=kind, n=_log(rng, 1_000, 60_000_000), mode=rng.choice(["compiled", "interpreted"]),
                    terms=",".join(names), width=rng.choice([0.0, 0.1, 0.3]))
    if kind == "join":
        n = _log(rng, 1_000, 60_000_000)
        m = max(16, min(15_000_000, int(n / 4 * math.exp(rng.uniform(math.log(0.25), math.log(4.0))))))
        return dict(kind=kind, n=n, m=m, zipf=rng.choice([0.0, 0.5, 0.8, 1.2]), stride=rng.choice([1, 1, 1, 3, 40]),
                    day_lt=rng.randrange(128, 2430), payload=rng.random() < 0.4)
    if kind == "groupby":
        hint = rng.random() < 0.5  # without one the table is sized for as many groups as rows
        n = _log(rng, 1_000, 20_000_000 if hint else 8_000_000)
        return dict(kind=kind, n=n, groups=_log(rng, 1, max(2, n // 4)), spread=rng.choice([1, 1, 1009, 1 << 33]),
                    selected=rng.choice([1.0, round(rng.uniform(0.1, 0.9), 3)]), hint=hint)
    if kind == "batch":
        hi = _log(rng, 4_000, 1_000_000)
        return dict(kind=kind, k=_log(rng, 8, 512), lo=1000, hi=hi, table_seed=rng.randrange(1000))
    return dict(kind=kind, rows=_log(rng, 1, 16_384))


# -- inputs ------------------------------------------------------------------------------------------------------------

#: The terms that a predicate case combines: column type, how its values are drawn, the operator and its literals. `width`
#: widens BETWEEN's range, so that other shares of the rows pass.
TERMS = {
    "day": (torch.int32, (0, DAYS), "between", lambda w: [100 - int(100 * w), 1800 + int(700 * w)]),
    "qty": (torch.int32, (1, 51), "in", lambda w: list(range(1, 33, 2))),
    "price": (torch.int64, (PRICE_LO, PRICE_HI + 1), "lt", lambda w: [6_000_000 + int(4_000_000 * w)]),
    "flag": (torch.int8, (0, 3), "ne", lambda w: [2]),
    "store": (torch.int16, (0, 1200), "ge", lambda w: [300 - int(300 * w)]),
    "discount": (torch.float32, None, "le", lambda w: [0.75 + 0.2 * w]),
    "weight": (torch.float64, None, "gt", lambda w: [0.25 - 0.2 * w]),
}

_ctx = None


def _context() -> rel.Context:
    """The one context of the program: it keeps the library's scratch memory."""
    global _ctx
    if _ctx is None:
        _ctx = rel.Context(0)
    return _ctx


def _dev():
    return torch.device("cuda:0")


def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=_dev()).manual_seed(seed)


def _ints(g, n, lo, hi, dtype):
    return torch.randint(lo, hi, (n,), generator=g, device=_dev(), dtype=dtype)


def _keys(g, n, m, s):
    """n ranks in [0, m): uniform, or Zipf(s) by its inverse distribution."""
    if not s:
        return _ints(g, n, 0, m, torch.int32)
    u = torch.rand(n, generator=g, device=_dev(), dtype=torch.float64)
    r = u.mul_((m + 1.0) ** (1 - s) - 1).add_(1).pow_(1 / (1 - s)).sub_(1)
    return r.clamp_(0, m - 1).to(torch.int32)


def _tables(case, seed):
    g, n, m, stride = _gen(seed), case["n"], case["m"], case["stride"]
    fact = {"fk": _keys(g, n, m, case["zipf"]).mul_(stride), "price_cents": _ints(g, n, PRICE_LO, PRICE_HI + 1, torch.int64),
            "qty": _ints(g, n, 1, 51, torch.int32), "day": _ints(g, n, 0, DAYS, torch.int32),
            "flag": _ints(g, n, 0, 3, torch.int8)}
    dim = {"pk": torch.randperm(m, generator=g, device=_dev(), dtype=torch.int32).mul_(stride),
           "prio": _ints(g, m, 0, 5, torch.int8),
           "grp": _ints(g, m, 0, case["groups"], torch.int32) if case.get("groups") else None}
    return fact, dim


def _batch_sizes(case):
    """Per instance: fact rows log-uniform, a quarter as many dim rows, groups log-uniform in [1, 65536], selectivity
    uniform in [0.05, 0.95]."""
    g = torch.Generator().manual_seed(case["table_seed"])
    u = torch.rand(case["k"], 3, generator=g, dtype=torch.float64).tolist()
    out = []
    for a, b, c in u:
        n = int(round(math.exp(math.log(case["lo"]) + a * math.log(case["hi"] / case["lo"]))))
        out.append((n, max(n // 4, 1), max(1, int(round(math.exp(b * math.log(65536.0))))), int(round((0.05 + 0.9 * c) * DAYS))))
    return out


def _batch_tables(case, seed):
    """All instances' columns in one tensor each (instances start at multiples of 16 rows), with per-instance views' bounds."""
    sizes, g = _batch_sizes(case), _gen(seed)
    fo, do = [0], [0]
    for n, m, _, _ in sizes:
        fo.append(fo[-1] + -(-n // 16) * 16)
        do.append(do[-1] + -(-m // 16) * 16)
    d = _dev()
    n_of = torch.tensor([s[0] for s in sizes], device=d)
    m_of = torch.tensor([s[1] for s in sizes], device=d)
    frows = torch.tensor([b - a for a, b in zip(fo, fo[1:])], device=d)
    drows = torch.tensor([b - a for a, b in zip(do, do[1:])], device=d)
    inst = torch.repeat_interleave(torch.arange(len(sizes), device=d), frows)
    dinst = torch.repeat_interleave(torch.arange(len(sizes), device=d), drows)
    N, M = fo[-1], do[-1]
    u = torch.rand(N, generator=g, device=d, dtype=torch.float64)
    fact = {"fk": (u * m_of[inst]).to(torch.int32), "price_cents": _ints(g, N, PRICE_LO, PRICE_HI + 1, torch.int64),
            "qty": _ints(g, N, 1, 51, torch.int32), "day": _ints(g, N, 0, DAYS, torch.int32), "flag": None}
    # a permutation of each instance's keys: its rows sorted by (instance, padding last, random)
    doff = torch.tensor(do[:-1], device=d)
    local = torch.arange(M, device=d) - doff[dinst]
    key = (dinst << 33) | ((local >= m_of[dinst]).to(torch.int64) << 32) | torch.randint(0, 1 << 32, (M,), generator=g, device=d)
    pk = (torch.argsort(key) - doff[dinst]).to(torch.int32)
    g_of = torch.tensor([s[2] for s in sizes], device=d)
    dim = {"pk": pk, "prio": None, "grp": (torch.rand(M, generator=g, device=d, dtype=torch.float64) * g_of[dinst]).to(torch.int32)}
    return sizes, fo, do, fact, dim


def _network(case, seed):
    g, B = _gen(seed), case["rows"]
    p = []
    for i, o in ((40, 64), (64, 64), (64, 2)):
        p += [torch.randn(i * o, generator=g, device=_dev()) * math.sqrt(2.0 / i), torch.zeros(o, device=_dev())]
    x = torch.randn(B, 40, generator=g, device=_dev())
    t = torch.randn(B, 2, generator=g, device=_dev()) * 2 - 3
    return torch.cat(p).contiguous(), x, t


def prepare(case: dict, seed: int) -> dict:
    kind, ctx = case["kind"], _context()
    st = {"case": case, "ctx": ctx}
    if kind != "mlp":
        st["size"] = _size(case)
    if kind in ("query", "planned"):
        st["fact"], st["dim"] = _tables(case, seed)
        if kind == "planned":
            g = _gen(seed + 1)
            st["samples"] = _ints(g, SAMPLE, 0, case["n"], torch.int64), _ints(g, SAMPLE, 0, case["m"], torch.int64)
            st["planner"] = rel.Planner(ctx, *planner_train.load_model()[:4])
    elif kind == "filter":
        st["col"] = _ints(_gen(seed), case["n"], 0, DAYS, torch.int32)
    elif kind == "pred":
        st["cols"] = _pred_columns(case, seed)
        names = case["terms"].split(",")
        terms = [dict(column=i, op=TERMS[t][2], values=TERMS[t][3](case["width"])) for i, t in enumerate(names)]
        st["pred"] = rel.Predicate(ctx, terms, [TERMS[t][0] for t in names], case["mode"])
    elif kind == "join":
        st["fact"], st["dim"] = _tables(case, seed)
        st["sel"] = ctx.filter_compact(st["fact"]["day"], "lt", case["day_lt"])[0]
    elif kind == "groupby":
        st["rows"] = _groupby_rows(case, seed)
    elif kind == "batch":
        sizes, fo, do, fact, dim = _batch_tables(case, seed)
        insts = []
        for i, (n, m, groups, day_lt) in enumerate(sizes):
            insts.append(({k: None if v is None else v[fo[i]:fo[i] + n] for k, v in fact.items()},
                          {k: None if v is None else v[do[i]:do[i] + m] for k, v in dim.items()}, day_lt, "dim_grp", groups))
        st["batch"] = rel.Batch(ctx, insts, tuning=autotune.load())
        st["batch"].run()  # a program's own first run: it loads the graph
        st["batch"].sync()
    else:
        st["params"], st["x"], st["t"] = _network(case, seed)
        st["m"], st["v"], st["step"] = torch.zeros_like(st["params"]), torch.zeros_like(st["params"]), 0
    return st


def _pred_columns(case, seed):
    g, n, cols = _gen(seed), case["n"], []
    for t in case["terms"].split(","):
        dtype, span = TERMS[t][:2]
        cols.append(torch.rand(n, generator=g, device=_dev(), dtype=dtype) if span is None else _ints(g, n, *span, dtype))
    return cols


def _groupby_rows(case, seed):
    g, n = _gen(seed), case["n"]
    key = _ints(g, n, 0, case["groups"], torch.int64).mul_(case["spread"])
    sel = None
    if case["selected"] < 1:
        sel = torch.nonzero(torch.rand(n, generator=g, device=_dev()) < case["selected"]).flatten().to(torch.int32)
    return key, _ints(g, n, PRICE_LO, PRICE_HI + 1, torch.int64), _ints(g, n, 1, 51, torch.int32), sel


# -- a pass ------------------------------------------------------------------------------------------------------------

class Rows(dict):
    """Columns of which the first `count` rows (a device word) are the result; what reads them gets `size` rows, with
    zeros after the result's. Where the library leaves the order of the rows open, they read in the order of column `by`:
    whoever looks at them sorts them, the pass itself does not."""

    def __init__(self, columns, count, size, by=None):
        super().__init__(columns, rows=count)
        self._count, self._size, self._by, self._order = count, size, by, None

    def __getitem__(self, name):
        if name == "rows":
            return self._count
        n, column = int(self._count), super().__getitem__(name)
        if self._by is not None and self._order is None:
            self._order = torch.argsort(super().__getitem__(self._by)[:n])
        return _padded(column[:n] if self._by is None else column[:n][self._order], self._size)


class Batches(dict):
    """The groups of all instances of a batch, instance after instance, each in the order of its keys."""

    def __init__(self, outs, size):
        super().__init__(key=None, sum_price=None, sum_qty=None, count=None, n_groups=None)
        self._outs, self._size, self._order = outs, size, None

    def __getitem__(self, name):
        counts = torch.cat([o.n_groups for o in self._outs])
        if name == "n_groups":
            return counts
        sizes = counts.tolist()
        rows = torch.cat([getattr(o, name)[:c] for o, c in zip(self._outs, sizes)])
        if self._order is None:
            key = torch.cat([o.key[:c] for o, c in zip(self._outs, sizes)])
            inst = torch.repeat_interleave(torch.arange(len(sizes), device=key.device), counts)
            self._order = torch.argsort((inst << 32) + key)
        return _padded(rows[self._order], self._size)


def _padded(rows, size):
    return torch.cat([rows, rows.new_zeros(max(0, size - rows.numel()))])


def _groups(out, size) -> Rows:
    return Rows(dict(key=out.key, sum_price=out.sum_price, sum_qty=out.sum_qty, count=out.count), out.n_groups, size, "key")


def _size(case) -> int:
    """The most rows that a pass can return."""
    if case["kind"] in ("query", "planned"):
        return {"prio_flag": 15, "fk": min(case["n"], case["m"]), "dim_grp": case["groups"]}[case["by"]]
    if case["kind"] == "batch":
        return sum(min(n, m, groups) for n, m, groups, _ in _batch_sizes(case))
    return case["groups"] if case["kind"] == "groupby" else case["n"]


def run(st: dict):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "query":
        out, stats = ctx.filter_join_agg(st["fact"], st["dim"], case["day_lt"], case["by"], stats=case["stats"])
        return [_groups(out, st["size"]), *([stats[k] for k in ("rows_passed", "join_matches", "groups")] if stats else [])]
    if kind == "planned":
        plan, pred = st["planner"].plan(st["fact"], st["dim"], case["day_lt"], case["by"], *st["samples"])
        out, _ = ctx.filter_join_agg(st["fact"], st["dim"], case["day_lt"], case["by"], plan=plan, stats=case["stats"])
        return [_groups(out, st["size"]), *pred]
    if kind == "filter":
        idx, count = ctx.filter_compact(st["col"], case["op"], case["day_lt"], sync=False)
        return Rows(dict(idx=idx), count, st["size"])
    if kind == "pred":
        idx, count = st["pred"].filter(st["cols"], sync=False)
        return Rows(dict(idx=idx), count, st["size"])
    if kind == "join":
        fact, dim = st["fact"], st["dim"]
        table = ctx.join_build(dim["pk"], dim["prio"].to(torch.int32) if case["payload"] else None)
        fi, di, count = table.probe(fact["fk"], st["sel"], sync=False)
        if case["payload"]:  # the table itself brings the one dim column
            cols = ctx.join_gather(fi, None, count, [(fact["price_cents"], "fact"), (fact["qty"], "fact")])
        else:
            cols = ctx.join_gather(fi, di, count, [(fact["price_cents"], "fact"), (fact["qty"], "fact"), (fact["day"], "fact"),
                                                   (dim["prio"], "dim")])
        table.close()
        return Rows({"row": fi, "payload": di, **{"col%d" % i: c for i, c in enumerate(cols)}}, count, st["size"], "row")
    if kind == "groupby":
        key, price, qty, sel = st["rows"]
        hint = case["groups"] if case["hint"] else 0
        return _groups(ctx.groupby_agg(key, price, qty, sel, capacity_hint=hint, out_cap=hint or None), st["size"])
    if kind == "batch":
        st["batch"].run()
        return Batches(st["batch"].outs, st["size"])
    st["step"] += 1
    y = rel.mlp_forward(ctx, st["params"], st["x"])
    grad, loss = rel.mlp_backward(ctx, st["params"], st["x"], st["t"])
    rel.mlp_adam_step(ctx, st["params"], st["m"], st["v"], grad, st["step"])
    return dict(y=y, loss=loss, grad=grad, params=st["params"], m=st["m"], v=st["v"])


# -- what a pass cannot do without -------------------------------------------------------------------------------------

def _distinct(rows, m, s):
    """Expected distinct keys of `rows` draws from m keys."""
    if not s:
        return m * -math.expm1(-rows / m)
    total, lo, tot = 0.0, 1.0, (m + 1.0) ** (1 - s) - 1
    while lo < m + 1:
        hi = min(lo * 1.05 + 1, m + 1.0)
        p = (hi ** (1 - s) - lo ** (1 - s)) / tot
        total += (hi - lo) * -math.expm1(-rows * p / (hi - lo))
        lo = hi
    return total


def work(case: dict) -> dict:
    kind = case["kind"]
    if kind in ("query", "planned"):
        n, m = case["n"], case["m"]
        r = n * case["day_lt"] / DAYS
        keys = _distinct(r, m, case["zipf"])
        g = {"fk": keys, "prio_flag": min(15.0, keys)}.get(case["by"]) or _distinct(keys, case["groups"], 0)
        return {"bytes": n * (21 if case["by"] == "prio_flag" else 20) + m * {"fk": 4, "prio_flag": 5, "dim_grp": 8}[case["by"]] + 32 * g,
                "flops": 0}
    if kind == "filter":
        lit = case["day_lt"]
        share = {"lt": lit, "le": lit + 1, "gt": DAYS - lit - 1, "ge": DAYS - lit, "eq": 1, "ne": DAYS - 1}[case["op"]] / DAYS
        return {"bytes": 4 * case["n"] * (1 + share), "flops": 0}
    if kind == "pred":
        share, width = 1.0, 0
        for t in case["terms"].split(","):
            dtype, span, op, lits = TERMS[t]
            v = lits(case["width"])
            lo, hi = span or (0.0, 1.0)
            share *= {"between": lambda: (v[-1] - v[0] + 1) / (hi - lo), "in": lambda: len(v) / (hi - lo), "lt": lambda: (v[0] - lo) / (hi - lo),
                      "ne": lambda: 1 - 1 / (hi - lo), "ge": lambda: (hi - v[0]) / (hi - lo), "le": lambda: (v[0] - lo) / (hi - lo),
                      "gt": lambda: (hi - v[0]) / (hi - lo)}[op]()
            width += torch.empty(0, dtype=dtype).element_size()
        return {"bytes": case["n"] * (width + 4 * min(1.0, share)), "flops": 0}
    if kind == "join":
        r = case["n"] * case["day_lt"] / DAYS
        out = 8 + (12 if case["payload"] else 17)
        return {"bytes": case["m"] * (8 if case["payload"] else 5) + r * (4 + 4 + (12 if case["payload"] else 16) + out), "flops": 0}
    if kind == "groupby":
        r = case["n"] * case["selected"]
        return {"bytes": r * (20 + (4 if case["selected"] < 1 else 0)) + 32 * _distinct(r, case["groups"], 0), "flops": 0}
    if kind == "batch":
        b = 0.0
        for n, m, groups, day_lt in _batch_sizes(case):
            b += 20 * n + 8 * m + 32 * _distinct(_distinct(n * day_lt / DAYS, m, 0), groups, 0)
        return {"bytes": b, "flops": 0}
    # forward; forward and backward; the update
    return {"bytes": 4 * (6914 * 8 + case["rows"] * 46), "flops": case["rows"] * 2 * 6784 * 4}


# -- the same in plain torch -------------------------------------------------------------------------------------------

def _rows(case, **columns) -> dict:
    """The columns as `Rows` reads them."""
    n = next(iter(columns.values())).numel()
    return {"rows": torch.tensor([n]), **{k: _padded(v, _size(case)) for k, v in columns.items()}}


def _sums(group, price, qty, size):
    """Groups in ascending order of their number: which have rows, and their sums."""
    d = group.device
    count = torch.zeros(size, dtype=torch.int64, device=d).scatter_add_(0, group, torch.ones_like(group))
    sp = torch.zeros(size, dtype=torch.int64, device=d).scatter_add_(0, group, price)
    sq = torch.zeros(size, dtype=torch.int64, device=d).scatter_add_(0, group, qty.to(torch.int64))
    own = torch.nonzero(count).flatten()
    return own, sp[own], sq[own], count[own]


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind in ("query", "planned"):
        fact, dim = _tables(case, seed)
        stride = case["stride"]
        keep = torch.nonzero(fact["day"] < case["day_lt"]).flatten()
        fk = (fact["fk"][keep] // stride).to(torch.int64)  # every fk is the key of a dim row
        pk = (dim["pk"] // stride).to(torch.int64)
        if case["by"] == "fk":
            group, size = fk, case["m"]
        else:
            attr = torch.empty(case["m"], dtype=torch.int64, device=_dev())
            attr[pk] = (dim["prio"] if case["by"] == "prio_flag" else dim["grp"]).to(torch.int64)
            group, size = attr[fk], case["groups"]
            if case["by"] == "prio_flag":
                group, size = group * 256 + fact["flag"][keep].to(torch.int64), 5 * 256
        key, sp, sq, count = _sums(group, fact["price_cents"][keep], fact["qty"][keep], size)
        groups = _rows(case, key=key * (stride if case["by"] == "fk" else 1), sum_price=sp, sum_qty=sq, count=count)
        if kind == "planned":
            return [groups, None, None]
        return [groups, *([keep.numel(), keep.numel(), key.numel()] if case["stats"] else [])]
    if kind == "filter":
        col, lit = _ints(_gen(seed), case["n"], 0, DAYS, torch.int32), case["day_lt"]
        return _rows(case, idx=torch.nonzero(getattr(torch, case["op"])(col, lit)).flatten())
    if kind == "pred":
        ok = torch.ones(case["n"], dtype=torch.bool, device=_dev())
        for t, c in zip(case["terms"].split(","), _pred_columns(case, seed)):
            op, v = TERMS[t][2], TERMS[t][3](case["width"])
            c = c.to(torch.float64) if c.is_floating_point() else c
            ok &= (c >= v[0]) & (c <= v[1]) if op == "between" else torch.isin(c, torch.tensor(v, device=_dev(), dtype=c.dtype)) \
                if op == "in" else getattr(torch, op)(c, v[0])
        return _rows(case, idx=torch.nonzero(ok).flatten())
    if kind == "join":
        fact, dim = _tables(case, seed)
        row = torch.nonzero(fact["day"] < case["day_lt"]).flatten()
        at = torch.empty(case["m"], dtype=torch.int64, device=_dev())
        at[(dim["pk"] // case["stride"]).to(torch.int64)] = torch.arange(case["m"], device=_dev())
        j = at[(fact["fk"][row] // case["stride"]).to(torch.int64)]
        cols = [fact["price_cents"][row], fact["qty"][row]]
        if not case["payload"]:
            cols += [fact["day"][row], dim["prio"][j]]
        return _rows(case, row=row, payload=dim["prio"][j] if case["payload"] else j, **{"col%d" % i: c for i, c in enumerate(cols)})
    if kind == "groupby":
        key, price, qty, sel = _groupby_rows(case, seed)
        if sel is not None:
            key, price, qty = key[sel], price[sel], qty[sel]
        own, sp, sq, count = _sums(key // case["spread"], price, qty, case["groups"])
        return _rows(case, key=own * case["spread"], sum_price=sp, sum_qty=sq, count=count)
    if kind == "batch":
        sizes, fo, do, fact, dim = _batch_tables(case, seed)
        got = {k: [] for k in ("key", "sum_price", "sum_qty", "count", "n_groups")}
        for i, (n, m, groups, day_lt) in enumerate(sizes):
            f, d = slice(fo[i], fo[i] + n), slice(do[i], do[i] + m)
            keep = fact["day"][f] < day_lt
            attr = torch.empty(m, dtype=torch.int64, device=_dev())
            attr[dim["pk"][d].to(torch.int64)] = dim["grp"][d].to(torch.int64)
            own = _sums(attr[fact["fk"][f][keep].to(torch.int64)], fact["price_cents"][f][keep], fact["qty"][f][keep], groups)
            for k, v in zip(("key", "sum_price", "sum_qty", "count"), own):
                got[k].append(v)
            got["n_groups"].append(torch.tensor([own[0].numel()], device=_dev()))
        got = {k: torch.cat(v) for k, v in got.items()}
        return {k: v if k == "n_groups" else _padded(v, _size(case)) for k, v in got.items()}
    params, x, t = _network(case, seed)
    p = params.double().requires_grad_()
    cut, layers = 0, []
    for i, o in ((40, 64), (64, 64), (64, 2)):
        layers.append((p[cut:cut + i * o].view(i, o), p[cut + i * o:cut + i * o + o]))
        cut += i * o + o
    h = x.double()
    for k, (w, b) in enumerate(layers):
        h = h @ w + b
        h = torch.relu(h) if k < 2 else h
    loss = (h - t.double()).square().sum() / (2 * case["rows"])
    (grad,) = torch.autograd.grad(loss, p)
    m, v = 0.1 * grad, 0.001 * grad.square()
    new = p.detach() - 1e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return dict(y=h.detach(), loss=loss.detach().reshape(1), grad=grad, params=new, m=m, v=v)
