"""The work a query optimiser has the library do, as cases that can be timed.

A case is a dict of plain values (the sizes of several tables are one
text).  ``listed()`` gives the named ones,
``draw(rng)`` one more of the same ranges, ``prepare(case, seed)`` what a
program holds before the call (resident tables, compiled programs it keeps,
output buffers), ``run(state)`` one pass through the binding's entry points,
``work(case)`` the bytes one pass cannot do without and ``exact(case, seed)``
the same outputs computed with plain torch.

Kinds
  count     SELECT COUNT(*) of one selection (Context.count)
  pushdown  count, limit check and ascending row ids; the selection is
            compiled in the pass, as each query brings its own
  sigma     row ids, then the projected columns at those rows
  star      one key bitmap per dimension, then the semi-join count
  spd       Algorithm 1's decision over the relations of a query
  batch     the counts of many candidate selections, eager or replayed
  serve     a burst of estimate requests answered by a server

Tables
  fact      date i32, qty i8, disc i8, price i64 (log-normal, 5 % NULL),
            s7, s25, s4500 i32 dictionary codes (Zipf)
  uniform3  three i32 columns uniform in [0, 10000)
  mixed     i8, i16, i32 and i64, every one with NULLs
"""
import math
import random

import numpy as np
import torch

from paper_1806_08384_amd import sel

FACT_WIDTH = {"date": 4, "qty": 1, "disc": 1, "price": 8, "s7": 4, "s25": 4, "s4500": 4}
DIM_ROWS = (2556, 30_000, 200_000, 3_200_000)
DIM_KEEP = (2 / 7, 1 / 5, 2 / 25, 2 / 250)
SIX_BYTES = 4 + 1 + 1 + 8 + 1 / 8 + 4 + 4
SPAN = 1 << 25                     # rows generated at a time


def listed():
    return [
        # the smallest call: one count on a dimension-sized table, all latency
        {"name": "count_10k", "kind": "count", "table": "fact", "rows": 10_007, "pred": "six", "window": 365},
        # three range tests on a million rows, count and id list
        {"name": "pushdown_1M", "kind": "pushdown", "table": "uniform3", "rows": 1_000_000, "pred": "range3",
         "window": 0},
        # a list of 1000 prices, too sparse for a bitmap, on an ordinary table
        {"name": "count_inlist_20M", "kind": "count", "table": "fact", "rows": 20_000_003, "pred": "inlist",
         "window": 1000},
        # the count query at full size: six leaves over 300M rows
        {"name": "count_300M", "kind": "count", "table": "fact", "rows": 300_000_000, "pred": "six", "window": 365},
        # the whole push-down step at full size: compile, count, limit, ids
        {"name": "pushdown_300M", "kind": "pushdown", "table": "fact", "rows": 300_000_000, "pred": "six",
         "window": 365},
        # an unselective push-down: half of 60M rows become ids
        {"name": "pushdown_dense_60M", "kind": "pushdown", "table": "fact", "rows": 60_000_000, "pred": "date",
         "window": 1279},
        # sigma(R) with its columns: NULL logic over every width, ids, gather
        {"name": "sigma_mixed_8M", "kind": "sigma", "rows": 8_000_017, "window": 80},
        # star semi-join at full size: four dimensions pushed down, 480M fact rows
        {"name": "star_480M", "kind": "star", "rows": 480_000_000, "fact_pred": False},
        # one query's relations through Algorithm 1
        {"name": "spd_query", "kind": "spd", "rows": "60000000 20000000 2000000 10000", "dims": True},
        # 64 candidate selections over tables of uneven size, counted together
        {"name": "batch_64", "kind": "batch", "rows": "10000 2000000 60000000 300000000", "per_table": 16,
         "replay": False},
        # a kept batch over small tables, replayed
        {"name": "batch_replay_2M", "kind": "batch", "rows": "10000 2000000", "per_table": 12, "replay": True},
        # a burst of requests of 1..12 selections over resident tables of 1M..480M rows
        {"name": "serve_24", "kind": "serve", "rows": "1000000 2000000 60000000 300000000 480000000",
         "requests": 24},
    ]


def _text(sizes):
    return " ".join(str(n) for n in sizes)


def _sizes(case):
    return [int(n) for n in case["rows"].split()]


def draw(rng):
    def rows(lo, hi):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return n if rng.random() < 0.3 else n | 1

    kind = rng.choice(["count", "count", "pushdown", "pushdown", "sigma", "star", "spd", "batch", "batch", "serve"])
    if kind in ("count", "pushdown"):
        pred = rng.choice(["six", "range3", "inlist", "date"])
        window = {"six": rng.randint(1, 2557), "range3": 0, "inlist": rng.choice([10, 100, 1000]),
                  "date": rng.randint(25, 2300)}[pred]
        return {"kind": kind, "table": "uniform3" if pred == "range3" else "fact",
                "rows": rows(1_000, 300_000_000), "pred": pred, "window": window}
    if kind == "sigma":
        return {"kind": kind, "rows": rows(1_000, 60_000_000), "window": rng.randint(3, 240)}
    if kind == "star":
        return {"kind": kind, "rows": rows(10_000, 480_000_000), "fact_pred": rng.random() < 0.5}
    if kind == "spd":
        n = rng.randint(2, 4)
        return {"kind": kind, "rows": _text([rows(2_000, 60_000_000) for _ in range(n)]), "dims": rng.random() < 0.5}
    if kind == "batch":
        n = rng.randint(1, 4)
        return {"kind": kind, "rows": _text([rows(1_000, 100_000_000) for _ in range(n)]),
                "per_table": rng.randint(1, 16), "replay": rng.random() < 0.5}
    sizes = [rows(10_000, 2_000_000), rows(10_000, 2_000_000), rows(1_000_000, 60_000_000),
             rows(1_000_000, 300_000_000), rows(1_000_000, 300_000_000)]
    return {"kind": "serve", "rows": _text(sizes), "requests": rng.randint(1, 24)}


# ------------------------------------------------------------------ inputs --

class Column:
    def __init__(self, ty, data, null=None, card=0):
        self.type, self.data, self.null, self.card = ty, data, null, card
        self.valid = None if null is None else pack_bits(~null)


def pack_bits(b):
    """uint32 words (as int32) with bit i % 32 of word i / 32 = b[i]."""
    n = b.numel()
    out = torch.empty((n + 31) // 32, dtype=torch.int32, device=b.device)
    w = torch.arange(32, device=b.device, dtype=torch.int64)
    for lo in range(0, n, SPAN):
        part = b[lo: lo + SPAN]
        pad = -part.numel() % 32
        if pad:
            part = torch.cat([part, torch.zeros(pad, dtype=torch.bool, device=b.device)])
        words = (part.view(-1, 32).to(torch.int64) << w).sum(1)
        out[lo // 32: lo // 32 + words.numel()] = torch.where(words >= 1 << 31, words - (1 << 32), words).int()
    return out


def _spans(n):
    return [(lo, min(n, lo + SPAN)) for lo in range(0, n, SPAN)]


def _uniform(g, n, lo, hi, dtype):
    out = torch.empty(n, dtype=dtype, device="cuda")
    for a, b in _spans(n):
        out[a:b] = torch.randint(lo, hi + 1, (b - a,), generator=g, device="cuda", dtype=torch.int32)
    return out


def _zipf(g, n, card):
    pmf = torch.arange(1, card + 1, dtype=torch.float64) ** -1.1
    cdf = (pmf / pmf.sum()).cumsum(0).float().cuda()
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    for a, b in _spans(n):
        u = torch.rand(b - a, generator=g, device="cuda")
        out[a:b] = torch.bucketize(u, cdf, out_int32=True).clamp_(max=card - 1)
    return out


def _nulls(g, n, rate):
    out = torch.empty(n, dtype=torch.bool, device="cuda")
    for a, b in _spans(n):
        out[a:b] = torch.rand(b - a, generator=g, device="cuda") < rate
    return out


def fact_table(g, n):
    price = torch.empty(n, dtype=torch.int64, device="cuda")
    for a, b in _spans(n):
        price[a:b] = torch.exp(10.0 + torch.randn(b - a, generator=g, device="cuda")).round_().long()
    null = _nulls(g, n, 0.05)
    for a, b in _spans(n):
        price[a:b].masked_fill_(null[a:b], 1_000_000)
    return [Column("i32", _uniform(g, n, 0, 2556, torch.int32)), Column("i8", _uniform(g, n, 1, 50, torch.int8)),
            Column("i8", _uniform(g, n, 0, 10, torch.int8)), Column("i64", price, null),
            Column("i32", _zipf(g, n, 7), card=7), Column("i32", _zipf(g, n, 25), card=25),
            Column("i32", _zipf(g, n, 4500), card=4500)]


def uniform3_table(g, n):
    return [Column("i32", _uniform(g, n, 0, 9999, torch.int32)) for _ in range(3)]


def mixed_table(g, n):
    big = _uniform(g, n, -1_000_000, 1_000_000, torch.int64)
    return [Column("i8", _uniform(g, n, -128, 127, torch.int8), _nulls(g, n, 0.1)),
            Column("i16", _uniform(g, n, -3000, 3000, torch.int16), _nulls(g, n, 0.2)),
            Column("i32", _uniform(g, n, 0, 99_999, torch.int32), _nulls(g, n, 0.05)),
            Column("i64", big.mul_(100_003), _nulls(g, n, 0.1))]


def star_table(g, n, dims):
    cols = [Column("i32", _uniform(g, n, 0, d - 1, torch.int32)) for d in dims]
    return cols + [Column("i32", _uniform(g, n, 0, 99, torch.int32))]


def dim_table(g, n, card):
    return [Column("i32", torch.arange(n, dtype=torch.int32, device="cuda")),
            Column("i32", _uniform(g, n, 0, card - 1, torch.int32), card=card)]


def dim_tables(g):
    cards = (7, 5, 25, 250)
    tabs = [dim_table(g, n, c) for n, c in zip(DIM_ROWS, cards)]
    preds = [("in", 1, (1, 2)), ("cmp", 1, "=", 2), ("or", ("cmp", 1, "=", 3), ("cmp", 1, "=", 7)),
             ("in", 1, (17, 101))]
    return tabs, preds


# --------------------------------------------------------------- selections --

def _code_words(codes, nbits):
    words = [0] * ((nbits + 31) // 32)
    for c in codes:
        words[c // 32] |= 1 << (c % 32)
    return words


def six_leaves(r, window):
    lo = r.randint(0, 2557 - window)
    like = [c for c in range(4500) if r.random() < 0.125]
    return ("and", ("between", 0, lo, lo + window - 1), ("or", ("cmp", 1, "<", 25), ("between", 2, 5, 7)),
            ("or", ("cmp", 3, ">=", 20_000), ("in", 5, tuple(range(0, 20, 2)))),
            ("codeset", 6, 4500, _code_words(like, 4500)))


def selection(case, r, cols):
    w = case["window"]
    if case["pred"] == "six":
        return six_leaves(r, w)
    if case["pred"] == "date":
        lo = r.randint(0, 2557 - w)
        return ("between", 0, lo, lo + w - 1)
    if case["pred"] == "inlist":
        data = cols[3].data
        at = torch.tensor([r.randrange(data.numel()) for _ in range(w // 2)], device="cuda")
        absent = [r.randint(10 ** 7, 10 ** 8) for _ in range(w - w // 2)]
        return ("in", 3, tuple(data[at].tolist() + absent))
    a, b, c = r.randint(2000, 4000), r.randint(0, 7000), r.randint(6000, 8000)
    return ("and", ("cmp", 0, "<", a), ("between", 1, b, b + 2999), ("cmp", 2, ">=", c))


def mixed_selection(r, window):
    lo = r.randint(-128, 127 - window)
    return ("and", ("between", 0, lo, lo + window - 1), ("or", ("cmp", 1, ">", 0), ("isnull", 2)),
            ("not", ("and", ("cmp", 2, "<", 20_000), ("cmp", 3, "<", 0))),
            ("or", ("notnull", 3), ("isunknown", ("cmp", 1, "=", 7))))


def _upper_quantile(q):
    """z with P(Z >= z) = q for a standard normal."""
    lo, hi = -8.0, 8.0
    for _ in range(60):
        mid = (lo + hi) / 2
        if 0.5 * math.erfc(mid / math.sqrt(2)) > q:
            lo = mid
        else:
            hi = mid
    return lo


def candidate_leaf(r, q):
    """A leaf over the fact columns that about a fraction q of the rows meet."""
    q = min(max(q, 1e-7), 1.0)
    col = r.choice([0, 1, 2, 3, 5, 6])
    if col == 0:
        w = max(1, round(q * 2557))
        a = r.randint(0, 2557 - w)
        return ("between", 0, a, a + w - 1)
    if col == 1:
        w = max(1, round(q * 50))
        return ("cmp", 1, "<", 1 + w) if r.random() < 0.5 else ("cmp", 1, ">", 50 - w)
    if col == 2:
        w = max(1, round(q * 11))
        a = r.randint(0, 11 - w)
        return ("between", 2, a, a + w - 1)
    if col == 3:
        return ("cmp", 3, ">=", round(math.exp(10 + _upper_quantile(q))))
    card = 25 if col == 5 else 4500
    total = sum((c + 1) ** -1.1 for c in range(card))
    codes, mass = [], 0.0
    for c in r.sample(range(card), card):
        p = (c + 1) ** -1.1 / total
        if mass >= q:
            break
        if mass + p > 1.5 * q and codes:
            continue
        codes.append(c)
        mass += p
    return ("in", 5, tuple(sorted(codes))) if col == 5 else ("codeset", 6, 4500, _code_words(codes, 4500))


def candidate(r):
    """A selection of 2..8 leaves, an AND of leaves and two-leaf ORs, with a
    target selectivity log-uniform in [1e-5, 0.9]."""
    leaves = r.randint(2, 8)
    pairs = r.randint(0, leaves // 2)
    m = leaves - pairs
    q = math.exp(r.uniform(math.log(1e-5), math.log(0.9))) ** (1 / m)
    half = 1 - math.sqrt(max(0.0, 1 - q))
    parts = [("or", candidate_leaf(r, half), candidate_leaf(r, half)) if k < pairs else candidate_leaf(r, q)
             for k in range(m)]
    return parts[0] if m == 1 else ("and", *parts)


def uniform3_candidate(r):
    k = r.randint(1, 3)
    leaves = []
    for c in r.sample(range(3), k):
        w = max(1, round(10_000 * math.exp(r.uniform(math.log(1e-3), math.log(0.9)))))
        a = r.randint(0, 10_000 - w)
        leaves.append(("between", c, a, a + w - 1))
    return leaves[0] if k == 1 else ("and", *leaves)


# ------------------------------------------------------------------- inputs --

def _generators(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g, random.Random(seed)


def inputs(case, seed):
    """Tables (lists of columns) and selections of a case."""
    g, r = _generators(seed)
    kind = case["kind"]
    if kind in ("count", "pushdown"):
        cols = (fact_table if case["table"] == "fact" else uniform3_table)(g, case["rows"])
        return {"tables": [cols], "trees": [(0, selection(case, r, cols))]}
    if kind == "sigma":
        return {"tables": [mixed_table(g, case["rows"])], "trees": [(0, mixed_selection(r, case["window"]))]}
    if kind == "star":
        dims, preds = dim_tables(g)
        fact = star_table(g, case["rows"], DIM_ROWS)
        return {"tables": dims + [fact], "trees": [(d, p) for d, p in enumerate(preds)],
                "fact_pred": ("cmp", 4, "<", 50) if case["fact_pred"] else None}
    if kind == "spd":
        tabs = [fact_table(g, n) for n in _sizes(case)]
        trees = [(k, six_leaves(r, r.randint(100, 1200))) for k in range(len(tabs))]
        if case["dims"]:
            dims, preds = dim_tables(g)
            trees += [(len(tabs) + d, p) for d, p in enumerate(preds)]
            tabs += dims
        return {"tables": tabs, "trees": trees}
    if kind == "batch":
        tabs = [fact_table(g, n) for n in _sizes(case)]
        return {"tables": tabs, "trees": [(k, candidate(r)) for k in range(len(tabs)) for _ in range(case["per_table"])]}
    # serve: pools of selections per table, and the requests drawn from them
    n0, n1, n2, n3, n4 = _sizes(case)
    tabs = [uniform3_table(g, n0), fact_table(g, n1), fact_table(g, n2), fact_table(g, n3),
            star_table(g, n4, DIM_ROWS)]
    trees = [(0, uniform3_candidate(r)) for _ in range(32)]
    trees += [(k, candidate(r)) for k in (1, 2, 3) for _ in range(32)]
    stars = []
    for _ in range(16):
        stars.append([_nulls(g, n, math.exp(r.uniform(math.log(0.02), math.log(0.6)))) for n in DIM_ROWS])
    # how many selections a request has, and which ask for row ids, on which
    # table, is the case's; the selections are the seed's
    shape, requests = random.Random(case["requests"]), []
    for _ in range(case["requests"]):
        items = []
        for _ in range(shape.randint(1, 12)):
            t = r.randrange(5)
            items.append(len(trees) + r.randrange(16) if t == 4 else 32 * t + r.randrange(32))
        requests.append((items, 32 * shape.randrange(4) + r.randrange(32) if shape.random() < 0.1 else None))
    return {"tables": tabs, "trees": trees, "stars": stars, "requests": requests}


# ---------------------------------------------------------------- the passes --

class State:
    pass


def _device_table(ctx, cols):
    keep = [c.data for c in cols] + [c.valid for c in cols if c.valid is not None]
    return ctx.table(cols[0].data.numel(),
                     [(c.type, c.card, c.data.data_ptr(), None if c.valid is None else c.valid.data_ptr())
                      for c in cols], keep)


def _ids(n, ids=None):
    """A buffer for n row ids, holding `ids` at its front."""
    out = torch.zeros(max(1, n), dtype=torch.int32, device="cuda")
    if ids is not None:
        out[:ids.numel()] = ids
    return out


def prepare(case, seed):
    s = State()
    inp = inputs(case, seed)
    s.kind = case["kind"]
    s.ctx = ctx = sel.Context(0)
    s.tables = [_device_table(ctx, t) for t in inp["tables"]]
    s.trees = inp["trees"]
    if s.kind != "pushdown":
        s.progs = [ctx.program(s.tables[t], tree) for t, tree in s.trees]
    if s.kind in ("pushdown", "sigma"):
        s.ids = _ids(s.tables[0].nrows)
    if s.kind == "sigma":
        cols = inp["tables"][0]
        n = s.tables[0].nrows
        s.values = [torch.zeros(n, dtype=c.data.dtype, device="cuda") for c in cols]
        s.valid = [torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda") for _ in cols]
    if s.kind == "star":
        s.bitmaps = [torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda") for n in DIM_ROWS]
        s.fact_pred = ctx.program(s.tables[4], inp["fact_pred"]) if inp["fact_pred"] else None
    if s.kind == "spd":
        s.relations = [(t, p, _ids(t.nrows // 20)) for t, p in zip(s.tables, s.progs)]
    if s.kind == "batch":
        s.pairs = [(s.tables[t], p) for (t, _), p in zip(s.trees, s.progs)]
        s.batch = ctx.batch(s.pairs) if case["replay"] else None
    if s.kind == "serve":
        s.bitmaps = [[pack_bits(b) for b in star] for star in inp["stars"]]
        s.progs += [ctx.star_program(s.tables[4], range(4), b, DIM_ROWS) for b in s.bitmaps]
        where = [t for t, _ in s.trees] + [4] * len(s.bitmaps)
        s.requests = []
        for items, pd in inp["requests"]:
            job = None
            if pd is not None:
                t = s.tables[where[pd]]
                limit = sel.max_rows(t.nrows, 0.05)
                job = (t, s.progs[pd], limit, _ids(limit))
            s.requests.append(([(s.tables[where[k]], s.progs[k]) for k in items], job))
        s.server = ctx.server()
    torch.cuda.synchronize()
    return s


def run(s):
    ctx = s.ctx
    if s.kind == "count":
        return ctx.count(s.tables[0], s.progs[0])
    if s.kind == "pushdown":
        prog = ctx.program(s.tables[0], s.trees[0][1])
        status, count = ctx.pushdown_rowids(s.tables[0], prog, sel.UINT64_MAX, s.ids)
        prog.destroy()
        return {"status": status, "count": count, "ids": s.ids}
    if s.kind == "sigma":
        status, count = ctx.pushdown_rowids(s.tables[0], s.progs[0], sel.UINT64_MAX, s.ids)
        ctx.gather(s.tables[0], s.ids, count, range(4), s.values, s.valid)
        return {"status": status, "count": count, "ids": s.ids, "values": s.values, "valid": s.valid}
    if s.kind == "star":
        sizes = [ctx.pushdown_keybitmap(s.tables[d], 0, 0, s.progs[d], s.bitmaps[d], DIM_ROWS[d]) for d in range(4)]
        count = ctx.star_count(s.tables[4], range(4), s.bitmaps, DIM_ROWS, s.fact_pred)
        return {"sizes": sizes, "bitmaps": s.bitmaps, "count": count}
    if s.kind == "spd":
        res = ctx.select_pushdown(s.relations)
        return [{"decision": sel.SPD_DECISIONS.index(x["decision"]), "status": x["status"], "count": x["count"],
                 "ids": rel[2]} for x, rel in zip(res, s.relations)]
    if s.kind == "batch":
        return s.batch.run() if s.batch else ctx.count_batch(s.pairs)
    tickets = [s.server.submit(items, job) for items, job in s.requests]
    done = [s.server.wait(ticket) for ticket in tickets]
    return {"counts": np.array([c for counts, _, _, _ in done for c in counts]),
            "status": np.array([status for _, status, _, _ in done]),
            "found": np.array([found for _, _, found, _ in done]),
            "ids": [job[3] for _, job in s.requests if job is not None]}


# ---------------------------------------------------------------------- work --

def _columns_of(tree):
    if tree[0] in ("and", "or", "not", "isunknown"):
        return set().union(*[_columns_of(t) for t in tree[1:]])
    return {tree[1]}


def work(case):
    kind = case["kind"]
    if kind in ("count", "pushdown"):
        n = case["rows"]
        b = n * {"six": SIX_BYTES, "range3": 12, "inlist": 8.125, "date": 4}[case["pred"]]
        if kind == "pushdown":
            keep = {"six": 0.038 * case["window"] / 2557, "range3": 0.027, "inlist": 0.03,
                    "date": case["window"] / 2557}[case["pred"]]
            b += 4 * n * keep
        return {"bytes": int(b), "flops": 0}
    if kind == "sigma":
        n = case["rows"]
        ids = 0.33 * n * case["window"] / 256
        return {"bytes": int(n * 15.5 + ids * 4 + ids * (15 + 0.5) * 2), "flops": 0}
    if kind == "star":
        dims = sum(n * 8 + n / 8 for n in DIM_ROWS)
        return {"bytes": int(case["rows"] * (20 if case["fact_pred"] else 16) + dims), "flops": 0}
    if kind == "spd":
        sizes = sorted(_sizes(case), reverse=True)
        b = 0.0
        if case["dims"]:
            sized = sorted(sizes + list(DIM_ROWS), reverse=True)
            b += sum(n * 4 for n in DIM_ROWS if n != sized[0])
            sizes = [n for n in sizes if n != sized[0]]
        else:
            sizes = sizes[1:]
        return {"bytes": int(b + sum(n * SIX_BYTES for n in sizes if n > 1000)), "flops": 0}
    if kind == "batch":
        return {"bytes": int(sum(_sizes(case)) * SIX_BYTES), "flops": 0}
    n0, n1, n2, n3, n4 = _sizes(case)
    return {"bytes": int(n0 * 12 + (n1 + n2 + n3) * SIX_BYTES + n4 * 16), "flops": 0}


# --------------------------------------------------------------------- exact --

def truth(tree, cols, a, b):
    """(TRUE, FALSE) masks of rows [a, b) in three-valued logic."""
    k = tree[0]
    if k in ("and", "or"):
        t, f = truth(tree[1], cols, a, b)
        for p in tree[2:]:
            u, v = truth(p, cols, a, b)
            t, f = (t & u, f | v) if k == "and" else (t | u, f & v)
        return t, f
    if k == "not":
        t, f = truth(tree[1], cols, a, b)
        return f, t
    if k == "isunknown":
        t, f = truth(tree[1], cols, a, b)
        return ~(t | f), t | f
    c = cols[tree[1]]
    null = torch.zeros(b - a, dtype=torch.bool, device="cuda") if c.null is None else c.null[a:b]
    if k == "isnull":
        return null, ~null
    if k == "notnull":
        return ~null, null
    x = c.data[a:b]
    if k == "cmp":
        v = tree[3]
        p = {"=": x == v, "<": x < v, ">": x > v, ">=": x >= v}[tree[2]]
    elif k == "between":
        p = (x >= tree[2]) & (x <= tree[3])
    elif k == "in":
        p = torch.isin(x, torch.tensor(tree[2], dtype=x.dtype, device="cuda"))
    else:  # a code set; the codes lie inside it
        words = torch.tensor(tree[3], dtype=torch.int64, device="cuda")
        bits = ((words.view(-1, 1) >> torch.arange(32, device="cuda")) & 1).bool().view(-1)
        p = bits[x.long()]
    return p & ~null, ~p & ~null


def _count(tree, cols):
    n = cols[0].data.numel()
    return sum(int(truth(tree, cols, a, b)[0].sum()) for a, b in _spans(n))


def _rows(tree, cols):
    n = cols[0].data.numel()
    parts = [truth(tree, cols, a, b)[0].nonzero().view(-1) + a for a, b in _spans(n)]
    return torch.cat(parts).int() if parts else torch.zeros(0, dtype=torch.int32, device="cuda")


def _star(fact, members, pred=None):
    total = 0
    for a, b in _spans(fact[0].data.numel()):
        m = torch.ones(b - a, dtype=torch.bool, device="cuda") if pred is None else truth(pred, fact, a, b)[0]
        for c, keep in zip(fact, members):
            m &= keep[c.data[a:b].long()]
        total += int(m.sum())
    return total


def exact(case, seed):
    inp = inputs(case, seed)
    tabs, trees, kind = inp["tables"], inp["trees"], case["kind"]
    if kind == "count":
        return _count(trees[0][1], tabs[0])
    if kind == "pushdown":
        ids = _rows(trees[0][1], tabs[0])
        return {"status": 0, "count": ids.numel(), "ids": _ids(case["rows"], ids)}
    if kind == "sigma":
        n, ids = case["rows"], _rows(trees[0][1], tabs[0])
        at = ids.long()
        values = [torch.zeros_like(c.data) for c in tabs[0]]
        valid = [torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda") for _ in tabs[0]]
        for c, v, w in zip(tabs[0], values, valid):
            v[:at.numel()] = c.data[at]
            w[:(at.numel() + 31) // 32] = pack_bits(~c.null[at])
        return {"status": 0, "count": ids.numel(), "ids": _ids(n, ids), "values": values, "valid": valid}
    if kind == "star":
        keep = []
        for d, p in trees:
            n = tabs[d][0].data.numel()
            keep.append(truth(p, tabs[d], 0, n)[0])
        return {"sizes": [(0, int(k.sum())) for k in keep], "bitmaps": [pack_bits(k) for k in keep],
                "count": _star(tabs[4], keep, inp["fact_pred"])}
    if kind == "spd":
        sizes = [t[0].data.numel() for t in tabs]
        probe = sizes.index(max(sizes))
        out = []
        for k, (_, tree) in enumerate(trees):
            cap = sizes[k] // 20
            if k == probe or sizes[k] <= 1000:
                out.append({"decision": 3 if sizes[k] <= 1000 else 2, "status": 0, "count": 0, "ids": _ids(cap)})
                continue
            ids = _rows(tree, tabs[k])
            over = ids.numel() > sizes[k] * 0.05
            out.append({"decision": int(over), "status": int(over), "count": ids.numel(),
                        "ids": _ids(cap, None if over else ids)})
        return out
    if kind == "batch":
        return [_count(tree, tabs[t]) for t, tree in trees]
    counts = {}

    def count_of(k):
        if k not in counts:
            counts[k] = (_star(tabs[4], inp["stars"][k - len(trees)]) if k >= len(trees)
                         else _count(trees[k][1], tabs[trees[k][0]]))
        return counts[k]

    status, found, ids = [], [], []
    for _, pd in inp["requests"]:
        status.append(0)
        found.append(0)
        if pd is not None:
            t, tree = trees[pd]
            limit = int(tabs[t][0].data.numel() * 0.05)
            found[-1] = count_of(pd)
            status[-1] = int(found[-1] > limit)
            ids.append(_ids(limit, None if status[-1] else _rows(tree, tabs[t])))
    return {"counts": np.array([count_of(k) for items, _ in inp["requests"] for k in items]),
            "status": np.array(status), "found": np.array(found), "ids": ids}
