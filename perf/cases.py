"""Workloads of the relational operators, from the smallest query to the largest.

listed() names the representative ones, draw() gives more of the same ranges;
prepare() builds the device tables and the plan a program keeps, run() is one
execution of the query or operator on them, work() the bytes and operations it
cannot do without and exact() the same answer from plain torch.

Every table is drawn on the GPU with a generator seeded from the seed alone.
All results are integers (exact modulo 2^64), so they do not depend on the
order of any reduction.  Plans return their own result buffers; a buffer is
sized for the plan's capacity and cleared once when the plan is built, so the
entries past the number of groups found are zeros.
"""
from __future__ import annotations

import math

import torch

import paper_2209_04579_amd as tqp
from paper_2209_04579_amd.batch import BatchStarQuery
from paper_2209_04579_amd.pipeline import PredictQuery, Q14Query, Q6Scan, StarQuery, StarQuery3

DAYS = 2557                                    # seven years of day numbers
NS_PER_DAY = 86_400 * 1_000_000_000
DAY0 = 8035                                    # 1992-01-01 after the epoch
PART_WORDS = (b"ECONOMY", b"LARGE", b"MEDIUM", b"PROMO", b"SMALL", b"STANDARD")


def listed():
    return [
        # the smallest query of a batch of uneven ones, run alone: every operator
        # works on a few tiles, so launches and latencies are what counts
        {"name": "star-10k", "kind": "star", "mode": "q1", "n": 10_007, "nd": 500, "zipf": 0.0,
         "cats": 25, "cut": 1278},
        # an interactive star query: filter, sort, join, group by category
        {"name": "star-1m", "kind": "star", "mode": "q1", "n": 1_000_000, "nd": 10_000, "zipf": 0.0,
         "cats": 25, "cut": 1278},
        # the skewed star over a large table, grouped by a packed low-cardinality
        # key and by the foreign key (every run of the sorted join output)
        {"name": "star-skewed-60m", "kind": "star", "mode": "q2", "n": 60_000_000, "nd": 2_000_000,
         "zipf": 1.0, "cats": 25, "cut": 1278},
        # three filtered dimensions in front of the largest fact table: the
        # semi-join scan, then sort-merge joins on the rows that survive
        {"name": "star3-300m", "kind": "star3", "n": 300_000_000, "nd1": 1_000_000,
         "nd2": 100_000, "nd3": 25, "cut": 20},
        # a scan with predicates of three types feeding one SUM and COUNT
        {"name": "q6-60m", "kind": "q6", "n": 60_000_000, "days": 365},
        # a selective filter (one month of seven years), string LIKE, join and CASE
        {"name": "q14-60m", "kind": "q14", "n": 60_000_000, "nd": 2_000_000, "width": 24, "days": 30},
        # PREDICT inside a query: filter, MLP over the kept rows, group by rating
        {"name": "predict-20m", "kind": "predict", "n": 20_000_000, "nfeat": 8, "hidden": 16,
         "year_min": 2016},
        # many uneven queries in one arena, replayed as one captured graph
        {"name": "batch-64", "kind": "batch", "k": 64, "lo": 10_000, "hi": 4_000_000, "cut": 1278},
        # a large-large join of clustered, lognormal and Zipf int64 keys: train the
        # learned CDF, partition-sort both sides, merge into ranges
        {"name": "learned-50m", "kind": "learned", "nl": 50_000_000, "nr": 12_500_000},
        # ORDER BY a 64-bit key of unknown range, carrying payload of mixed types
        {"name": "sort-10m", "kind": "sort", "n": 10_000_019, "bits": 64, "dtype": "int64",
         "rows": True, "pay8": 1, "pay64": 1},
        # GROUP BY a high-cardinality key that is not sorted, three aggregates
        {"name": "groupby-5m", "kind": "groupby", "n": 5_000_011, "span": 1_000_003,
         "dtype": "int64", "zipf": 0.0},
        # an unsorted many-to-many equi-join with its key written
        {"name": "join-1m", "kind": "join", "nl": 1_500_007, "nr": 400_009, "keys": 200_003,
         "dtype": "int32"},
    ]


def _log(rng, lo, hi):
    """An integer log-uniform on [lo, hi], as odd as it falls."""
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["star", "star", "star3", "q6", "q14", "predict", "batch", "learned", "sort",
                       "sort", "groupby", "join"])
    if kind == "star":
        n = _log(rng, 10_000, 60_000_000)
        nd = max(25, int(n / rng.uniform(20, 100)))
        return {"kind": kind, "mode": rng.choice(["q1", "q2"]), "n": n, "nd": nd,
                "zipf": round(rng.uniform(0, 1.5), 2), "cats": min(_log(rng, 2, 500), nd),
                "cut": rng.randrange(60, DAYS + 1)}
    if kind == "star3":
        return {"kind": kind, "n": _log(rng, 100_000, 300_000_000), "nd1": _log(rng, 10_000, 1_000_000),
                "nd2": _log(rng, 1_000, 100_000), "nd3": rng.randrange(5, 40),
                "cut": rng.randrange(8, 60)}
    if kind == "q6":
        return {"kind": kind, "n": _log(rng, 10_000, 60_000_000), "days": rng.randrange(7, 1500)}
    if kind == "q14":
        n = _log(rng, 50_000, 60_000_000)
        return {"kind": kind, "n": n, "nd": max(100, int(n / rng.uniform(15, 60))),
                "width": rng.randrange(12, 33), "days": rng.randrange(7, 1200)}
    if kind == "predict":
        return {"kind": kind, "n": _log(rng, 10_000, 20_000_000), "nfeat": rng.randrange(3, 17),
                "hidden": rng.randrange(4, 33), "year_min": rng.randrange(2010, 2024)}
    if kind == "batch":
        return {"kind": kind, "k": rng.randrange(4, 65), "lo": 10_000,
                "hi": _log(rng, 20_000, 4_000_000), "cut": rng.randrange(200, DAYS + 1)}
    if kind == "learned":
        n = _log(rng, 500_000, 50_000_000)
        return {"kind": kind, "nl": n, "nr": int(n / rng.uniform(1, 8))}
    dtype = rng.choice(["int32", "int64"])
    if kind == "sort":
        return {"kind": kind, "n": _log(rng, 1_000, 10_000_000), "dtype": dtype,
                "bits": rng.randrange(1, 33 if dtype == "int32" else 65),
                "rows": rng.random() < 0.7, "pay8": rng.randrange(2), "pay64": rng.randrange(3)}
    if kind == "groupby":
        n = _log(rng, 1_000, 5_000_000)
        return {"kind": kind, "n": n, "span": _log(rng, 3, 2 * n), "dtype": dtype,
                "zipf": round(rng.choice([0.0, rng.uniform(0.5, 1.4)]), 2)}
    nl = _log(rng, 1_000, 1_500_000)
    return {"kind": kind, "nl": nl, "nr": max(1, int(nl / rng.uniform(1, 20))),
            "keys": max(2, int(nl / rng.uniform(1, 12))), "dtype": dtype}


# ---------------------------------------------------------------- tables ----

class _Draw:
    """Seeded columns on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def ints(self, n, lo, hi, dtype=torch.int64):
        return torch.randint(lo, hi, (n,), generator=self.g, device="cuda", dtype=dtype)

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device="cuda").to(torch.int32)

    def unit(self, n):
        return torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64)

    def cats(self, n, cats):
        """int32 categories below cats, the first and the last among them."""
        c = self.ints(n, 0, cats, torch.int32)
        c[0], c[-1] = 0, cats - 1
        return c

    def ranks(self, n, size, s):
        """0-based bounded Zipf(s) ranks below size (s = 0: uniform)."""
        if s == 0:
            return self.ints(n, 0, size)
        w = torch.arange(1, size + 1, device="cuda", dtype=torch.float64) ** -s
        cdf = torch.cumsum(w, 0)
        return torch.searchsorted(cdf / cdf[-1], self.unit(n)).clamp_(max=size - 1)

    def ship(self, n):
        """int64 epoch nanoseconds over seven years, to the second."""
        return ((self.ints(n, 0, DAYS) + DAY0) * 86_400 + self.ints(n, 0, 86_400)) * 1_000_000_000

    def mixed_keys(self, n, centres):
        """int64 keys: a third lognormal, a third in dense clusters, a third Zipf scattered."""
        comp = self.ints(n, 0, 3)
        z = torch.randn(n, generator=self.g, device="cuda", dtype=torch.float64)
        ln = torch.exp(30.0 + 2.0 * z).clamp_(max=2.0 ** 62).to(torch.int64)
        cl = centres[self.ints(n, 0, len(centres))] + self.ints(n, 0, 1 << 20)
        zs = ((self.ranks(n, 1_000_000, 1.2) + 1) * 0x2545F4914F6CDD1D) & ((1 << 62) - 1)
        return torch.where(comp == 0, ln, torch.where(comp == 1, cl, zs))


def _dtype(name):
    return {"int32": torch.int32, "int64": torch.int64}[name]


def _tables(c, seed):
    d, k = _Draw(seed), c["kind"]
    if k == "star":
        n, nd = c["n"], c["nd"]
        fact = {"fk": d.ranks(n, nd, c["zipf"]).to(torch.int32), "qty": d.ints(n, 1, 5001),
                "day": d.ints(n, 0, DAYS, torch.int32)}
        if c["mode"] == "q2":
            fact["price"] = d.ints(n, 100, 10_000_001)
            fact["flag"] = d.ints(n, 0, 3, torch.int8)
        return {"fact": fact, "dim": {"pk": d.perm(nd), "cat": d.cats(nd, c["cats"])}}
    if k == "star3":
        n = c["n"]
        t = {"fact": {"fk%d" % i: d.ints(n, 0, c["nd%d" % i], torch.int32) for i in (1, 2, 3)}}
        t["fact"].update(qty=d.ints(n, 1, 5001), price=d.ints(n, 100, 10_000_001))
        for i, cats in ((1, 25), (2, 5), (3, 1)):
            nd = c["nd%d" % i]
            t["d%d" % i] = {"pk": d.perm(nd), "cat": d.cats(nd, cats),
                            "attr": d.ints(nd, 0, 100, torch.int32)}
        # the smallest dimension's filter keeps the same share of it for every seed
        t["d3"]["attr"] = (t["d3"]["pk"] * 100).div(c["nd3"], rounding_mode="floor").to(torch.int32)
        return t
    if k == "q6":
        n = c["n"]
        return {"items": {"ship": d.ship(n), "discount": d.ints(n, 0, 11, torch.int8),
                          "quantity": d.ints(n, 1, 51, torch.int32),
                          "price": d.ints(n, 90_000, 10_494_951)}}
    if k == "q14":
        n, nd = c["n"], c["nd"]
        items = {"ship": d.ship(n), "partkey": d.ints(n, 0, nd, torch.int32),
                 "price": d.ints(n, 90_000, 10_494_951), "discount": d.ints(n, 0, 11, torch.int8)}
        names = torch.zeros(len(PART_WORDS), c["width"], dtype=torch.uint8)
        for i, w in enumerate(PART_WORDS):
            names[i, :len(w)] = torch.tensor(list(w), dtype=torch.uint8)
        kind = d.ints(nd, 0, len(PART_WORDS))
        text = names.cuda()[kind]
        text[:, 9:11] = d.ints(2 * nd, 65, 91, torch.uint8).view(nd, 2)
        return {"items": items, "part": {"pk": d.perm(nd), "type": text.contiguous()}}
    if k == "predict":
        n, f, h = c["n"], c["nfeat"], c["hidden"]
        rating = d.ints(n, 1, 6, torch.int8)
        rev = {"rating": rating, "year": d.ints(n, 2010, 2024, torch.int32)}
        for j in range(f):
            rev["f%d" % j] = (rating.to(torch.int32) - 3) * (4 * (j % 4 - 1)) + d.ints(n, -8, 9, torch.int32)
        parts = [((2 * d.unit(m) - 1) / math.sqrt(fan)).to(torch.float32)
                 for m, fan in ((h * f, f), (h, f), (2 * h, h), (2, h))]
        return {"reviews": rev, "model": torch.cat(parts)}
    if k == "batch":
        # sizes spread evenly over the logarithm of the range, the same for every
        # seed; skew and group count vary between the queries
        out = []
        for i in range(c["k"]):
            u = (i + 0.5) / c["k"]
            n = int(c["lo"] * (c["hi"] / c["lo"]) ** u)
            nd = max(1, n // 20)
            out.append({"fact": {"fk": d.ranks(n, nd, 1.5 * ((i * 7) % 16) / 16).to(torch.int32),
                                 "qty": d.ints(n, 1, 5001), "day": d.ints(n, 0, DAYS, torch.int32)},
                        "dim": {"pk": d.perm(nd), "cat": d.cats(nd, min(nd, 25 << (i % 8)))}})
        return {"instances": out}
    if k == "learned":
        centres = d.ints(64, 0, (1 << 62) - (1 << 20))
        return {"left": d.mixed_keys(c["nl"], centres), "right": d.mixed_keys(c["nr"], centres)}
    dt = _dtype(c["dtype"])
    if k == "sort":
        n, bits = c["n"], c["bits"]
        key = d.ints(n, -(1 << 63), (1 << 63) - 1)
        key = key if bits == 64 else ((key >> 1) & ((1 << min(bits, 63)) - 1)) - (1 << (bits - 1))
        return {"key": key.to(dt), "pay": [d.ints(n, -128, 128, torch.int8) for _ in range(c["pay8"])]
                + [d.ints(n, -(1 << 40), 1 << 40) for _ in range(c["pay64"])]}
    if k == "groupby":
        n = c["n"]
        return {"key": (d.ranks(n, c["span"], c["zipf"]) - c["span"] // 3).to(dt),
                "vals": [d.ints(n, -(1 << 40), 1 << 40), d.ints(n, 0, 11, torch.int8)]}
    return {"left": d.ints(c["nl"], 0, c["keys"]).to(dt) * 3, "right": d.ints(c["nr"], 0, c["keys"]).to(dt) * 3}


# --------------------------------------------------------- plans and runs ----

def _ship_range(days):
    lo = 9374 - min(days, 1200)
    return lo * NS_PER_DAY, (lo + days) * NS_PER_DAY


def _cleared(*buffers):
    for b in buffers:
        b.zero_()
    return list(buffers)


def prepare(case, seed):
    c, k = case, case["kind"]
    t = _tables(c, seed)
    if k == "star":
        q = StarQuery(t["fact"], t["dim"], c["cut"], mode=c["mode"])
        out = [q.cnt, q.npairs, q.ga_ng, q.ga_key, *q.ga_out]
        if c["mode"] == "q2":
            out += [q.gb_ng, q.gb_key, *q.gb_out]
        return {"kind": k, "q": q, "out": _cleared(*out)}
    if k == "star3":
        q = StarQuery3(t["fact"], t["d1"], t["d2"], t["d3"], c["cut"])
        return {"kind": k, "q": q, "out": _cleared(q.cnt[2], q.g_ng, q.g_key, *q.g_out)}
    if k == "q6":
        lo, hi = _ship_range(c["days"])
        q = Q6Scan(t["items"], {"ship_lo": lo, "ship_hi": hi, "disc_lo": 5, "disc_hi": 7, "qty_cut": 24})
        return {"kind": k, "q": q, "out": _cleared(q.d_sum, q.d_count)}
    if k == "q14":
        q = Q14Query(t["items"], t["part"], b"PROMO", *_ship_range(c["days"]))
        return {"kind": k, "q": q, "out": _cleared(q.cnt, q.npairs, q.g_ng, q.g_key, *q.g_out,
                                                   q.t_ng, q.t_key, *q.t_out)}
    if k == "predict":
        q = PredictQuery(t["reviews"], t["model"], c["nfeat"], c["hidden"], 2, c["year_min"], 6)
        return {"kind": k, "q": q, "out": _cleared(q.cnt, q.g_ng, q.g_key, *q.g_out)}
    if k == "batch":
        b = BatchStarQuery(t["instances"], c["cut"])
        out = _cleared(b.q.cnt, b.q.npairs, b.q.ga_ng, b.q.ga_key, *b.q.ga_out)
        b.capture()
        return {"kind": k, "q": b, "out": out}
    if k == "learned":
        n, nr = max(c["nl"], c["nr"]), c["nr"]
        t["bits"] = max(1, math.ceil(math.log2(n / 3072))) if n > 3072 else 1
        flags = tqp.JOIN_SORTED | tqp.JOIN_RANGES
        # at most one range per row of the smaller side
        return {"kind": k, **t, "ranges": [_zeros(min(c["nl"], nr)) for _ in range(5)], "flags": flags,
                "count": _zeros(1), "nranges": _zeros(1),
                "ws": tqp.workspace(tqp.join_workspace_bytes(c["nl"], nr, torch.int64, flags))}
    if k == "sort":
        return {"kind": k, "rows": c["rows"], **t}
    dt = _dtype(c["dtype"])
    if k == "groupby":
        n, aggs = c["n"], [("sum", 0), ("sum_product", 0, 1), ("count",)]
        return {"kind": k, **t, "aggs": aggs, "groups": _zeros(1), "out_key": _zeros(n, dt),
                "out": [_zeros(n) for _ in aggs],
                "ws": tqp.workspace(tqp.groupby_workspace_bytes(n, dt, len(aggs), 0))}
    # room for the pairs expected from uniform keys and a quarter more
    cap = int(1.25 * c["nl"] * c["nr"] / c["keys"]) + 4096
    return {"kind": k, **t, "cap": cap, "count": _zeros(1), "out_l": _zeros(cap, torch.int32),
            "out_r": _zeros(cap, torch.int32), "out_key": _zeros(cap, dt),
            "ws": tqp.workspace(tqp.join_workspace_bytes(c["nl"], c["nr"], dt, 0, cap))}


def _zeros(n, dtype=torch.int64):
    return torch.zeros(n, dtype=dtype, device="cuda")


def run(state):
    s, k = state, state["kind"]
    if "q" in s:
        s["q"].run()
        return s["out"]
    if k == "learned":
        left, right, bits = s["left"], s["right"], s["bits"]
        model = tqp.lcdf_train([left, right])
        lk, lr, _ = tqp.partition_sort(left, model=model, bucket_bits=bits)
        rk, rr, _ = tqp.partition_sort(right, model=model, bucket_bits=bits)
        tqp.join_into(lk, rk, s["flags"], None, None, None, 0, s["count"], s["ws"], ranges=s["ranges"],
                      range_cap=s["ranges"][0].numel(), d_nranges=s["nranges"])
        return [lk, lr, rk, rr, s["count"], s["nranges"], s["ranges"]]
    if k == "sort":
        got = tqp.sort(s["key"], payload=s["pay"], want_rows=s["rows"])
        return [x for x in got if x is not None]
    if k == "groupby":
        tqp.groupby_agg_into(s["key"], s["vals"], s["aggs"], s["out_key"], s["out"], s["groups"], s["ws"])
        return [s["groups"], s["out_key"], s["out"]]
    tqp.join_into(s["left"], s["right"], 0, s["out_l"], s["out_r"], s["out_key"], s["cap"], s["count"],
                  s["ws"])
    return [s["count"], s["out_l"], s["out_r"], s["out_key"]]


# ----------------------------------------------- what a pass cannot avoid ----

def work(case):
    """Each input column read once and each result written once; a table's
    columns behind a selective filter count for the rows expected to be kept."""
    c, k = case, case["kind"]
    if k == "star":
        keep, nd = min(1.0, c["cut"] / DAYS), c["nd"]
        pay = 12 if c["mode"] == "q1" else 21
        b = c["n"] * (4 + keep * pay) + 8 * nd + 24 * 2 * c["cats"]
        if c["mode"] == "q2":
            b += 20 * min(nd, int(c["n"] * keep))
        return {"bytes": b, "flops": 0}
    if k == "star3":
        kept = c["n"] * (min(100, c["cut"]) / 100) ** 3
        return {"bytes": 12 * c["n"] + 16 * kept + 12 * (c["nd1"] + c["nd2"] + c["nd3"]), "flops": 0}
    if k == "q6":
        kept = c["n"] * c["days"] / DAYS * 3 / 11 * 23 / 50
        return {"bytes": 13 * c["n"] + 8 * kept, "flops": 0}
    if k == "q14":
        kept = c["n"] * min(1.0, c["days"] / DAYS)
        return {"bytes": 8 * c["n"] + 13 * kept + (4 + 9) * c["nd"], "flops": 0}
    if k == "predict":
        kept = c["n"] * (2024 - c["year_min"]) / 14
        return {"bytes": 4 * c["n"] + kept * (1 + 4 * c["nfeat"]),
                "flops": kept * 2 * c["hidden"] * (c["nfeat"] + 2)}
    if k == "batch":
        n = sum(int(c["lo"] * (c["hi"] / c["lo"]) ** ((i + 0.5) / c["k"])) for i in range(c["k"]))
        return {"bytes": n * (4 + min(1.0, c["cut"] / DAYS) * 12) + 8 * n / 20, "flops": 0}
    if k == "learned":
        return {"bytes": (8 + 12) * (c["nl"] + c["nr"]) + 40 * 0.2 * c["nr"], "flops": 0}
    size = 4 if c.get("dtype") == "int32" else 8
    if k == "sort":
        return {"bytes": c["n"] * (2 * (size + c["pay8"] + 8 * c["pay64"]) + 4 * c["rows"]), "flops": 0}
    if k == "groupby":
        return {"bytes": c["n"] * (size + 9) + min(c["n"], c["span"]) * (size + 24), "flops": 0}
    return {"bytes": size * (c["nl"] + c["nr"]) + (8 + size) * c["nl"] * c["nr"] / c["keys"], "flops": 0}


# ------------------------------------------------- the answer, plain torch ----

def _one(value):
    return torch.tensor([int(value)])


def _padded(values, size):
    out = _zeros(size)
    m = min(len(values), size)
    out[:m] = values[:m]
    return out


def _grouped(key, vals, size):
    """Groups of an integer key, ascending: count of groups, keys, sums, counts; padded to size."""
    uniq, inv, cnt = torch.unique(key, return_inverse=True, return_counts=True)
    sums = [torch.zeros(len(uniq), dtype=torch.int64, device="cuda").index_add_(0, inv, v) for v in vals]
    return [_one(len(uniq)), *(_padded(x, size) for x in (uniq.to(torch.int64), *sums, cnt))]


def _span(col):
    return int(col.max()) - int(col.min()) + 1


def _ranges(left, right):
    lu, lc = torch.unique_consecutive(left, return_counts=True)
    ru, rc = torch.unique_consecutive(right, return_counts=True)
    ls, rs = torch.cumsum(lc, 0) - lc, torch.cumsum(rc, 0) - rc
    at = torch.searchsorted(ru, lu).clamp_(max=len(ru) - 1)
    hit = ru[at] == lu
    at = at[hit]
    return {"key": lu[hit].to(torch.int64), "lstart": ls[hit], "lcnt": lc[hit], "rstart": rs[at],
            "rcnt": rc[at], "total": int((lc[hit] * rc[at]).sum())}


def exact(case, seed):
    c, k = case, case["kind"]
    if k == "batch":
        return None
    t = _tables(c, seed)
    if k == "star":
        f, dim = t["fact"], t["dim"]
        rows = torch.nonzero(f["day"] < c["cut"]).view(-1)
        cat = torch.empty(c["nd"], dtype=torch.int64, device="cuda")
        cat[dim["pk"].long()] = dim["cat"].long()
        fk, qty = f["fk"][rows].long(), f["qty"][rows]
        m = _one(len(rows))
        if c["mode"] == "q1":
            return [m, m, *_grouped(cat[fk], [qty], _span(dim["cat"]))]
        g = _grouped(f["flag"][rows].long() * 2 + cat[fk] % 2, [qty, f["price"][rows]],
                     2 * _span(f["flag"]))
        return [m, m, *g, *_grouped(fk, [qty], c["n"])]
    if k == "star3":
        f, keep, cats = t["fact"], None, []
        for i in (1, 2, 3):
            d, fk = t["d%d" % i], f["fk%d" % i]
            size = c["nd%d" % i]
            ok = torch.zeros(size, dtype=torch.bool, device="cuda")
            ok[d["pk"].long()] = d["attr"] < c["cut"]
            cat = torch.empty(size, dtype=torch.int64, device="cuda")
            cat[d["pk"].long()] = d["cat"].long()
            cats.append(cat)
            hit = torch.cat([ok[x.long()] for x in fk.split(1 << 26)])
            keep = hit if keep is None else keep & hit
        rows = torch.nonzero(keep).view(-1)
        key = cats[0][f["fk1"][rows].long()] * 5 + cats[1][f["fk2"][rows].long()]
        size = max(int(t["d1"]["cat"].max()) * 5 + int(t["d2"]["cat"].max()) + 1, 1)
        return [_one(len(rows)), *_grouped(key, [f["qty"][rows] * f["price"][rows]], size)]
    if k == "q6":
        it, (lo, hi) = t["items"], _ship_range(c["days"])
        keep = ((it["ship"] >= lo) & (it["ship"] < hi) & (it["discount"] >= 5) & (it["discount"] <= 7)
                & (it["quantity"] < 24))
        return [(it["price"][keep] * it["discount"][keep]).sum().view(1), keep.sum().view(1)]
    if k == "q14":
        it, part, (lo, hi) = t["items"], t["part"], _ship_range(c["days"])
        rows = torch.nonzero((it["ship"] >= lo) & (it["ship"] < hi)).view(-1)
        want = torch.tensor(list(b"PROMO"), dtype=torch.uint8, device="cuda")
        flag = torch.empty(c["nd"], dtype=torch.int64, device="cuda")
        flag[part["pk"].long()] = (part["type"][:, :5] == want).all(1).long()
        promo = flag[it["partkey"][rows].long()]
        rev = it["price"][rows] * (100 - it["discount"][rows].long())
        m = _one(len(rows))
        return [m, m, *_grouped(promo, [rev], 2), *_grouped(torch.zeros_like(promo), [rev], 1)]
    if k == "predict":
        r = t["reviews"]
        keep = r["year"] >= c["year_min"]
        g = _grouped(r["rating"][keep].long(), [], 6)
        # the class is decided by float32 rounding, so its sum has no 64-bit value
        return [keep.sum().view(1), g[0], g[1], None, g[2]]
    if k == "learned":
        (lk, lr), (rk, rr) = (torch.sort(t[s], stable=True) for s in ("left", "right"))
        r, size = _ranges(lk, rk), min(c["nl"], c["nr"])
        return [lk, lr, rk, rr, _one(r["total"]), _one(len(r["key"])),
                [_padded(r[x], size) for x in ("key", "lstart", "lcnt", "rstart", "rcnt")]]
    if k == "sort":
        key, rows = torch.sort(t["key"], stable=True)
        out = [key] + ([rows] if c["rows"] else [])
        return out + [[p[rows] for p in t["pay"]]] if t["pay"] else out
    if k == "groupby":
        v, w = t["vals"]
        g = _grouped(t["key"].long(), [v, v * w], c["n"])
        return [g[0], g[1], g[2:]]
    (lk, lr), (rk, rr) = (torch.sort(t[s], stable=True) for s in ("left", "right"))
    r = _ranges(lk, rk)
    m = r["lcnt"] * r["rcnt"]
    at = torch.repeat_interleave(torch.arange(len(m), device="cuda"), m)
    p = torch.arange(r["total"], device="cuda") - (torch.cumsum(m, 0) - m)[at]
    i, j = p // r["rcnt"][at], p % r["rcnt"][at]
    cap = int(1.25 * c["nl"] * c["nr"] / c["keys"]) + 4096
    return [_one(r["total"]), *(_padded(x, cap) for x in (lr[r["lstart"][at] + i], rr[r["rstart"][at] + j],
                                                          r["key"][at]))]
