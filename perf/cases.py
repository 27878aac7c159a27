"""The work that performance is measured on: one pass of each public operation,
as a query engine calls it, over the range of sizes that this repository's
workloads cover.

The engine of these cases keeps one context (its device arena), and for every
query its plan, its input columns and its result buffers; a pass enqueues calls
of the C ABI on the current stream and reads nothing back except where a count
is needed to go on.  Result buffers are cleared once, when they are made, so
that entries past a result's count are zero.  Fused queries return their groups
in no fixed order: the engine puts sums beside the dimension they belong to
(`dense`: one sum per dimension key), or orders the groups by key.

Tables follow the synthetic recipes of gen/ (shuffled surrogate keys 1..N,
segment U[0, 4], date U[0, 2406], price U[90000, 10500000], discount U[0, 10],
Zipf foreign keys, unique build keys with hit ratio 0.5, order keys U[1, N] with
quantity U[1, 50]), drawn on the GPU.
"""
import ctypes
import math

import torch

from paper_2512_02862_amd import pyst

ARENA = 16 << 30
DATE_MAX, DATE_LT = 2406, 1200
PRICE_LO, PRICE_HI, PRICE_GE = 90_000, 10_500_000, 1_000_000
HALF = 1 << 62
ID_STEP, ID_BASE = 1_000_003, -(1 << 40)  # sparse 64-bit identifiers: ID_BASE + i * ID_STEP

_engine = None


def engine():
    """The program's context, made once."""
    global _engine
    if _engine is None:
        _engine = pyst.Ctx(0, ARENA)
    return _engine


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # latency: a query over a small table, as an interactive dashboard sends it (six launches)
        {"name": "star_small", "op": "star", "build": 150_000, "probe": 1_500_000},
        # the measured star query: 1.5M dimension rows, 60M fact rows
        {"name": "star_full", "op": "star", "build": 1_500_000, "probe": 60_000_000},
        # the two-join query at its full size with skewed foreign keys, groups delivered in key order
        {"name": "chain_full", "op": "chain", "a": 3_000_000, "b": 300_000, "fact": 120_000_000, "skew": 1.0},
        # many uneven query fragments in one call (10k to 20M fact rows each)
        {"name": "batch_64", "op": "batch", "fragments": 64, "lo": 10_000, "hi": 20_000_000, "tuned": True},
        # the send side of a shuffle: the star's fact table to 64 destinations
        {"name": "shuffle_64", "op": "shuffle", "rows": 60_000_000, "fanout": 64, "key64": False, "pay32": 1,
         "pay64": 1, "filtered": False},
        # a pushed-down filter, then the send side of the rows that are left, with wide rows, 64-bit keys,
        # ragged sizes and a fanout that is no power of two
        {"name": "filter_shuffle_200", "op": "shuffle", "rows": 20_000_017, "fanout": 200, "key64": True, "pay32": 1,
         "pay64": 4, "filtered": True},
        # the join microbenchmark, one GPU's share: build, probe and materialize 4 columns a side
        {"name": "join_k4", "op": "join", "build": 60_000_000, "probe": 160_000_000, "cols": 4, "key64": False},
        # a table built over sparse 64-bit identifiers and probed once, values looked up
        {"name": "lookup_ids", "op": "lookup", "build": 1_000_003, "probe": 20_000_017, "key64": True, "pay64": True},
        # aggregation with groups far beyond the caches (order totals), ordered by key
        {"name": "groupby_orders", "op": "groupby", "rows": 60_000_000, "groups": 15_000_000, "key64": False,
         "val64": False, "bounded": True},
        # aggregation into few groups (revenue per day), ordered by key
        {"name": "groupby_dates", "op": "groupby", "rows": 60_000_000, "groups": 2407, "key64": False, "val64": True,
         "bounded": True},
        # latency: a small aggregation over 64-bit identifiers, ordered by key, its number of groups not known
        {"name": "groupby_small", "op": "groupby", "rows": 100_003, "groups": 5_000, "key64": True, "val64": True,
         "bounded": False},
        # a fact table in pinned host memory streamed through the device in chunks
        {"name": "streamed_8m", "op": "streamed", "build": 300_000, "rows": 8_000_000, "chunk": 2_000_000,
         "packed": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["star", "star", "chain", "batch", "shuffle", "shuffle", "join", "lookup", "groupby", "groupby",
                     "groupby", "streamed"])
    if op == "star":
        build = _log(rng, 1_000, 1_500_000)
        return {"op": op, "build": build, "probe": min(60_000_000, int(build * rng.uniform(5, 60)) + 1)}
    if op == "chain":
        fact = _log(rng, 100_000, 100_000_000)
        return {"op": op, "a": fact // 40 + 1, "b": fact // 400 + 7, "fact": fact, "skew": rng.choice([0.0, 0.5, 1.0])}
    if op == "batch":
        lo = _log(rng, 1_000, 20_000)
        return {"op": op, "fragments": rng.randint(3, 96), "lo": lo, "hi": _log(rng, 4 * lo, 8_000_000),
                "tuned": rng.random() < 0.5}
    if op == "shuffle":
        return {"op": op, "rows": _log(rng, 10_000, 40_000_000), "fanout": _log(rng, 2, 1024),
                "key64": rng.random() < 0.5, "pay32": rng.randint(0, 2), "pay64": rng.randint(0, 4),
                "filtered": rng.random() < 0.5}
    if op == "join":
        build = _log(rng, 10_000, 50_000_000)
        return {"op": op, "build": build, "probe": min(150_000_000, int(build * rng.uniform(0.8, 4)) + 1),
                "cols": rng.randint(1, 4), "key64": rng.random() < 0.3}
    if op == "lookup":
        build = _log(rng, 1_000, 10_000_000)
        return {"op": op, "build": build, "probe": int(build * rng.uniform(1, 8)) + 1, "key64": rng.random() < 0.5,
                "pay64": rng.random() < 0.5}
    if op == "groupby":
        rows = _log(rng, 5_000, 60_000_000)
        return {"op": op, "rows": rows, "groups": min(15_000_000, _log(rng, 4, max(8, rows // 2))),
                "key64": rng.random() < 0.5, "val64": rng.random() < 0.5, "bounded": rng.random() < 0.7}
    return {"op": "streamed", "build": _log(rng, 10_000, 300_000), "rows": _log(rng, 500_000, 12_000_000),
            "chunk": 1024 * rng.randint(256, 4096), "packed": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs

class _Draw:
    """Seeded random columns on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def ints(self, n, lo, hi, dtype=torch.int32):
        """n values uniform over [lo, hi]."""
        return torch.randint(lo, hi + 1, (n,), generator=self.g, device="cuda", dtype=dtype)

    def perm(self, n, dtype=torch.int32):
        """1..n, shuffled."""
        return (torch.randperm(n, generator=self.g, device="cuda") + 1).to(dtype)

    def zipf(self, n, keys, s):
        """n keys of 1..keys, P(k) ~ k^-s."""
        if s == 0.0:
            return self.ints(n, 1, keys)
        w = torch.arange(1, keys + 1, device="cuda", dtype=torch.float64).pow(-s).cumsum(0)
        u = torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64) * w[-1]
        return (torch.searchsorted(w, u).clamp_(max=keys - 1) + 1).to(torch.int32)


def _star_tables(d, build, probe):
    b = {"key": d.perm(build), "segment": d.ints(build, 0, 4)}
    return b, [d.ints(probe, 1, build), d.ints(probe, 0, DATE_MAX), d.ints(probe, PRICE_LO, PRICE_HI, torch.int64)]


def _chain_tables(d, c):
    a = {"key": d.perm(c["a"]), "date": d.ints(c["a"], 0, DATE_MAX)}
    b = {"key": d.perm(c["b"]), "segment": d.ints(c["b"], 0, 4)}
    return a, b, _chain_fact(d, c["fact"], c["a"], c["b"], c["skew"])


def _chain_fact(d, n, na, nb, skew):
    return [d.ints(n, 1, na), d.zipf(n, nb, skew), d.ints(n, 0, DATE_MAX), d.ints(n, PRICE_LO, PRICE_HI, torch.int64),
            d.ints(n, 0, 10)]


def _sizes(c):
    """Fragment sizes spread evenly over the logarithm of [lo, hi], the large and the small mixed."""
    f = c["fragments"]
    s = [int(c["lo"] * (c["hi"] / c["lo"]) ** (i / max(1, f - 1))) for i in range(f)]
    return [s[(i * 37) % f] if math.gcd(37, f) == 1 else s[i] for i in range(f)]


def _fragments(d, c):
    return [_star_tables(d, max(1, n // 10), n) for n in _sizes(c)]


def _shuffle_tables(d, c):
    n = c["rows"]
    key = d.ints(n, 1, max(1, n // 40)) if not c["key64"] else d.ints(n, 0, max(1, n // 4), torch.int64) * ID_STEP + ID_BASE
    pays = [d.ints(n, 0, DATE_MAX) for _ in range(c["pay32"])]
    pays += [d.ints(n, PRICE_LO, PRICE_HI, torch.int64) for _ in range(c["pay64"])]
    return key, pays, d.ints(n, 0, DATE_MAX) if c["filtered"] else None


def _join_cap(c):
    """Half of the probes find a partner."""
    return int(0.51 * c["probe"] + 8 * math.sqrt(c["probe"])) + 64


def _join_tables(d, c):
    nb, np_ = c["build"], c["probe"]
    if c["key64"]:
        bk = d.perm(nb, torch.int64) * ID_STEP + ID_BASE
        pk = d.ints(np_, 1, 2 * nb, torch.int64) * ID_STEP + ID_BASE
    else:
        bk, pk = d.perm(nb), d.ints(np_, 1, 2 * nb)
    return bk, pk


def _groupby_tables(d, c):
    k = d.ints(c["rows"], 1, c["groups"], torch.int64 if c["key64"] else torch.int32)
    k = k * ID_STEP + ID_BASE if c["key64"] else k
    v = d.ints(c["rows"], PRICE_LO, PRICE_HI, torch.int64) if c["val64"] else d.ints(c["rows"], 1, 50)
    return k, v


def _zeros(n, dtype=torch.int64):
    return torch.zeros(max(1, n), dtype=dtype, device="cuda")


def _result(s, cap):
    s.update(keys=_zeros(cap), sums=_zeros(cap), count=_zeros(1), cap=cap)


def _cols(ts, make=None):
    make = make or pyst.col
    return (pyst.Col * max(1, len(ts)))(*[make(t) for t in ts])


def _ptrs(ts):
    return (ctypes.c_void_p * max(1, len(ts)))(*[t.data_ptr() for t in ts])


def prepare(case, seed):
    c, d = case, _Draw(seed)
    s = {"op": c["op"], "case": c, "ctx": engine(), "lib": pyst.load()}
    op = c["op"]
    if op == "star":
        b, fact = _star_tables(d, c["build"], c["probe"])
        s.update(hold=(b, fact), plan=pyst.star_plan(b).to_c(), fact=_cols(fact), dense=_zeros(c["build"] + 1))
        _result(s, c["build"])
    elif op == "chain":
        a, b, fact = _chain_tables(d, c)
        s.update(hold=(a, b, fact), plan=pyst.chain_plan(a, b).to_c(), fact=_cols(fact))
        _result(s, max(1024, c["fact"] // 4))  # about a tenth of the rows: 1/5 of the segments, 1/2 of the dates
        s.update(okeys=_zeros(s["cap"]), osums=_zeros(s["cap"]))
    elif op == "batch":
        frags = _fragments(d, c)
        caps = [b["key"].numel() for b, _ in frags]
        _result(s, sum(caps))
        s["count"] = _zeros(len(frags))
        base = torch.cumsum(torch.tensor([0] + [x + 1 for x in caps[:-1]]), 0)
        s["base"] = torch.repeat_interleave(base, torch.tensor(caps)).cuda()
        s["dense"] = _zeros(sum(caps) + len(caps))
        arr, hold, at = (pyst.Fragment * len(frags))(), [], 0
        for i, (b, fact) in enumerate(frags):
            plan, keep = pyst.star_plan(b).to_c()
            plan, cols = ctypes.pointer(plan), _cols(fact)
            hold += [b, fact, plan, keep, cols]
            arr[i] = pyst.Fragment(plan, ctypes.cast(cols, ctypes.POINTER(pyst.Col)), len(fact), 0,
                                   s["keys"].data_ptr() + 8 * at, s["sums"].data_ptr() + 8 * at, caps[i],
                                   s["count"].data_ptr() + 8 * i)
            at += caps[i]
        s.update(hold=hold, frags=arr, tuning=pyst.Tuning(16, 1024, 0.7) if c["tuned"] else None)
    elif op == "shuffle":
        key, pays, date = _shuffle_tables(d, c)
        outs = [_zeros(c["rows"], t.dtype) for t in [key] + pays]
        s.update(hold=(key, pays, date), key=_cols([key]), pays=_cols(pays), npay=len(pays), outs=outs,
                 outp=_ptrs(outs), offsets=_zeros(c["fanout"] + 1))
        if date is not None:
            s.update(date=_cols([date]), pred=(pyst.Pred * 1)(pyst.Pred(0, pyst.CMP["<"], DATE_LT)),
                     sel=_zeros(c["rows"], torch.int32), nsel=_zeros(1))
    elif op == "join":
        bk, pk = _join_tables(d, c)
        bc = [d.ints(c["build"], -HALF, HALF, torch.int64) for _ in range(c["cols"])]
        pc = [d.ints(c["probe"], -HALF, HALF, torch.int64) for _ in range(c["cols"])]
        cap = _join_cap(c)
        outs = [_zeros(cap, t.dtype) for t in pc + bc]
        s.update(hold=(bk, pk, bc, pc), bk=_cols([bk]), pk=_cols([pk]), bc=_cols(bc), pc=_cols(pc), outs=outs,
                 outp=_ptrs(outs), prow=_zeros(cap, torch.int32), brow=_zeros(cap, torch.int32), count=_zeros(1), cap=cap)
    elif op == "lookup":
        bk, pk = _join_tables(d, c)
        pay = d.ints(c["build"], -HALF, HALF, torch.int64) if c["pay64"] else d.ints(c["build"], 0, DATE_MAX)
        s.update(hold=(bk, pk, pay), bk=bk, pay=pay, pk=_cols([pk]), rows=_zeros(c["probe"], torch.int32),
                 vals=_zeros(c["probe"]), count=_zeros(1), cap=c["probe"])
    elif op == "groupby":
        k, v = _groupby_tables(d, c)
        s.update(hold=(k, v), k=_cols([k]), v=_cols([v]), bound=c["groups"] if c["bounded"] else 0)
        _result(s, c["groups"] if c["bounded"] else c["rows"])
    else:
        b = {"key": d.perm(c["build"]), "segment": d.ints(c["build"], 0, 4)}
        fact = [t.cpu().pin_memory() for t in _chain_fact(d, c["rows"], 10 * c["build"], c["build"], 0.0)]
        s.update(plan=pyst.fact_star_plan(b).to_c(), dense=_zeros(c["build"] + 1))
        if c["packed"]:
            packed = [pyst.pack(t) for t in fact]
            s.update(hold=(b, packed), nfact=len(fact), fact=(pyst.PackedCol * len(fact))(
                *[pyst.packed_col(bl, w, t.numel(), t.dtype) for t, (bl, w) in zip(fact, packed)]))
        else:
            s.update(hold=(b, fact), nfact=len(fact), fact=_cols(fact, pyst.host_col))
        _result(s, c["build"])
    return s


# ------------------------------------------------------------------ one pass

def _ok(lib, status):
    if status != pyst.OK:
        raise pyst.PystError(status, lib.pyst_last_error().decode())


def _dense(s):
    """One sum per dimension key: what the query found, beside the dimension."""
    s["dense"].zero_()
    return s["dense"].scatter_(0, s["keys"] + s["base"] if "base" in s else s["keys"], s["sums"])


def run(s):
    lib, h, c, ref = s["lib"], s["ctx"].h, s["case"], ctypes.byref
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def p(t):
        return ctypes.c_void_p(t.data_ptr())

    op = s["op"]
    if op in ("star", "chain"):
        _ok(lib, lib.pyst_query(h, ref(s["plan"][0]), s["fact"], len(s["fact"]), p(s["keys"]), p(s["sums"]), s["cap"],
                                p(s["count"]), st))
        if op == "star":
            return {"dense": _dense(s), "count": s["count"]}
        m = int(s["count"].item())
        order = torch.empty(m, dtype=torch.int64, device="cuda")
        torch.sort(s["keys"][:m], out=(s["okeys"][:m], order))
        torch.index_select(s["sums"][:m], 0, order, out=s["osums"][:m])
        return {"keys": s["okeys"], "sums": s["osums"], "count": s["count"]}
    if op == "batch":
        _ok(lib, lib.pyst_query_batch(h, s["frags"], len(s["frags"]), None if s["tuning"] is None else ref(s["tuning"]),
                                      st))
        return {"dense": _dense(s), "count": s["count"]}
    if op == "shuffle":
        sel = nsel = None
        if c["filtered"]:
            sel, nsel = p(s["sel"]), p(s["nsel"])
            _ok(lib, lib.pyst_filter(h, s["date"], 1, s["pred"], 1, sel, nsel, st))
        _ok(lib, lib.pyst_partition(h, s["key"], s["pays"], s["npay"], sel, nsel, c["fanout"], s["outp"],
                                    p(s["offsets"]), st))
        out = {"cols": s["outs"], "offsets": s["offsets"]}
        return dict(out, sel=s["sel"], nsel=s["nsel"]) if c["filtered"] else out
    if op == "join":
        k = c["cols"]
        _ok(lib, lib.pyst_join_materialize(h, s["bk"], s["bc"], k, s["pk"], s["pc"], k, 0.5, 1, s["outp"], p(s["prow"]),
                                           p(s["brow"]), s["cap"], p(s["count"]), st))
        return {"cols": s["outs"], "prow": s["prow"], "brow": s["brow"], "count": s["count"]}
    if op == "lookup":
        table = pyst.join_build(s["ctx"], s["bk"], s["pay"])
        _ok(lib, lib.pyst_join_probe(h, table.h, s["pk"], None, None, p(s["rows"]), p(s["vals"]), s["cap"],
                                     p(s["count"]), st))
        table.destroy()
        return {"rows": s["rows"], "vals": s["vals"], "count": s["count"]}
    if op == "groupby":
        _ok(lib, lib.pyst_groupby_sum(h, s["k"], s["v"], None, None, s["bound"], 0.5, p(s["keys"]), p(s["sums"]),
                                      p(s["count"]), 1, st))
        return {"keys": s["keys"], "sums": s["sums"], "count": s["count"]}
    call = lib.pyst_query_streamed_packed if c["packed"] else lib.pyst_query_streamed
    _ok(lib, call(h, ref(s["plan"][0]), s["fact"], s["nfact"], c["chunk"], 2, p(s["keys"]), p(s["sums"]), s["cap"],
                  p(s["count"]), st))
    return {"dense": _dense(s), "count": s["count"]}


# ------------------------------------------------------------------ what a pass cannot do without

def _groups(rows, keys):
    """Distinct keys among `rows` rows uniform over `keys` keys, expected."""
    return keys * -math.expm1(-rows / max(keys, 1))


def work(case):
    c, op = case, case["op"]
    live = 0.2 * DATE_LT / (DATE_MAX + 1)  # one segment of five, the dates below DATE_LT
    if op == "star":
        g = _groups(c["probe"] * live, 0.2 * c["build"])
        return {"bytes": 16 * c["probe"] + 8 * c["build"] + 16 * g + 8 * c["build"], "flops": 0}
    if op == "chain":
        w = torch.arange(1, c["b"] + 1, dtype=torch.float64).pow(-c["skew"])
        rows = c["fact"] * DATE_LT / (DATE_MAX + 1) * w / w.sum()
        g = 0.2 * float((-(DATE_MAX + 1) * torch.expm1(-rows / (DATE_MAX + 1))).sum())
        return {"bytes": 24 * c["fact"] + 8 * c["a"] + 8 * c["b"] + 16 * g, "flops": 0}
    if op == "batch":
        return {"bytes": sum(work({"op": "star", "build": max(1, n // 10), "probe": n})["bytes"] for n in _sizes(c)),
                "flops": 0}
    if op == "shuffle":
        row = (8 if c["key64"] else 4) + 4 * c["pay32"] + 8 * c["pay64"]
        part = DATE_LT / (DATE_MAX + 1) if c["filtered"] else 1.0
        return {"bytes": c["rows"] * (2 * row * part + (4 + 4 * part if c["filtered"] else 0)) + 8 * c["fanout"],
                "flops": 0}
    if op == "join":
        kb = 8 if c["key64"] else 4
        hits = 0.5 * c["probe"]
        return {"bytes": (kb + 8 * c["cols"]) * (c["build"] + c["probe"]) + hits * (8 + 16 * c["cols"]), "flops": 0}
    if op == "lookup":
        kb = 8 if c["key64"] else 4
        return {"bytes": c["build"] * (kb + (8 if c["pay64"] else 4)) + c["probe"] * kb + 0.5 * c["probe"] * 12,
                "flops": 0}
    if op == "groupby":
        row = (8 if c["key64"] else 4) + (8 if c["val64"] else 4)
        return {"bytes": row * c["rows"] + 16 * _groups(c["rows"], c["groups"]), "flops": 0}
    g = _groups(c["rows"] * live, 0.2 * c["build"])
    return {"bytes": 16 * c["rows"] + 16 * c["build"] + 16 * g, "flops": 0}  # three of the five columns are needed


# ------------------------------------------------------------------ the same in plain torch

def _exact_star(b, fk, date, price):
    n = b["key"].numel()
    one = torch.zeros(n + 1, dtype=torch.bool, device="cuda")
    one[b["key"].long()] = b["segment"] == 1
    fk = fk.long()
    live = one[fk] & (date < DATE_LT)
    dense, seen = _zeros(n + 1), torch.zeros(n + 1, dtype=torch.bool, device="cuda")
    dense.scatter_add_(0, fk[live], price[live])
    seen[fk[live]] = True
    return dense, seen.sum().reshape(1)


def _mix32(h):
    for shift, mul in ((16, 0x85EBCA6B), (13, 0xC2B2AE35), (16, 1)):
        h = h ^ (h >> shift)
        h = (h * (mul & 0xFFFF) + (((h * (mul >> 16)) & 0xFFFF) << 16)) & 0xFFFFFFFF
    return h


def _mix64(h):
    def shr(x):
        return (x >> 33) & ((1 << 31) - 1)

    for mul in (0xFF51AFD7ED558CCD - (1 << 64), 0xC4CEB9FE1A85EC53 - (1 << 64)):
        h = (h ^ shr(h)) * mul  # wraps modulo 2^64
    return h ^ shr(h)


def _padded(t, n):
    out = _zeros(n, t.dtype)
    out[:t.numel()] = t
    return out


def exact(case, seed):
    c, d, op = case, _Draw(seed), case["op"]
    if op == "star":
        b, (fk, date, price) = _star_tables(d, c["build"], c["probe"])
        dense, count = _exact_star(b, fk, date, price)
        return {"dense": dense, "count": count}
    if op == "chain":
        a, b, (afk, bfk, date, price, disc) = _chain_tables(d, c)
        one = torch.zeros(c["b"] + 1, dtype=torch.bool, device="cuda")
        one[b["key"].long()] = b["segment"] == 1
        when = _zeros(c["a"] + 1)
        when[a["key"].long()] = a["date"].long()
        at = ((date < DATE_LT) & one[bfk.long()]).nonzero().reshape(-1)
        keys, inv = torch.unique((bfk[at].long() << 32) | when[afk[at].long()], return_inverse=True)
        sums = _zeros(keys.numel()).scatter_add_(0, inv, price[at] * (100 - disc[at].long()))
        cap = max(1024, c["fact"] // 4)
        return {"keys": _padded(keys, cap), "sums": _padded(sums, cap),
                "count": torch.tensor([keys.numel()], device="cuda")}
    if op == "batch":
        got = [_exact_star(b, *fact) for b, fact in _fragments(d, c)]
        return {"dense": torch.cat([x for x, _ in got]), "count": torch.cat([n for _, n in got])}
    if op == "shuffle":
        key, pays, date = _shuffle_tables(d, c)
        at = torch.arange(c["rows"], device="cuda") if date is None else (date < DATE_LT).nonzero().reshape(-1)
        k = key[at]
        h = _mix64(k) & 0xFFFFFFFF if c["key64"] else _mix32(k.long() & 0xFFFFFFFF)
        to = h % c["fanout"]
        order = torch.sort(to, stable=True)[1]
        offs = torch.zeros(c["fanout"] + 1, dtype=torch.int64, device="cuda")
        offs[1:] = torch.cumsum(torch.bincount(to, minlength=c["fanout"]), 0)
        out = {"cols": [_padded(t[at][order], c["rows"]) for t in [key] + pays], "offsets": offs}
        if date is not None:
            out.update(sel=_padded(at.to(torch.int32), c["rows"]), nsel=torch.tensor([at.numel()], device="cuda"))
        return out
    if op in ("join", "lookup"):
        bk, pk = _join_tables(d, c)
        if c["key64"]:
            bk, pk = (bk - ID_BASE) // ID_STEP, (pk - ID_BASE) // ID_STEP
        row = torch.full((2 * c["build"] + 1,), -1, dtype=torch.int32, device="cuda")
        row[bk.long()] = torch.arange(c["build"], dtype=torch.int32, device="cuda")
        brow = row[pk.long()]
        prow = (brow >= 0).nonzero().reshape(-1)
        brow, count = brow[prow], torch.tensor([prow.numel()], device="cuda")
        if op == "lookup":
            pay = d.ints(c["build"], -HALF, HALF, torch.int64) if c["pay64"] else d.ints(c["build"], 0, DATE_MAX)
            return {"rows": _padded(prow.to(torch.int32), c["probe"]), "vals": _padded(pay[brow.long()].long(), c["probe"]),
                    "count": count}
        cap = _join_cap(c)
        bc = [_padded(d.ints(c["build"], -HALF, HALF, torch.int64)[brow.long()], cap) for _ in range(c["cols"])]
        pc = [_padded(d.ints(c["probe"], -HALF, HALF, torch.int64)[prow], cap) for _ in range(c["cols"])]
        return {"cols": pc + bc, "prow": _padded(prow.to(torch.int32), cap), "brow": _padded(brow, cap), "count": count}
    if op == "groupby":
        k, v = _groupby_tables(d, c)
        keys, inv = torch.unique(k.long(), return_inverse=True)
        cap = c["groups"] if c["bounded"] else c["rows"]
        sums = _zeros(keys.numel()).scatter_add_(0, inv, v.long())
        return {"keys": _padded(keys, cap), "sums": _padded(sums, cap), "count": torch.tensor([keys.numel()], device="cuda")}
    b = {"key": d.perm(c["build"]), "segment": d.ints(c["build"], 0, 4)}
    _, bfk, date, price, _ = _chain_fact(d, c["rows"], 10 * c["build"], c["build"], 0.0)
    dense, count = _exact_star(b, bfk, date, price)
    return {"dense": dense, "count": count}
