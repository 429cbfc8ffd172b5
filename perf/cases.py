"""Timed cases of the calling-context-tree library: builds, merges, activity flushes,
reports and lookups through the package's public calls, on synthetic traces made on the
GPU from a seed.

A case fixes the program and how often each of its call paths occurs, so that every seed
gives trees of the same shape; the seed gives the frame ids (and with them the canonical
order), the order of the events and their metrics.

A trace follows the shape a profiler hands over: root-first call paths (Python frames,
framework operators, C/C++ frames, a kernel leaf) drawn with Zipf popularity from a
program's call paths, which share prefixes, with time-like, byte-like and count-like
integer metrics.  Traces, merges and flushes take the sizes of the repository's bench
workloads where they are named after them, and draw() spreads over the range between.

    listed() / draw(rng)  cases       prepare(case, seed)  device inputs, kept trees
    run(state)            one pass    exact(case, seed)    the same outputs in plain torch
    work(case)            bytes       tolerance(case)      allowed difference
"""
import math
import zlib

import numpy as np
import torch

import paper_2411_02797_amd as cct

#: Keys every case has: what is called, and the program and trace it is called on.
#:   op         "build", "merge", "activity", "stats", "report", "query" or "filter"
#:   program    "layered" (templates branching off earlier ones), "deep" (a recursion cycle)
#:   events     events of the trace (of the base, where batches are merged into it)
#:   templates, roots, dmin, dmax, ids, zipf, hot: call paths of the program, top-level
#:              frames, path lengths, distinct frames, popularity exponent, share of events
#:              under the first eight top-level frames (0: all alike)
#:   metrics    integer metrics of an event
#:   batches, batch   merges or flushes that follow, and events (registered paths) in each
#:   dense      correlation IDs from a counter (True) or spread over 64 bits
#:   unsigned   frames and metrics handed over as uint32/uint64 tensors
_BASE = dict(op="build", program="layered", events=0, templates=0, roots=64, dmin=1, dmax=16, ids=2000, zipf=1.1, hot=0.0,
             metrics=1, batches=0, batch=0, dense=True, unsigned=False)
_L1M = dict(templates=65536, dmin=8, dmax=64, ids=50000, zipf=1.2)
_L16M = dict(templates=262144, dmin=16, dmax=128, ids=200000, zipf=1.1, hot=0.9)


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # a short profile of a small script: one build, bound by launches and latencies
        _case("build_10k", events=10_000, templates=6000, roots=8),
        # ragged paths, empty and one-frame ones up to several thousand frames long, all
        # eight metrics: a profile with deep Python stacks on some threads; odd sizes
        _case("build_ragged_60k", events=60_013, templates=20_011, roots=37, dmin=0, dmax=2500, ids=30_011, zipf=0.7, metrics=8,
              unsigned=True),
        # an ordinary training-step profile (the bench's layered_1m)
        _case("build_1m", events=1 << 20, metrics=3, **_L1M),
        # a whole training run's trace, the largest build (the bench's layered_16m)
        _case("build_16m", events=1 << 24, metrics=2, **_L16M),
        # deep recursive call paths (the bench's deep_recursion)
        _case("build_deep_4m", program="deep", events=1 << 22, dmin=256, dmax=512, ids=20_000),
        # a live profile: many small buffer flushes into a tree of moderate size
        _case("merge_small", op="merge", events=1 << 18, metrics=4, batches=8, batch=16_381, **_L1M),
        # large buffer flushes into a large tree (the bench's merge, four of its flushes)
        _case("merge_large", op="merge", events=1 << 23, metrics=4, batches=4, batch=1 << 21, **dict(_L16M, hot=0.0)),
        # GPU activity records joined with their call paths by correlation ID, then merged
        _case("activity_1m", op="activity", events=1 << 21, metrics=4, batches=2, batch=1 << 20, **dict(_L16M, hot=0.0)),
        # a build that keeps counts, minima and squares, and every node's statistics
        _case("stats_4m", op="stats", events=1 << 22, metrics=2, **_L16M),
        # a report on a fresh profile: build, bottom-up view, hotspots, small kernels
        _case("report_2m", op="report", events=1 << 21, metrics=2, **_L16M),
        # lookups of many call paths in a kept large tree (one in 1,024 is absent)
        _case("query_1m", op="query", events=1 << 24, metrics=2, batch=1 << 20, **_L16M),
        # the example analyses over a kept large tree
        _case("filter_16m", op="filter", events=1 << 24, metrics=2, **_L16M),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["build", "build", "build", "merge", "activity", "stats", "report", "query", "filter"])
    c = dict(_BASE, op=op, metrics=rng.randint(1, 8), unsigned=rng.random() < 0.5)
    c["events"] = _log_int(rng, 5_000, 6_000_000)
    if op == "build" and rng.random() < 0.25:
        c.update(program="deep", events=min(c["events"], 1_500_000), dmin=rng.randint(20, 250), dmax=rng.randint(251, 520),
                 ids=rng.randint(5_000, 40_000), metrics=rng.randint(1, 3))
        return c
    c["dmin"] = rng.choice([0, 1, 8, 16, 24])
    c["dmax"] = c["dmin"] + _log_int(rng, 8, 160)
    if c["events"] < 100_000 and rng.random() < 0.3:
        c["dmax"] = _log_int(rng, 300, 3000)
    c["templates"] = max(64, min(300_000, int(c["events"] * rng.uniform(0.02, 0.8))))
    if c["dmax"] > 250:
        c["templates"] = min(c["templates"], 20_000)
    c["roots"] = min(c["templates"], rng.randint(1, 80))
    c["ids"] = _log_int(rng, 500, 250_000)
    c["zipf"] = round(rng.uniform(0.6, 1.3), 3)
    c["hot"] = rng.choice([0.0, 0.9])
    if op in ("merge", "activity"):
        c["hot"] = 0.0
        c["events"] = min(c["events"], 3_000_000)
        c["batches"] = rng.randint(1, 5)
        c["batch"] = _log_int(rng, 1_000, 1_200_000)
        c["dense"] = rng.random() < 0.5
    if op == "query":
        c["batch"] = _log_int(rng, 200, 1_500_000)
    return c


# ---- the program and its traces --------------------------------------------------------


def _generators(c, seed):
    """The case's generator, for what all its seeds share, and the seed's."""
    text = repr(sorted((k, v) for k, v in c.items() if k != "name"))
    pair = torch.Generator(device="cuda"), torch.Generator(device="cuda")
    pair[0].manual_seed(zlib.crc32(text.encode()))
    pair[1].manual_seed(seed)
    return pair


def _frame_ids(n, h):
    """n distinct ids spread over uint32: a bijection of 32 bits, drawn from the seed."""
    mask = 0xFFFFFFFF
    a, b, c = torch.randint(0, 1 << 31, (3,), generator=h, device=h.device).tolist()
    x = (torch.arange(n, device=h.device) * (2 * a + 1) + b) & mask
    x = ((x ^ (x >> 16)) * ((2 * c + 1) & mask)) & mask
    return (x ^ (x >> 15)).to(torch.int32)


def _order(n, h):
    return torch.randperm(n, generator=h, device=h.device)


class _Program:
    """The call paths of a layered program as rows of a [templates, dmax] matrix."""

    def __init__(self, c, g, h):
        dev = g.device
        T, dmin, dmax = c["templates"], c["dmin"], c["dmax"]
        u = torch.rand(T, generator=g, device=dev, dtype=torch.float64)
        if dmax > 250:  # ragged: lengths spread over their logarithm
            length = torch.exp(u * math.log(dmax - dmin + 1)).long() - 1 + dmin
        else:
            length = dmin + (u * (dmax - dmin + 1)).long()
        length = length.clamp_(dmin, dmax)
        idx = torch.arange(T, device=dev)
        parent = (torch.rand(T, generator=g, device=dev, dtype=torch.float64) * idx).long()
        parent = torch.where(idx < c["roots"], idx, parent)
        # a template leaves its parent a geometric number of frames (mean 8) above its leaf
        u = torch.rand(T, generator=g, device=dev, dtype=torch.float64)
        leave = length - 2 - (torch.log1p(-u) / math.log(7.0 / 8.0)).floor().long()
        split = torch.minimum(leave, length[parent]).clamp_(min=1)
        split = torch.where(idx < c["roots"], torch.zeros_like(split), torch.minimum(split, (length - 1).clamp(min=0)))
        split = torch.minimum(split, length[parent])
        # frames: Python, framework, C/C++ and kernel ids from ranges of a pool over uint32
        pool = _frame_ids(c["ids"], h)
        rows = torch.empty(T, dmax, dtype=torch.int32, device=dev)
        n_py = torch.clamp(length - 2, min=0, max=20)
        fw_end = n_py + 1 + (torch.rand(T, generator=g, device=dev) * 4).long()
        for a in range(0, T, 1 << 16):
            b = min(T, a + (1 << 16))
            col = torch.arange(dmax, device=dev)[None, :]
            layer = (col >= n_py[a:b, None]).long() + (col >= fw_end[a:b, None]).long()
            layer = torch.where(col + 1 >= length[a:b, None], torch.full_like(layer, 3), layer)
            lo = torch.tensor([0.0, 0.4, 0.5, 0.9], device=dev, dtype=torch.float64)[layer]
            span = torch.tensor([0.4, 0.1, 0.4, 0.1], device=dev, dtype=torch.float64)[layer]
            at = (lo + span * torch.rand(b - a, dmax, generator=g, device=dev, dtype=torch.float64)) * c["ids"]
            rows[a:b] = pool[at.long().clamp_(max=c["ids"] - 1)]
        # prefixes, generation by generation (a parent's row is final before its children's)
        gen = torch.zeros(T, dtype=torch.long, device=dev)
        root = idx.clone()
        while True:
            nxt = torch.where(idx < c["roots"], torch.zeros_like(gen), gen[parent] + 1)
            root = root[parent]
            if torch.equal(nxt, gen):
                break
            gen = nxt
        col = torch.arange(dmax, device=dev)[None, :]
        for k in range(1, int(gen.max()) + 1):
            at = (gen == k).nonzero().squeeze(1)
            for part in at.split(1 << 16):
                rows[part] = torch.where(col < split[part, None], rows[parent[part]], rows[part])
        self.rows, self.length, self.root = rows, length, root

    def take(self, ev):
        return _flatten(self.length[ev], self.rows.shape[1], lambda a, b: self.rows[ev[a:b]])


def _flatten(length, width, rows_of):
    """(offsets, frames) of events whose frames are the first `length` columns of their rows."""
    n = length.numel()
    offsets = torch.zeros(n + 1, dtype=torch.int64, device=length.device)
    torch.cumsum(length, 0, out=offsets[1:])
    frames = torch.empty(int(offsets[-1]), dtype=torch.int32, device=length.device)
    step = max(1, (1 << 25) // max(width, 1))
    cut = offsets[torch.arange(0, n + step, step, device=length.device).clamp_(max=n)].tolist()
    col = torch.arange(width, device=length.device)[None, :]
    for k, a in enumerate(range(0, n, step)):
        b = min(n, a + step)
        frames[cut[k]:cut[k + 1]] = rows_of(a, b)[col < length[a:b, None]]
    return offsets, frames


def _zipf(n, s, count, g):
    """`count` ranks below n with weights (rank + 1)^-s."""
    cdf = torch.cumsum(torch.arange(1, n + 1, device=g.device, dtype=torch.float64) ** -s, 0)
    u = torch.rand(count, generator=g, device=g.device, dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=n - 1)


def _metrics(n, m, g):
    """Columns in turn: a time in ns, bytes, a count, and an unconstrained 64-bit value."""
    w = torch.empty(n, m, dtype=torch.int64, device=g.device)
    for j in range(m):
        if j % 4 == 0:
            w[:, j] = torch.randint(1000, 1_000_001, (n,), generator=g, device=g.device)
        elif j % 4 == 1:
            w[:, j] = torch.randint(0, (1 << 26) + 1, (n,), generator=g, device=g.device)
        elif j % 4 == 2:
            w[:, j] = 1
        else:
            w[:, j] = torch.randint(0, 1 << 62, (n,), generator=g, device=g.device) * 4 + 3
    return w


def _event_metrics(c, order, g, h):
    """Metrics of the events in their order.  The lengths of a filter's lists depend on them,
    so there they belong to the case's events, in units of the seed's clock; elsewhere they
    are the seed's."""
    if c["op"] in ("report", "filter"):
        unit = int(torch.randint(1, 100, (1,), generator=h, device=h.device))
        return _metrics(order.numel(), c["metrics"], g)[order] * unit
    return _metrics(order.numel(), c["metrics"], h)


def _deep(c, g, h):
    """Four entry frames, a 12-frame cycle repeated, then one of 64 tails of 1 to 8 frames;
    one event in a hundred is a single frame."""
    n, dev = c["events"], g.device
    pool = _frame_ids(c["ids"], h)
    length = torch.randint(c["dmin"], c["dmax"] + 1, (n,), generator=g, device=dev)
    k = torch.randint(1, 9, (n,), generator=g, device=dev)
    tail = torch.randint(0, 64, (n,), generator=g, device=dev)
    tails = torch.randint(0, c["ids"], (64, 8), generator=g, device=dev)
    single = torch.rand(n, generator=g, device=dev) < 0.01
    one = torch.randint(0, c["ids"], (n,), generator=g, device=dev)
    length = torch.where(single, torch.ones_like(length), length)
    order = _order(n, h)
    length, k, tail, single, one = (t[order] for t in (length, k, tail, single, one))
    col = torch.arange(c["dmax"], device=dev)[None, :]
    body = torch.where(col < 4, col, 4 + (col - 4).remainder(12))  # entry 0..3, cycle 4..15

    def rows(a, b):
        end = (length[a:b] - k[a:b])[:, None]
        q = (col - end).clamp(0, 7)
        ids = torch.where(col < end, body, tails[tail[a:b, None], q])
        return pool[torch.where(single[a:b, None], one[a:b, None], ids)]

    o, f = _flatten(length, c["dmax"], rows)
    return [(o, f, _event_metrics(c, order, g, h))]


def _traces(c, g, h):
    """The base trace and the batches that follow it, each (offsets, frames, metrics)."""
    if c["program"] == "deep":
        return _deep(c, g, h)
    p = _Program(c, g, h)
    T, n = c["templates"], c["events"]
    if c["op"] in ("merge", "activity"):  # the base runs 60% of the program, batches bring in the rest
        base = max(1, int(T * 0.6))
        part = max(1, (T - base) // (8 * c["batches"]))
        order = torch.randperm(T, generator=g, device=g.device)
        out = [order[_zipf(base, c["zipf"], n, g)]]
        for b in range(c["batches"]):
            seen = min(T - 1, base + b * part)
            ev = _zipf(seen, c["zipf"], c["batch"], g)
            fresh = torch.randint(seen, min(T, seen + part), (c["batch"],), generator=g, device=g.device)
            out.append(order[torch.where(torch.rand(c["batch"], generator=g, device=g.device) < 0.2, fresh, ev)])
    else:
        hot = (p.root < 8).nonzero().squeeze(1)
        cold = (p.root >= 8).nonzero().squeeze(1)
        if c["hot"] and hot.numel() and cold.numel():
            hot = hot[torch.randperm(hot.numel(), generator=g, device=g.device)]
            cold = cold[torch.randperm(cold.numel(), generator=g, device=g.device)]
            in_hot = torch.rand(n, generator=g, device=g.device) < c["hot"]
            out = [torch.where(in_hot, hot[_zipf(hot.numel(), c["zipf"], n, g)], cold[_zipf(cold.numel(), c["zipf"], n, g)])]
        else:
            out = [torch.randperm(T, generator=g, device=g.device)[_zipf(T, c["zipf"], n, g)]]
    orders = [_order(ev.numel(), h) for ev in out]
    return [p.take(ev[order]) + (_event_metrics(c, order, g, h),) for ev, order in zip(out, orders)]


def _flush(batch, c, g):
    """One activity flush: the batch's paths registered under IDs, every ID's record once,
    shuffled, 10% repeated IDs and 2% IDs that are not registered."""
    o, f, w = batch
    n, dev = c["batch"], g.device
    if c["dense"]:
        ids = 1_000_000 + torch.randperm(n, generator=g, device=dev)
        stray = 1_000_000 + n + torch.arange(max(1, n // 50), device=dev)
    else:  # an odd multiplier permutes 64-bit integers, so the IDs stay distinct
        ids = (1 + torch.randperm(n, generator=g, device=dev)) * 0x1E3779B97F4A7C15
        stray = (n + 1 + torch.arange(max(1, n // 50), device=dev)) * 0x1E3779B97F4A7C15
    again = ids[torch.randint(0, n, (n // 10,), generator=g, device=dev)]
    rec = torch.cat([ids, again, stray])
    rec = rec[torch.randperm(rec.numel(), generator=g, device=dev)].contiguous()
    return o, f, ids, rec, _metrics(rec.numel(), c["metrics"], g)


def _queries(c, base):
    """The first events' paths as queries, every 1,024th with its last frame changed (and
    so absent, but for a rare chance)."""
    o, f, _ = base
    dev, n, q = o.device, o.numel() - 1, c["batch"]
    at = torch.arange(q, device=dev) % n
    length = (o[1:] - o[:-1])[at]
    offsets = torch.zeros(q + 1, dtype=torch.int64, device=dev)
    torch.cumsum(length, 0, out=offsets[1:])
    src = torch.repeat_interleave(o[:-1][at] - offsets[:-1], length) + torch.arange(int(offsets[-1]), device=dev)
    frames = f[src].contiguous()
    odd = torch.arange(0, q, 1024, device=dev)
    odd = odd[length[odd] > 0]
    frames[offsets[odd + 1] - 1] ^= 0x5A5A5A5
    return offsets, frames


# ---- what is timed ------------------------------------------------------------------------


def _inputs(c, seed):
    """The device tensors of a case: "traces", and its "flushes" or "queries"."""
    g, h = _generators(c, seed)
    traces = _traces(c, g, h)
    got = {"traces": traces}
    if c["op"] == "activity":
        got["flushes"] = [_flush(b, c, h) for b in traces[1:]]
        got["traces"] = traces[:1]
    if c["op"] == "query":
        got["queries"] = _queries(c, traces[0])
    return got


def _as(t, unsigned):
    return t.view(torch.uint32 if t.dtype == torch.int32 else torch.uint64) if unsigned else t


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    s["traces"] = [(o, _as(f, c["unsigned"]), _as(w, c["unsigned"])) for o, f, w in s["traces"]]
    if c["op"] in ("query", "filter"):  # a program that looks things up keeps its tree
        s["tree"] = cct.build(*s.pop("traces")[0])
    return s


def _hot_and_small(tree, c):
    """Leaves above a thousandth of the whole time, and nodes whose time per byte (per unit
    time, with one metric) is below the threshold."""
    return (tree.hotspots(0, 1, 1000), tree.small_kernels(0, min(1, c["metrics"] - 1), 1, 67))


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "query":
        return state["tree"].query(*state["queries"])
    if op == "filter":
        return _hot_and_small(state["tree"], c) + (state["tree"].cpu_latency(0, min(1, c["metrics"] - 1), 1, 60),)
    tree = cct.build(*state["traces"][0], stats=op == "stats")
    if op == "stats":
        out = tree.stats()
    elif op == "report":
        out = [tree.bottom_up(), _hot_and_small(tree, c)]
    else:
        unmatched = []
        for b in state["traces"][1:]:
            tree.merge(*b)
        for b in state.get("flushes", ()):
            unmatched.append(tree.merge_activity(*b))
        out = tree.to_tensors()
        if op == "activity":
            out["unmatched"] = unmatched
    tree.free()
    return out


# ---- what a pass cannot do without -------------------------------------------------------


def _mean_length(c):
    if c["dmax"] > 250 and c["program"] == "layered":
        r = c["dmax"] - c["dmin"] + 1
        return (r - 1) / math.log(r) - 1.5 + c["dmin"]
    return (c["dmin"] + c["dmax"]) / 2


def _nodes(c):
    """About how many nodes the tree has: distinct paths expected under the popularity, and
    the share of a path's frames that is not shared with its neighbours."""
    n = c["events"] + (c["batches"] * c["batch"] if c["op"] in ("merge", "activity") else 0)
    if c["program"] == "deep":
        cells = 64 * 8 * (c["dmax"] - c["dmin"] + 1)
        return int(min(c["ids"], n / 100) + cells * (1 - math.exp(-n / cells)))
    T, z = c["templates"], c["zipf"]
    hot = min(1.0, 8 / c["roots"])
    pools = [(T, n)]
    if c["batches"]:  # batches draw a fifth of their events from paths new to them
        extra = min(0.4 * T / 8, 0.2 * n)
        pools = [(0.6 * T, n - extra), (extra, 3 * extra)]
    elif c["hot"] and hot < 1:
        pools = [(hot * T, c["hot"] * n), ((1 - hot) * T, (1 - c["hot"]) * n)]
    paths = 0.0
    for size, drawn in pools:
        w = np.arange(1, int(size) + 2) ** -z
        paths += float(np.sum(1 - np.exp(-drawn * w / w.sum())))
    share = 0.5 if c["dmax"] > 250 else 0.25
    return int(1 + paths * min(_mean_length(c), 9 + share * _mean_length(c)))


def work(case):
    c = case
    m, u, mean = c["metrics"], _nodes(c), _mean_length(c)
    read = c["events"] * (8 + 4 * mean + 8 * m)
    out = u * (12 + 16 * m)
    op = c["op"]
    if op == "merge":
        read += c["batches"] * c["batch"] * (8 + 4 * mean + 8 * m)
    elif op == "activity":  # registered paths and IDs, records' IDs and metrics
        read += c["batches"] * c["batch"] * (16 + 4 * mean + 1.12 * (8 + 8 * m))
    elif op == "stats":
        out = u * 2 * (8 + 8 * m + 16 * m + 8 * m + 8 * m)
    elif op == "report":  # a row per frame, ids of a third of the nodes
        out = min(u, c["ids"]) * (4 + 16 * m) + u * 8 // 3
    elif op == "query":
        read = c["batch"] * (8 + 4 * mean)
        out = c["batch"] * (8 + 16 * m)
    elif op == "filter":  # both sums of every node, three times, ids of a part of them
        read = 3 * u * 16
        out = u * 8
    return {"bytes": float(read + out), "flops": 0.0}


def tolerance(case):
    """Integers are exact; a mean is one float64 division, a deviation a conversion, a
    square root and a division of an exact integer (up to 2.5 units in the last place)."""
    return {"rel": 1e-15, "max": 2e-15} if case["op"] == "stats" else "exact"


# ---- the same outputs in plain torch -----------------------------------------------------


def _u32(t):
    return t.view(torch.int32).long() & 0xFFFFFFFF


def _levels(batches):
    """Walk all events down the tree together, a level at a time.  Returns per level the
    sorted keys (index of the parent in the level above << 32 | frame), and per event the
    level and index of the node its path ends on."""
    o = torch.cat([b[0][:-1] + sum(int(x[0][-1]) for x in batches[:i]) for i, b in enumerate(batches)])
    length = torch.cat([b[0][1:] - b[0][:-1] for b in batches])
    f = torch.cat([b[1].view(torch.int32) for b in batches])
    keys, at = [], torch.zeros_like(length)
    ev, cur, lvl = torch.arange(length.numel(), device=o.device), torch.zeros_like(length), 0
    while True:
        go = length[ev] > lvl
        at[ev[~go]] = cur[~go]
        ev, cur = ev[go], cur[go]
        if not ev.numel():
            return keys, length, at
        k, cur = torch.unique((cur << 32) | _u32(f[o[ev] + lvl]), return_inverse=True)
        keys.append(k)
        lvl += 1


def _up(values, parents, add):
    """Per-level values folded into their parents' level, deepest first."""
    for l in range(len(parents) - 1, -1, -1):
        add(values[l], parents[l], values[l + 1])
    return values


class _Exact:
    """The canonical tree of some batches, by its definition."""

    def __init__(self, batches, stats=False):
        keys, length, at = _levels(batches)
        dev, m = length.device, batches[0][2].shape[1]
        w = torch.cat([b[2].view(torch.int64) for b in batches])
        sizes = [1] + [k.numel() for k in keys]
        parents = [k >> 32 for k in keys]
        by_level = torch.argsort(length, stable=True)
        cut = torch.searchsorted(length[by_level], torch.arange(len(sizes) + 1, device=dev)).tolist()

        def at_end(v, fill=0, how=None):
            out = []
            for l, n in enumerate(sizes):
                e = by_level[cut[l]:cut[l + 1]]
                x = torch.full((n,) + v.shape[1:], fill, dtype=torch.int64, device=dev)
                if how == "min":
                    x.scatter_reduce_(0, at[e][:, None].expand(-1, v.shape[1]), v[e], "amin")
                else:
                    x.index_add_(0, at[e], v[e])
                out.append(x)
            return out

        add = lambda into, p, v: into.index_add_(0, p, v)  # noqa: E731
        low = lambda into, p, v: into.scatter_reduce_(0, p[:, None].expand(-1, v.shape[1]), v, "amin")  # noqa: E731
        total = _up([torch.ones(n, dtype=torch.int64, device=dev) for n in sizes], parents, add)
        ids = [torch.zeros(1, dtype=torch.int64, device=dev)]
        for p, size in zip(parents, total[1:]):  # preorder, siblings by ascending frame
            before = torch.cumsum(size, 0) - size
            first = torch.searchsorted(p, p)
            ids.append(ids[-1][p] + 1 + before - before[first])
        self.ids, self.keys, self.u = ids, keys, sum(sizes)
        self.subend = self._place([i + t for i, t in zip(ids, total)])
        self.excl = self._place(at_end(w))
        self.incl = self._place(_up(at_end(w), parents, add))
        self.parent = self._place([torch.full((1,), -1, dtype=torch.int64, device=dev)] + [ids[l][p] for l, p in enumerate(parents)])
        self.frame = self._place([torch.zeros(1, dtype=torch.int64, device=dev)] + [k & 0xFFFFFFFF for k in keys])
        self.depth = self._place([torch.full((n,), l, dtype=torch.int64, device=dev) for l, n in enumerate(sizes)])
        if stats:  # metrics below 2^32: a square is two 32-bit limbs
            one = torch.ones_like(w[:, :1])
            limbs = torch.cat([(w * w) & 0xFFFFFFFF, ((w * w) >> 32) & 0xFFFFFFFF], 1)
            top = (1 << 63) - 1
            self.stat = {"count_excl": at_end(one), "count_incl": _up(at_end(one), parents, add), "min_excl": at_end(w, top, "min"),
                         "min_incl": _up(at_end(w, top, "min"), parents, low), "sumsq_excl": at_end(limbs),
                         "sumsq_incl": _up(at_end(limbs), parents, add)}
            self.stat = {k: self._place(v) for k, v in self.stat.items()}

    def _place(self, per_level):
        out = torch.empty((self.u,) + per_level[0].shape[1:], dtype=torch.int64, device=per_level[0].device)
        for i, v in zip(self.ids, per_level):
            out[i] = v
        return out

    def tensors(self):
        return {"parent": self.parent.to(torch.int32), "frame": self.frame.to(torch.int32), "depth": self.depth.to(torch.int32),
                "excl": self.excl, "incl": self.incl}

    def statistics(self):
        s, out = self.stat, {}
        m = self.excl.shape[1]
        for k, total in (("excl", self.excl), ("incl", self.incl)):
            n = s["count_" + k][:, 0]
            out["count_" + k] = n
            low = s["min_" + k].clone()
            low[n == 0] = -1  # all bits set: no sample
            out["min_" + k] = low
            lo, hi = s["sumsq_" + k][:, :m], s["sumsq_" + k][:, m:]
            out["sumsq_" + k] = torch.stack([lo + (hi << 32), (hi + (lo >> 32)) >> 32], 2)
            count = n.cpu().numpy().astype(object)[:, None]
            t = total.cpu().numpy().astype(object)
            sq = lo.cpu().numpy().astype(object) + (hi.cpu().numpy().astype(object) << 32)
            some = n.cpu().numpy()[:, None].astype(np.float64)
            with np.errstate(all="ignore"):
                spread = np.sqrt((count * sq - t * t).astype(np.float64))
                out["mean_" + k] = torch.from_numpy(np.where(some > 0, t.astype(np.float64) / some, np.nan))
                out["std_" + k] = torch.from_numpy(np.where(some > 0, spread / some, np.nan))
        return out

    def filter(self, num, op, p, q, den, leaves=False):
        """Nodes with incl[num] / den above (below) p / q, in 64-bit products."""
        a, b = self.incl[:, num] * q, den * p
        hit = a > b if op > 0 else a < b
        if leaves:
            hit &= self.subend == torch.arange(1, self.u + 1, device=hit.device)
        return hit.nonzero().squeeze(1)

    def find(self, offsets, frames):
        """Node ids of query paths, -1 where there is none."""
        length = offsets[1:] - offsets[:-1]
        f = frames.view(torch.int32)
        out = torch.full_like(length, -1)
        q, cur, lvl = torch.arange(length.numel(), device=length.device), torch.zeros_like(length), 0
        while q.numel():
            done = length[q] == lvl
            out[q[done]] = self.ids[lvl][cur[done]]
            q, cur = q[~done], cur[~done]
            if lvl == len(self.keys) or not q.numel():
                return out
            want = (cur << 32) | _u32(f[offsets[q] + lvl])
            cur = torch.searchsorted(self.keys[lvl], want).clamp_(max=self.keys[lvl].numel() - 1)
            here = self.keys[lvl][cur] == want
            q, cur, lvl = q[here], cur[here], lvl + 1
        return out


def _by_frame(o, f, w):
    """Bottom-up view from the events: sums by last frame, and by every frame of a path once."""
    length = o[1:] - o[:-1]
    frames = torch.unique(_u32(f))
    out = {"frames": frames.to(torch.int32)}
    full = length > 0
    last = torch.searchsorted(frames, _u32(f)[o[1:][full] - 1])
    z = torch.zeros(frames.numel(), w.shape[1], dtype=torch.int64, device=w.device)
    out["excl"] = z.clone().index_add_(0, last, w[full])
    out["incl"] = z
    for a in range(0, length.numel(), 1 << 18):
        b = min(length.numel(), a + (1 << 18))
        ev = torch.repeat_interleave(torch.arange(a, b, device=o.device), length[a:b])
        pair = torch.unique((ev << 32) | _u32(f[int(o[a]):int(o[b])]))
        z.index_add_(0, torch.searchsorted(frames, pair & 0xFFFFFFFF), w[pair >> 32])
    return out


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    op, unmatched = c["op"], []
    for o, f, ids, rec, w in s.get("flushes", ()):
        order = torch.argsort(ids)
        at = torch.searchsorted(ids[order], rec).clamp_(max=ids.numel() - 1)
        reg = order[at]
        hit = ids[reg] == rec
        unmatched.append(int((~hit).sum()))
        sums = torch.zeros(ids.numel(), w.shape[1], dtype=torch.int64, device=w.device).index_add_(0, reg[hit], w[hit])
        named = torch.zeros(ids.numel(), dtype=torch.bool, device=w.device)
        named[reg[hit]] = True
        if not bool(named.all()):
            return None  # every registered path has a record in these flushes
        s["traces"].append((o, f, sums))
    t = _Exact(s["traces"], stats=op == "stats")
    j = min(1, c["metrics"] - 1)
    if op == "stats":
        if c["metrics"] > 3:
            return None  # the 64-bit column's squares need more than two limbs
        return t.statistics()
    hot = t.filter(0, +1, 1, 1000, t.incl[0, 0].expand(t.u), leaves=True) if op in ("report", "filter") else None
    small = t.filter(0, -1, 1, 67, t.incl[:, j]) if op in ("report", "filter") else None
    if op == "report":
        return [_by_frame(*s["traces"][0]), (hot, small)]
    if op == "filter":
        return (hot, small, t.filter(0, +1, 1, 60, t.incl[:, j]))
    if op == "query":
        ids = t.find(*s["queries"])
        ok = (ids >= 0)[:, None]
        zero = torch.zeros((), dtype=torch.int64, device=ids.device)
        return ids, torch.where(ok, t.excl[ids], zero), torch.where(ok, t.incl[ids], zero)
    out = t.tensors()
    if op == "activity":
        out["unmatched"] = unmatched
    return out
