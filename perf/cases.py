"""Timed cases of the mini-batch path: the calls a TGNN training loop makes, through the package's public functions.

A case names its kind (which calls one pass makes), the shape of the synthetic data and the sizes of the call. The
shapes are those of the datasets that the workloads of this package stand for (Wikipedia, Reddit, Flights, GDELT), with
GDELT's event count scaled down so that inputs are made in a moment; all inputs are drawn on the GPU from the seed.
Everything here moves whole values (ids, timestamps, feature bytes, integer weights): results are compared exactly.
"""
import numpy as np
import torch

import paper_2402_05396_amd as T

POLICY = {"recent": T.RECENT, "uniform": T.UNIFORM, "weighted": T.WEIGHTED, "inverse_timespan": T.INVERSE_TIMESPAN}


def listed():
    return [
        # One mini-batch of a 1-layer model on a small graph: 600 edges, their endpoints and negatives, 10 neighbors
        # each with their edge rows. The smallest call of a training loop; launches and host work count.
        dict(name="wiki_recent_rows", kind="finder", nodes=9000, destinations=1000, skew=1.2, events=160_000, span=2_500_000,
             policy="recent", k=10, hops=1, m=0, roots=1800, dtype="float32", dim=172),
        # Two hops of the uniform finder with half-precision edge rows (344 bytes, no padding): a 2-layer model on Reddit.
        dict(name="reddit_uniform_rows", kind="finder", nodes=11_000, destinations=1000, skew=1.2, events=670_000, span=2_700_000,
             policy="uniform", k=10, hops=2, m=0, roots=6000, dtype="float16", dim=172),
        # Two hops of n-of-m selection by given edge weights with short rows: adaptive sampling on a dense flight graph.
        dict(name="flights_weighted_rows", kind="finder", nodes=13_000, destinations=0, skew=0.9, events=1_900_000, span=10_000_000,
             policy="weighted", k=10, hops=2, m=25, roots=4000, dtype="float32", dim=16),
        # The heuristic finder whose weights depend on the query time: it has to look at whole lists.
        dict(name="flights_inverse_timespan", kind="finder", nodes=13_000, destinations=0, skew=0.9, events=1_900_000, span=10_000_000,
             policy="inverse_timespan", k=10, hops=2, m=0, roots=4000, dtype="", dim=0),
        # Neighbor finding alone at the largest batch: 12 000 roots, 132 000 queries over long lists with many ties.
        dict(name="gdelt_recent_finder", kind="finder", nodes=17_000, destinations=0, skew=1.0, events=40_000_000, span=20_000_000,
             policy="recent", k=10, hops=2, m=0, roots=12_000, dtype="", dim=0),
        # Slicing the edge rows of that batch out of a device table with a padded pitch (372 bytes of 384).
        dict(name="gdelt_edge_gather", kind="gather", rows=8_000_000, dim=186, dtype="float16", padded=True, skew=0.0, n=1_320_000),
        # Half-precision node rows of odd width (826 bytes, so rows start at any even address) from a device table.
        dict(name="gdelt_half_node_gather", kind="gather", rows=17_000, dim=413, dtype="float16", padded=False, skew=1.0, n=1_332_000),
        # Node rows through the device cache over pinned host memory, a fifth of the rows resident, requests counted
        # for the epoch's replacement as in the paper's Algorithm 3.
        dict(name="gdelt_node_lookup", kind="lookup", rows=17_000, dim=413, skew=1.0, n=1_332_000, ratio=0.2, counting=True),
        # Building the graph of an event stream that arrives in time order (every event in both directions).
        dict(name="gdelt_tcsr_build", kind="build", nodes=17_000, destinations=0, skew=1.0, events=32_000_000, span=16_000_000, sorted=True),
        # Building a smaller graph from events in no order, as when logs are merged.
        dict(name="reddit_tcsr_build_unsorted", kind="build", nodes=11_000, destinations=1000, skew=1.2, events=670_000, span=2_700_000,
             sorted=False),
        # The adaptive sampler's second layer around its network: candidates of 40 000 roots, their frequency and
        # identity encodings, and the selection of 10 of 25 by one weight per candidate.
        dict(name="flights_adaptive_window", kind="window", nodes=13_000, destinations=0, skew=0.9, events=1_900_000, span=10_000_000,
             roots=40_000, m=25, k=10),
        # One iteration of importance-based batch selection: scores of the last batch stored, the next batch drawn,
        # the scores read. Three small launches over a million training edges.
        dict(name="selector_step", kind="selector", edges=1_000_000, batch=2000),
    ]


def _log(rng, low, high):
    return int(round(low * (high / low) ** rng.random()))


def draw(rng):
    kind = rng.choice(["finder", "finder", "finder", "finder", "gather", "gather", "lookup", "build", "window", "selector"])
    if kind in ("finder", "build", "window"):
        events = _log(rng, 20_000, 32_000_000 if kind != "window" else 4_000_000)
        nodes = _log(rng, 1000, 20_000)
        graph = dict(nodes=nodes, destinations=rng.choice([0, max(1, nodes // 9)]), skew=round(rng.uniform(0.7, 1.2), 3), span=_log(rng, 50_000, 100_000_000))
    if kind == "finder":
        policy = rng.choice(["recent", "uniform", "weighted", "inverse_timespan"])
        k, hops = rng.choice([5, 10, 10, 10, 15, 20, 32]), rng.choice([1, 2, 2])
        roots = min(_log(rng, 600, 12_000), 1_300_000 // k ** hops)
        dtype = rng.choice(["", "float16", "float32"])
        if policy == "inverse_timespan":   # reads whole lists: kept to the listed case's order of work
            events, roots, k, hops = min(events, 1_500_000), min(roots, 3000), min(k, 10), hops
        if dtype:
            events = min(events, 4_000_000)
        dim = rng.choice([16, 32, 100, 172, 186, rng.randrange(8, 266)]) if dtype else 0
        while dim and roots * k ** hops * dim * 4 > 1_200_000_000:
            roots //= 2
        return dict(graph, kind=kind, events=events, policy=policy, k=k, hops=hops, m=max(k, rng.randrange(k, 33)) if policy == "weighted" else 0,
                    roots=max(1, roots), dtype=dtype, dim=dim)
    if kind == "build":
        ordered = rng.random() < 0.6
        return dict(graph, kind=kind, events=events if ordered else min(events, 3_000_000), sorted=ordered)
    if kind == "window":
        m = rng.randrange(8, 50)
        return dict(graph, kind=kind, events=events, roots=min(_log(rng, 600, 60_000), 40_000_000 // (m * m)), m=m, k=rng.randrange(4, m))
    if kind == "selector":
        return dict(kind=kind, edges=_log(rng, 20_000, 4_000_000), batch=_log(rng, 200, 8000))
    dim = rng.choice([16, 100, 172, 186, 266, 413, rng.randrange(8, 500)])
    if kind == "gather":
        dtype = rng.choice(["float16", "float32"])
        size = 2 if dtype == "float16" else 4
        return dict(kind=kind, rows=min(_log(rng, 5000, 8_000_000), 3_000_000_000 // (dim * size)), dim=dim, dtype=dtype, padded=rng.random() < 0.4,
                    skew=rng.choice([0.0, 1.0]), n=min(_log(rng, 1800, 1_300_000), 1_100_000_000 // (dim * size)))
    return dict(kind=kind, rows=min(_log(rng, 1000, 100_000), 28_000_000 // (dim * 4)), dim=dim, skew=round(rng.uniform(0.8, 1.2), 3),
                n=min(_log(rng, 1800, 1_300_000), 2_100_000_000 // (dim * 4)), ratio=rng.choice([0.1, 0.2, 0.3, 0.5]), counting=rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _power_law(gen, n, skew, size):
    """`size` ids of [0, n), the id of rank r drawn with a probability proportional to (r + 1)^-skew, ranks in random order."""
    if skew == 0.0:
        return torch.randint(0, n, (size,), generator=gen, device="cuda", dtype=torch.int32)
    cdf = torch.cumsum(torch.arange(1, n + 1, device="cuda", dtype=torch.float64) ** -skew, 0)
    u = torch.rand(size, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=n - 1)
    return torch.randperm(n, generator=gen, device="cuda").to(torch.int32)[rank]


def _events(gen, case):
    """An event stream in both directions, in time order: entries 2i and 2i + 1 are event i's."""
    n, dest, e = case["nodes"], case["destinations"], case["events"]
    u = _power_law(gen, n - dest, case["skew"], e)
    v = _power_law(gen, dest, case["skew"], e) + (n - dest) if dest else _power_law(gen, n, case["skew"], e)
    ts = torch.randint(0, case["span"], (e,), generator=gen, device="cuda", dtype=torch.int64).sort().values
    src, dst = torch.stack([u, v], 1).reshape(-1), torch.stack([v, u], 1).reshape(-1)
    eid = torch.arange(e, dtype=torch.int32, device="cuda").repeat_interleave(2)
    return u, v, ts, (src, dst, ts.repeat_interleave(2), eid)


def _queries(gen, case, u, v, ts):
    """Roots of a link-prediction batch from the last third of the stream: sources, destinations, negative destinations."""
    e, r = case["events"], case["roots"]
    pick = torch.randint(int(0.7 * e), e, ((r + 2) // 3,), generator=gen, device="cuda")
    neg = torch.randint(case["nodes"] - case["destinations"] if case["destinations"] else 0, case["nodes"], pick.shape,
                        generator=gen, device="cuda", dtype=torch.int32)
    return torch.cat([u[pick], v[pick], neg])[:r].contiguous(), ts[pick].repeat(3)[:r].contiguous()


def _table(gen, rows, dim, dtype, padded=False):
    """A device table of normal values; padded: rows start at multiples of 64 elements."""
    pitch = (dim + 63) // 64 * 64 if padded else dim
    return torch.randn((rows, pitch), generator=gen, device="cuda", dtype=getattr(torch, dtype))[:, :dim]


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind in ("finder", "build", "window"):
        u, v, ts, entries = _events(gen, case)
        if kind == "build":
            if not case["sorted"]:
                order = torch.randperm(2 * case["events"], generator=gen, device="cuda")
                entries = tuple(x[order].contiguous() for x in entries)
            return dict(case=case, entries=entries)
        roots, times = _queries(gen, case, u, v, ts)
        s = dict(case=case, graph=T.tcsr_build(*entries, case["nodes"]), roots=roots, times=times)
        if kind == "window":
            s["weight"] = torch.randint(1, 65536, (case["roots"], case["m"]), generator=gen, device="cuda", dtype=torch.int32)
            return s
        s["table"] = _table(gen, case["events"], case["dim"], case["dtype"]) if case["dtype"] else None
        z = torch.randn(case["events"], generator=gen, device="cuda")
        s["weight"] = torch.clamp(torch.round(torch.exp(z) * 4096), 1, 65536).to(torch.int32) if case["policy"] == "weighted" else None
        if case["policy"] == "inverse_timespan":   # the first call of this policy on a graph lays out its timestamps
            T.sample_temporal(s["graph"], roots[:1], times[:1], 1, 1, T.INVERSE_TIMESPAN, 0)
        return s
    if kind == "gather":
        return dict(case=case, table=_table(gen, case["rows"], case["dim"], case["dtype"], case["padded"]), ids=_gather_ids(gen, case))
    if kind == "lookup":
        host = _table(gen, case["rows"], case["dim"], "float32").cpu().pin_memory()
        epoch, ids = _gather_ids(gen, case), _gather_ids(gen, case)
        capacity = int(case["rows"] * case["ratio"])
        cache = T.cache_init(host, capacity, None, seed=seed, staging_rows=case["rows"] - capacity)
        # an epoch of counted requests decides the content, as in a training loop
        T.cache_count_accesses(cache)
        T.cache_prefetch(cache, epoch)
        T.cache_epoch_end(cache, capacity)
        T.cache_count_accesses(cache, case["counting"])
        return dict(case=case, cache=cache, ids=ids, hit_miss=torch.zeros(2, dtype=torch.int64, device="cuda"))
    scores = torch.randint(0, 6554, (case["edges"],), generator=gen, device="cuda", dtype=torch.int32)
    batch = torch.randint(0, case["edges"], (case["batch"],), generator=gen, device="cuda", dtype=torch.int32)
    new = torch.randint(0, 6554, (case["batch"],), generator=gen, device="cuda", dtype=torch.int32)
    return dict(case=case, selector=T.selector_init(scores), batch=batch, new=new)


def _gather_ids(gen, case):
    """Requested rows: by popularity (its order is the same in every batch), one in thirty a padding slot (id -1)."""
    rows, n = case["rows"], case["n"]
    if case["skew"] == 0.0:
        ids = torch.randint(0, rows, (n,), generator=gen, device="cuda", dtype=torch.int32)
    else:
        cdf = torch.cumsum(torch.arange(1, rows + 1, device="cuda", dtype=torch.float64) ** -case["skew"], 0)
        rank = torch.searchsorted(cdf, torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]).clamp_(max=rows - 1)
        order = torch.randperm(rows, generator=_generator(rows), device="cuda").to(torch.int32)
        ids = order[rank]
    ids[torch.rand(n, generator=gen, device="cuda") < 1 / 30] = -1
    return ids


# ---- one pass -----------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "finder":
        policy = POLICY[case["policy"]]
        if s["table"] is None:
            return T.sample_temporal(s["graph"], s["roots"], s["times"], case["k"], case["hops"], policy, 42, m=case["m"], edge_weight=s["weight"])
        return T.sample_temporal_rows(s["graph"], s["roots"], s["times"], case["k"], case["hops"], policy, 42, s["table"], m=case["m"],
                                      edge_weight=s["weight"])
    if kind == "gather":
        return T.gather_features(s["table"], s["ids"])
    if kind == "lookup":
        s["hit_miss"].zero_()
        return T.cache_lookup(s["cache"], s["ids"], hit_miss=s["hit_miss"]), s["hit_miss"]
    if kind == "build":
        return T.tcsr_view(T.tcsr_build(*s["entries"], case["nodes"]))
    if kind == "window":
        cand = T.sample_temporal(s["graph"], s["roots"], s["times"], case["m"], 1, T.RECENT, 0)[0]
        freq, identity = T.candidate_encodings(cand["nbr"], cand["count"])
        sel, count, kept = T.select_weighted(s["weight"], cand["count"], case["k"], 42, 1, candidates=cand)
        return cand, freq, identity, sel, count, kept
    T.selector_update(s["selector"], s["batch"], s["new"])
    drawn = T.selector_draw(s["selector"], case["batch"], 42, 7)
    return drawn, T.selector_scores(s["selector"], want_total=False)[0]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _distinct(rows, skew, n):
    """Expected number of distinct rows among n requests."""
    p = np.full(rows, 1.0 / rows) if skew == 0.0 else np.arange(1, rows + 1, dtype=np.float64) ** -skew
    return float(np.sum(-np.expm1(-n * p / p.sum())))


def work(case):
    kind = case["kind"]
    if kind == "finder":
        slots = sum(case["roots"] * case["k"] ** (h + 1) for h in range(case["hops"]))
        queries = sum(case["roots"] * case["k"] ** h for h in range(case["hops"]))
        size = {"": 0, "float16": 2, "float32": 4}[case["dtype"]] * case["dim"]
        taken = slots * case["m"] // case["k"] if case["m"] else slots              # records looked at
        entries = 2 * case["events"]
        read = 16 * min(taken, entries) + (4 * min(taken, case["events"]) if case["m"] else 0) + 12 * case["roots"]
        ops = 0
        if case["policy"] == "inverse_timespan":
            # every entry of a list is weighed per query; a root is met in proportion to its degree
            p = np.arange(1, case["nodes"] - case["destinations"] + 1, dtype=np.float64) ** -case["skew"]
            p /= p.sum()
            read += 8 * entries
            ops = 8.0 * queries * (1.0 if case["destinations"] else 2.0) * case["events"] * float(np.sum(p * p)) * 0.5
        distinct = case["events"] * -np.expm1(-slots / case["events"])              # edge rows asked for at least once
        return {"bytes": float(read + 16 * slots + 4 * queries + size * (slots + distinct)), "flops": ops}
    if kind == "gather":
        size = case["dim"] * (2 if case["dtype"] == "float16" else 4)
        return {"bytes": size * (case["n"] + _distinct(case["rows"], case["skew"], case["n"])) + 4.0 * case["n"], "flops": 0}
    if kind == "lookup":
        return {"bytes": case["dim"] * 4 * (case["n"] + _distinct(case["rows"], case["skew"], case["n"])) + 4.0 * case["n"], "flops": 0}
    if kind == "build":   # 20 bytes of input per entry, the graph's record, the plain view
        return {"bytes": 2.0 * case["events"] * (20 + 16 + 16) + 8 * case["nodes"], "flops": 0}
    if kind == "window":
        r, m, k = case["roots"], case["m"], case["k"]
        return {"bytes": float(r * (12 + m * (16 + 16 + 4 + m + 4) + k * 20 + 8)), "flops": 0}
    return {"bytes": 8.0 * case["edges"] + 12.0 * case["batch"], "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    kind = case["kind"]
    gen = _generator(seed)
    if kind == "gather":
        table = _table(gen, case["rows"], case["dim"], case["dtype"], case["padded"])
        return _rows64(table, _gather_ids(gen, case))
    if kind == "lookup":
        table = _table(gen, case["rows"], case["dim"], "float32")
        _gather_ids(gen, case)   # the epoch's requests
        return _rows64(table, _gather_ids(gen, case)), None
    if kind == "finder" and case["policy"] == "recent" and case["dtype"]:
        u, v, ts, (src, dst, ts2, eid) = _events(gen, case)
        roots, times = _queries(gen, case, u, v, ts)
        table = _table(gen, case["events"], case["dim"], case["dtype"])
        key, order = torch.sort(src.to(torch.int64) * case["span"] + ts2, stable=True)
        rows, none = [], dict(nbr=None, eid=None, ts=None, count=None)
        for _ in range(case["hops"]):
            base = roots.to(torch.int64) * case["span"]
            lo, hi = torch.searchsorted(key, base), torch.searchsorted(key, base + times)
            at = hi[:, None] - 1 - torch.arange(case["k"], device="cuda")[None, :]
            have = (at >= lo[:, None]) & (roots >= 0)[:, None]
            at = order[at.clamp_(min=0)]
            rows.append(_rows64(table, torch.where(have, eid[at], -1).reshape(-1)))
            roots = torch.where(have, dst[at], -1).reshape(-1)
            times = torch.where(have, ts2[at], 0).reshape(-1)
        return [none] * case["hops"], rows
    return None


def _rows64(table, ids):
    out = table[ids.clamp(min=0).to(torch.int64)].to(torch.float64)
    out[ids < 0] = 0
    return out
