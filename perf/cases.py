"""The work a user of this library has it do, as cases that can be timed and whose results can be compared.

Four kinds of case, all through the public entry points:

  hop     one tns_run over a batch of queries: one layer of neighbours, padded and dense results
  khop    one tns_run_khop from a training mini-batch (or an epoch) of roots
  ingest  a stream that arrives in batches: every batch is added to a store on the GPU, then its own events are
          sampled (the continuous-learning loop of section 3 of the paper)
  cache   one batch of ids through the vectorised feature cache

Streams follow the synthetic recipes of workloads.py (uniform or Zipf node ids, |V| = n / 16, sorted times), drawn
on the GPU; queries are the last events of the stream, each asking for the neighbours of its source before its time.
Everything is an int32 id or a copied fp32 value, so results are compared for equality.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2311_17410_amd import binding as B
from paper_2311_17410_amd import cache_binding as KB

DEV = torch.device("cuda", 0)
INGEST_BATCH = 1 << 17          # edges per batch when a store is built beforehand
POLICIES = {"recent": B.TNS_POLICY_RECENT, "uniform": B.TNS_POLICY_UNIFORM}
CACHE_POLICIES = {"lru": KB.TNS_CACHE_LRU, "lfu": KB.TNS_CACHE_LFU, "fifo": KB.TNS_CACHE_FIFO}
CACHE_BATCHES = 8               # different id batches a cache case goes round
CACHE_WARM = 4                  # fetches before the first timed one


# ---- the cases -----------------------------------------------------------------------------------

def _hop(edges, queries, **kw):
    c = dict(kind="hop", edges=edges, queries=queries, fanout=10, policy="recent", layout="blocks", ids="uniform", tau=48,
             window=0.0, inclusive=0, instances=1, static=False)
    c.update(kw)
    return c


def _khop(edges, queries, **kw):
    c = dict(kind="khop", edges=edges, queries=queries, fanouts="10,10", policy="recent", layout="blocks", ids="uniform", tau=48,
             window=0.0, padded=True)
    c.update(kw)
    return c


def _ingest(batch, batches, **kw):
    c = dict(kind="ingest", batch=batch, batches=batches, nodes=max(batch * batches // 16, 2), fanout=10, ids="uniform", tau=48)
    c.update(kw)
    return c


def _cache(num_ids, batch, **kw):
    c = dict(kind="cache", num_ids=num_ids, batch=batch, dim=172, ratio=0.01, policy="lru", zipf=1.05)
    c.update(kw)
    return c


def listed():
    return [
        # a training mini-batch of a two-layer model: 600 events, most recent neighbours; launches and latency count
        dict(_khop(1 << 24, 600), name="khop 600 recent"),
        # the largest mini-batch the paper trains with, neighbours drawn uniformly
        dict(_khop(1 << 24, 4000, policy="uniform"), name="khop 4000 uniform"),
        # a whole epoch's roots through two layers with a window of a quarter of the time span, dense results only
        dict(_khop(1 << 22, 1 << 20, layout="prefix", window=0.25, padded=False), name="khop 1M window prefix"),
        # the smallest workload of this repository: one call on a small graph (the serving entry point without a workspace)
        dict(_hop(1 << 10, 1 << 10, static=True), name="hop 1k static"),
        # one layer over a million queries, in the layout made for nodes of a few dozen edges
        dict(_hop(1_500_007, 1_000_003, layout="prefix"), name="hop 1M prefix"),
        # power-law degrees: hubs of hundreds of thousands of edges in blocks of up to 8192, uniform policy
        dict(_hop(1 << 23, 1 << 23, policy="uniform", ids="zipf", tau=8192), name="hop 8M zipf uniform"),
        # many independent small graphs in one call, windowed
        dict(_hop(1 << 16, 1 << 16, instances=256, window=0.25), name="hop 256 graphs window"),
        # ingestion in batches of the paper's size, each followed by the sampling of its events
        dict(_ingest(100_000, 32, nodes=1 << 18), name="ingest 100k batches"),
        # the same for a stream whose batches are single mini-batches, with power-law ids
        dict(_ingest(2000, 64, ids="zipf", nodes=1 << 16), name="ingest 2k batches"),
        # features of one mini-batch's sampled neighbourhood (600 roots and two layers of ten)
        dict(_cache(1 << 22, 66_600), name="cache 66k lru"),
        # features of a large batch; access counts instead of recency
        dict(_cache(1 << 24, 1 << 20, policy="lfu"), name="cache 1M lfu"),
        # an epoch of a large stream in one call
        dict(_hop(1 << 26, 1 << 26), name="hop 64M recent"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["hop", "hop", "khop", "khop", "ingest", "cache"])
    ids = rng.choice(["uniform", "uniform", "zipf"])
    tau = 48 if ids == "uniform" else rng.choice([48, 8192])
    policy = rng.choice(["recent", "uniform"])
    window = rng.choice([0.0, 0.0, round(rng.uniform(0.02, 0.5), 3)])
    layout = rng.choice(["blocks", "blocks", "prefix"])
    most = 1 << (22 if layout == "prefix" else 24)       # a store in the prefix layout is built on the host
    if kind == "hop":
        edges = _log_uniform(rng, 1 << 10, most)
        instances = rng.choice([1, 1, 1, rng.randint(2, 64)])
        return _hop(max(edges // instances, 64), max(int(edges * rng.uniform(0.2, 1.0)) // instances, 1), instances=instances,
                    fanout=rng.choice([5, 10, 10, 15, 20]), policy=policy, layout=layout, ids=ids, tau=tau, window=window,
                    inclusive=rng.choice([0, 0, 1]))
    if kind == "khop":
        edges = _log_uniform(rng, 1 << 18, most)
        return _khop(edges, min(_log_uniform(rng, 200, 1 << 20), edges), fanouts=rng.choice(["10,10", "10,10", "15,10", "10", "5,5,5"]),
                     policy=policy, layout=layout, ids=ids, tau=tau, window=window, padded=rng.choice([True, False]))
    if kind == "ingest":
        batch = _log_uniform(rng, 600, 300_000)
        batches = rng.randint(8, 40)
        return _ingest(batch, batches, ids=ids, tau=tau, nodes=_log_uniform(rng, 1 << 10, 1 << 20))
    return _cache(_log_uniform(rng, 1 << 16, 1 << 23), _log_uniform(rng, 600, 1 << 20), dim=rng.choice([32, 100, 128, 172, 173]),
                  ratio=round(rng.uniform(0.005, 0.1), 4), policy=rng.choice(["lru", "lru", "lfu", "fifo"]))


# ---- inputs --------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _zipf_ids(g, count, n, s):
    """`count` ids of 0 .. n-1 whose ranks follow Zipf(s); the ranks are dealt to the ids at random."""
    cdf = torch.arange(1, n + 1, dtype=torch.float64, device=DEV).pow_(-s).cumsum_(0)
    cdf /= cdf[-1].clone()
    deal = torch.randperm(n, generator=g, device=DEV)
    u = torch.rand(count, dtype=torch.float64, generator=g, device=DEV)
    return deal[torch.searchsorted(cdf, u).clamp_(max=n - 1)].to(torch.int32)


def _stream(g, edges, nodes, ids):
    """src, dst, ts of `edges` events in time order."""
    if ids == "zipf":
        src, dst = _zipf_ids(g, edges, nodes, 1.1), _zipf_ids(g, edges, nodes, 1.1)
        ts = torch.randn(edges, generator=g, device=DEV)
    else:
        src, dst = (torch.randint(0, nodes, (edges,), dtype=torch.int32, generator=g, device=DEV) for _ in range(2))
        ts = torch.rand(edges, generator=g, device=DEV)
    return src, dst, ts.sort().values


def _nodes(edges):
    return max(edges // 16, 2)


def _store(case, g, fanout):
    """The plan with its store built, and the events of every instance."""
    nodes, instances = _nodes(case["edges"]), case.get("instances", 1)
    prefix = case["layout"] == "prefix"
    plan = B.Plan(nodes, fanout, POLICIES[case["policy"]], case["tau"], instances, inclusive_end=case.get("inclusive", 0), seed=11,
                  flags=B.TNS_FLAG_PREFIX_LAYOUT if prefix else B.TNS_FLAG_DEVICE_INGEST)
    step = INGEST_BATCH if instances == 1 and case["edges"] >= 8 * INGEST_BATCH else max(case["edges"] // 8, 1)
    events = []
    for i in range(instances):
        src, dst, ts = _stream(g, case["edges"], nodes, case["ids"])
        host = [t.cpu().numpy() for t in (src, dst, ts)] if prefix else None
        for lo in range(0, case["edges"], step):
            part = slice(lo, min(lo + step, case["edges"]))
            if prefix:
                plan.add_edges(*(a[part] for a in host), instance=i)
            else:
                plan.add_edges_device(src[part], dst[part], ts[part], instance=i)
        events.append((src, ts))
    plan.commit()
    return plan, events


def _queries(case, events):
    """The last events of every instance as queries: targets, window starts (None: unbounded), window ends, instance offsets."""
    k = min(case["queries"], case["edges"])
    targets = torch.cat([src[-k:] for src, _ in events])
    t_end = torch.cat([ts[-k:] for _, ts in events])
    t_start = None
    if case["window"]:
        t_start = t_end - torch.cat([(case["window"] * (ts[-1] - ts[0])).expand(k) for _, ts in events])
    offsets = torch.arange(len(events) + 1, dtype=torch.int64, device=DEV) * k if len(events) > 1 else None
    return targets, t_start, t_end, offsets


def _outputs(cap, fanout, padded):
    """Result buffers of one hop for at most `cap` queries; what a pass does not write stays zero."""
    new = lambda n, dt: torch.zeros(n, dtype=dt, device=DEV)  # noqa: E731
    i32, f32, i64 = torch.int32, torch.float32, torch.int64
    out = dict(rowptr=new(cap + 1, i64), cmp_nbr=new(cap * fanout, i32), cmp_eid=new(cap * fanout, i32), cmp_ts=new(cap * fanout, f32))
    if padded:
        out.update(nbr=new(cap * fanout, i32), eid=new(cap * fanout, i32), ts=new(cap * fanout, f32), count=new(cap, i32))
    return out


def prepare(case, seed):
    g = _generator(seed)
    if case["kind"] == "hop":
        plan, events = _store(case, g, case["fanout"])
        targets, t_start, t_end, offsets = _queries(case, events)
        out = _outputs(targets.numel(), case["fanout"], True)
        results = dict(out)
        if not case["static"]:
            out["workspace"] = torch.zeros(B.tns_workspace(plan.handle, targets.numel()), dtype=torch.uint8, device=DEV)
        return dict(case=case, plan=plan, queries=(targets, t_start, t_end, offsets), out=out, results=results)
    if case["kind"] == "khop":
        fanouts = [int(f) for f in case["fanouts"].split(",")]
        plan, events = _store(case, g, fanouts[0])
        targets, t_start, t_end, _ = _queries(case, events)
        ts = events[0][1]
        delta = float(case["window"] * (ts[-1] - ts[0])) if case["window"] else math.inf
        hops, cap = [], targets.numel()
        for f in fanouts:
            hops.append(_outputs(cap, f, case["padded"]))
            cap *= f
        names = [n for n, _ in B.tns_hop_buffers._fields_]
        pointers = [{n: h[n].data_ptr() if n in h else 0 for n in names} for h in hops]
        workspace = torch.zeros(B.tns_workspace_khop(plan.handle, fanouts, targets.numel()), dtype=torch.uint8, device=DEV)
        return dict(case=case, plan=plan, queries=(targets, t_start, t_end), fanouts=fanouts, delta=delta, pointers=pointers,
                    workspace=workspace, results=hops)
    if case["kind"] == "ingest":
        m = case["batch"] * case["batches"]
        src, dst, ts = _stream(g, m, case["nodes"], case["ids"])
        results = _outputs(m, case["fanout"], True)
        results["rowptr"] = torch.zeros((case["batches"], case["batch"] + 1), dtype=torch.int64, device=DEV)
        batches = []
        for b in range(case["batches"]):
            part = slice(b * case["batch"], (b + 1) * case["batch"])
            rows = slice(part.start * case["fanout"], part.stop * case["fanout"])
            out = {n: t[rows] for n, t in results.items() if n not in ("rowptr", "count")}
            out.update(rowptr=results["rowptr"][b], count=results["count"][part])
            batches.append((src[part], dst[part], ts[part], out))
        probe = B.Plan(2, case["fanout"])
        workspace = torch.zeros(B.tns_workspace(probe.handle, case["batch"]), dtype=torch.uint8, device=DEV)
        probe.close()
        for *_, out in batches:
            out["workspace"] = workspace
        return dict(case=case, batches=batches, results=results)
    n, batch, d = case["num_ids"], case["batch"], case["dim"]
    store = torch.randn((n, d), generator=g, device=DEV)
    ids = _zipf_ids(g, CACHE_BATCHES * batch, n, case["zipf"]).view(CACHE_BATCHES, batch)
    cache = KB.Cache(n, max(int(n * case["ratio"]), 1), d, CACHE_POLICIES[case["policy"]], 0.2)
    out = torch.zeros((batch, d), dtype=torch.float32, device=DEV)
    hit = torch.zeros(batch, dtype=torch.uint8, device=DEV)
    for i in range(CACHE_WARM):
        cache.fetch(ids[i], store, out, hit)
    return dict(case=case, cache=cache, store=store, ids=list(ids), out=out, hit=hit, next=CACHE_WARM)


# ---- one pass ------------------------------------------------------------------------------------

def _address(t):
    return 0 if t is None else t.data_ptr()


def run(state):
    case = state["case"]
    if case["kind"] == "hop":
        targets, t_start, t_end, offsets = state["queries"]
        out = state["out"]
        if case["static"]:
            B.tns_run_static(state["plan"].handle, targets.numel(), _address(targets), _address(t_start), _address(t_end),
                             _address(offsets), 0, *(out[n].data_ptr() for n in ("nbr", "eid", "ts", "count", "rowptr", "cmp_nbr",
                                                                                  "cmp_eid", "cmp_ts")),
                             torch.cuda.current_stream().cuda_stream)
        else:
            state["plan"].run(targets, t_start, t_end, offsets, out=out)
        return state["results"]
    if case["kind"] == "khop":
        targets, t_start, t_end = state["queries"]
        B.tns_run_khop(state["plan"].handle, state["fanouts"], state["delta"], targets.numel(), _address(targets), _address(t_start),
                       _address(t_end), 0, 0, state["pointers"], state["workspace"].data_ptr(), state["workspace"].numel(),
                       torch.cuda.current_stream().cuda_stream)
        return state["results"]
    if case["kind"] == "ingest":
        plan = B.Plan(case["nodes"], case["fanout"], B.TNS_POLICY_RECENT, case["tau"], flags=B.TNS_FLAG_DEVICE_INGEST)
        for src, dst, ts, out in state["batches"]:
            plan.add_edges_device(src, dst, ts)
            plan.run(src, None, ts, out=out)
        plan.close()
        return state["results"]
    ids = state["ids"][state["next"] % CACHE_BATCHES]
    state["next"] += 1
    return state["cache"].fetch(ids, state["store"], state["out"], state["hit"])


# ---- what a pass cannot do without ---------------------------------------------------------------

def _edges_per_query(edges, queries, nodes, ids, fanout, window):
    """Expected number of sampled edges of a query at an event of a stream: the number of a node's earlier events
    (inside the window) is close to a Poisson variable whose mean is its share of the stream's past."""
    if ids == "zipf":
        w = np.arange(1, nodes + 1, dtype=np.float64) ** -1.1
        w /= w.sum()
        bounds = np.unique(np.concatenate([np.arange(0, min(64, nodes)), np.geomspace(min(64, nodes), nodes, 64).astype(np.int64)]))
        cum = np.concatenate([[0.0], np.cumsum(w)])
        share = np.diff(cum[bounds])                      # chance that a query's node lies in the group of ranks
        rate = share / np.diff(bounds)                    # chance of one node of the group
    else:
        share, rate = np.ones(1), np.full(1, 1.0 / nodes)
    at = edges - min(queries, edges) * (np.arange(64) + 0.5) / 64
    past = np.minimum(at, window * edges) if window else at
    lam = rate[:, None] * past[None, :]
    p = np.exp(-lam)
    expect, below = np.zeros_like(lam), np.zeros_like(lam)
    for k in range(fanout):                               # sum over k of P(more than k)
        below = below + p
        expect += np.maximum(1.0 - below, 0.0)
        p = p * lam / (k + 1)
    return float((share[:, None] * expect).sum() / 64)


def _hop_bytes(queries, edges, nodes, fanout, k, padded, windowed):
    read = queries * (12 if windowed else 8) + 16 * min(queries, nodes) + 12 * min(queries * k, edges)
    write = queries * (8 + 12 * k) + (queries * (12 * fanout + 4) if padded else 0)
    return read + write


def work(case):
    if case["kind"] == "hop":
        e, nodes = case["edges"], _nodes(case["edges"])
        q = min(case["queries"], e)
        k = _edges_per_query(e, q, nodes, case["ids"], case["fanout"], case["window"])
        return {"bytes": case["instances"] * _hop_bytes(q, e, nodes, case["fanout"], k, True, case["window"] > 0), "flops": 0}
    if case["kind"] == "khop":
        e, nodes = case["edges"], _nodes(case["edges"])
        q, total = min(case["queries"], e), 0.0
        for f in (int(x) for x in case["fanouts"].split(",")):
            k = _edges_per_query(e, q, nodes, case["ids"], f, case["window"])
            total += _hop_bytes(q, e, nodes, f, k, case["padded"], case["window"] > 0)
            q *= k
        return {"bytes": total, "flops": 0}
    if case["kind"] == "ingest":
        m, nodes = case["batch"] * case["batches"], case["nodes"]
        k = _edges_per_query(m, m, nodes, case["ids"], case["fanout"], 0.0)
        per_batch = _hop_bytes(case["batch"], m, nodes, case["fanout"], k, True, False) + 24 * case["batch"]
        return {"bytes": case["batches"] * per_batch, "flops": 0}
    row = 4 * case["dim"]
    return {"bytes": case["batch"] * (4 + 1 + 2 * row) + 8 * max(int(case["num_ids"] * case["ratio"]), 1), "flops": 0}


def tolerance(case):
    return "exact"       # ids, times and feature rows are selected and copied, never computed
