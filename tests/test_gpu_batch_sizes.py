"""A batch may be run in pieces of any size: the pieces (sixteen lanes per query) and the whole (a query per lane) must
give the oracle's result bit for bit, on nodes with no edge, with inline block lists and with long directory runs."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from _harness import assert_same, gpu_sample

pytestmark = pytest.mark.gpu

PIECES = [1, 3, 4, 63, 64, 65, 127, 128, 129, 1024, 16384, 16385, 32700]       # edges of the tiles and of the dispatch


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2311_17410_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("fanout,incl,tau,ties", [(10, 0, 8192, False), (16, 1, 48, True), (17, 0, 5, False), (64, 1, 1, True), (1, 0, 48, True)])
def test_pieces_equal_whole(B, oracle_lib, policy, fanout, incl, tau, ties):
    import torch
    rng = np.random.default_rng(fanout * 7 + policy)
    nodes, n = 3000, 60_000
    src = (rng.zipf(1.2, n) % (nodes - 5)).astype(np.int32)
    dst = rng.integers(0, nodes, n, dtype=np.int32)
    ts = np.sort(rng.integers(0, n // 20, n) if ties else rng.standard_normal(n)).astype(np.float32)
    plan = B.Plan(nodes, fanout, policy=policy, block_threshold=tau, inclusive_end=incl, seed=9, flags=B.TNS_FLAG_DEVICE_INGEST)
    bounds = list(range(0, n, 1500)) + [n]
    d = [torch.from_numpy(a).cuda() for a in (src, dst, ts)]
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        plan.add_edges_device(d[0][lo:hi], d[1][lo:hi], d[2][lo:hi])
    st = W.Stream(nodes, src, dst, ts, 1500)
    Q = 1 + sum(PIECES) + 300
    targets, t_start, t_end = W.random_queries(3, st, Q)
    adj = oracle_lib.Adjacency(nodes, src, dst, ts, batch_rowptr=bounds)
    assert Q > 1 << 16                                   # the whole takes the other kernel
    for tb in (None, t_start):
        ref = adj.sample(targets, tb, t_end, fanout, policy=policy, inclusive_end=incl, seed=9)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, "whole")
        lo = 0
        for size in PIECES + [Q - sum(PIECES)]:
            hi = lo + size
            part = oracle_lib.Sampled(size, fanout)
            for name in ("nbr", "eid", "ts", "count"):
                setattr(part, name, getattr(ref, name)[lo:hi])
            got = gpu_sample(plan, targets[lo:hi], None if tb is None else tb[lo:hi], t_end[lo:hi], query_id_base=lo)
            assert_same(got, part, oracle_lib, f"piece {lo}..{hi}")
            lo = hi
    adj.close()
    plan.close()


@pytest.mark.parametrize("batch", [2, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("nodes", [1, 700, 1 << 17])
def test_ingestion_batches_around_the_small_plan(B, oracle_lib, batch, nodes):
    import torch
    rng = np.random.default_rng(batch + nodes)
    n = 4 * batch + 1
    src = rng.integers(0, nodes, n, dtype=np.int32)
    src[rng.random(n) < 0.3] = nodes - 1
    dst = rng.integers(0, nodes, n, dtype=np.int32)
    ts = np.sort(rng.integers(0, n // 2, n)).astype(np.float32)
    eid = rng.permutation(n).astype(np.int32)
    ts[2 * batch], ts[3 * batch - 1] = ts[3 * batch - 1], ts[2 * batch]           # the third batch is not in time order
    plan = B.Plan(nodes, 10, block_threshold=48, flags=B.TNS_FLAG_DEVICE_INGEST)
    bs = oracle_lib.BlockStore(nodes, 48, 0)
    d = [torch.from_numpy(a).cuda() for a in (src, dst, ts, eid)]
    bounds = list(range(0, n, batch)) + [n]
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        plan.add_edges_device(*(a[lo:hi] for a in d))
    bs.add_stream(src, dst, ts, batch)
    ref, got = bs.stats(), plan.stats()
    for name in ("num_blocks", "wasted_slots", "max_list_len"):
        assert got[name] == ref[name], name
    st = W.Stream(nodes, src, dst, ts, batch)
    targets, t_start, t_end = W.random_queries(5, st, 3000)
    adj = oracle_lib.Adjacency(nodes, src, dst, ts, batch_rowptr=bounds)
    want = adj.sample(targets, t_start, t_end, 10)
    out = gpu_sample(plan, targets, t_start, t_end)
    out["eid"] = np.where(out["eid"] >= 0, np.argsort(eid)[np.maximum(out["eid"], 0)], -1).astype(np.int32)   # back to stream positions
    for name in ("count", "nbr", "eid", "ts"):
        assert np.array_equal(out[name], getattr(want, name)), name
    adj.close()
    with pytest.raises(B.TnsError):                                # a rejected batch changes nothing
        plan.add_edges_device(torch.full((batch,), nodes, dtype=torch.int32, device="cuda"), d[1][:batch], d[2][-1].repeat(batch))
    assert plan.stats()["num_edges"] == n
    plan.close()


@pytest.mark.parametrize("batch", [(1 << 16) - 1, 1 << 16, (1 << 16) + 1, (1 << 18) - 1, 1 << 18, (1 << 18) + 1])
def test_ingestion_batches_of_many_plan_tiles(B, oracle_lib, batch):
    # 128, 129, 512 and 513 tiles of sorted positions; a node of a tenth of every batch spans dozens of them
    import torch
    rng = np.random.default_rng(batch)
    n, nodes = 2 * batch, 30_000
    src = rng.integers(0, nodes, n, dtype=np.int32)
    src[rng.random(n) < 0.1] = nodes // 2
    dst = rng.integers(0, nodes, n, dtype=np.int32)
    ts = np.sort(rng.random(n)).astype(np.float32)
    plan = B.Plan(nodes, 10, block_threshold=48, flags=B.TNS_FLAG_DEVICE_INGEST)
    bs = oracle_lib.BlockStore(nodes, 48, 0)
    d = [torch.from_numpy(a).cuda() for a in (src, dst, ts)]
    for lo in (0, batch):
        plan.add_edges_device(*(a[lo:lo + batch] for a in d))
    bs.add_stream(src, dst, ts, batch)
    ref, got = bs.stats(), plan.stats()
    for name in ("num_blocks", "wasted_slots", "max_list_len"):
        assert got[name] == ref[name], name
    st = W.Stream(nodes, src, dst, ts, batch)
    targets, t_start, t_end = W.random_queries(5, st, 3000)
    targets[:50] = nodes // 2
    adj = oracle_lib.Adjacency(nodes, src, dst, ts)
    for tb in (None, t_start):
        assert_same(gpu_sample(plan, targets, tb, t_end), adj.sample(targets, tb, t_end, 10), oracle_lib, f"start={tb is not None}")
    adj.close()
    plan.close()


def test_stores_built_one_after_another_by_two_threads(B, oracle_lib):
    # memory of a closed plan is kept for the next one: plans of two threads, each on a stream of its own, of changing
    # sizes, must not see each other's (or an earlier plan's) data
    import threading
    import torch
    rng = np.random.default_rng(8)
    nodes, n = 2000, 40_000
    src, dst = (rng.integers(0, nodes, n, dtype=np.int32) for _ in range(2))
    ts = np.sort(rng.standard_normal(n)).astype(np.float32)
    sizes = (n, 3000, 20_000, 500, n)
    want = {}
    for m in sizes:
        adj = oracle_lib.Adjacency(nodes, src[:m], dst[:m], ts[:m])
        want[m] = adj.sample(src[:m], None, ts[:m], 10)
        adj.close()
    errors = []

    def work(shift):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                d = [torch.from_numpy(a).cuda() for a in (src, dst, ts)]
                for i in range(10):
                    m = sizes[(i + shift) % len(sizes)]
                    plan = B.Plan(nodes, 10, flags=B.TNS_FLAG_DEVICE_INGEST)
                    for lo in range(0, m, 2500):
                        hi = min(lo + 2500, m)
                        plan.add_edges_device(*(a[lo:hi] for a in d))
                    out = plan.run(d[0][:m], None, d[2][:m])
                    torch.cuda.current_stream().synchronize()
                    for name in ("nbr", "eid", "ts"):
                        assert np.array_equal(out[name].cpu().numpy().reshape(m, 10), getattr(want[m], name)), (i, m, name)
                    plan.close()
        except Exception as e:       # noqa: BLE001 -- reported by the test's own thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("m", [1, 64, 2048, 2049, 4096, 4097, 20_000, 100_000])
def test_an_edge_out_of_order_is_found_wherever_its_node_lies(B, m):
    # one wave of the plan meets the node whose newest edge is younger than the batch; the host must hear of it every
    # time, of the smallest such node where there are several, and the store must stay as it was
    import torch
    nodes = m + 3
    late = sorted({0, m // 3, m // 2, m - 1})
    plan = B.Plan(nodes, 4, flags=B.TNS_FLAG_DEVICE_INGEST)
    ids = torch.tensor(late, dtype=torch.int32, device="cuda")
    plan.add_edges_device(ids, ids, torch.full((len(late),), 100.0, device="cuda"))
    src = torch.arange(m, dtype=torch.int32, device="cuda")
    ts = torch.linspace(1.0, 2.0, m, device="cuda")
    shuffled = src[torch.randperm(m, device="cuda")]
    for rep in range(10):
        for v in late:
            part = torch.where(torch.isin(src, ids) & (src != v), nodes - 1, src)       # `v` alone is late
            with pytest.raises(B.TnsError, match=f"node {v} would receive") as e:
                plan.add_edges_device(part, part, ts)
            assert e.value.status == B.TNS_EORDER
        with pytest.raises(B.TnsError, match="node 0 would receive"):
            plan.add_edges_device(shuffled, shuffled, ts)
    assert plan.stats()["num_edges"] == len(late)
    out = plan.run(src, None, torch.full((m,), 1000.0, device="cuda"))
    assert torch.equal(torch.nonzero(out["count"])[:, 0].int(), ids)
    plan.close()


@pytest.mark.parametrize("m", [700, 5000])
def test_batches_behind_a_busy_stream(B, oracle_lib, m):
    # the host gives up polling for a batch's plan after 2 ms and waits for the stream: same store, same refusals
    import torch
    rng = np.random.default_rng(m)
    nodes, n = 400, 6 * m
    src, dst = (rng.integers(0, nodes, n, dtype=np.int32) for _ in range(2))
    ts = np.sort(rng.standard_normal(n)).astype(np.float32)
    ts[3 * m:4 * m] = rng.permutation(ts[3 * m:4 * m])                     # this batch is not in time order
    d = [torch.from_numpy(a).cuda() for a in (src, dst, ts)]
    plan = B.Plan(nodes, 10, flags=B.TNS_FLAG_DEVICE_INGEST)
    block = torch.zeros(1 << 28, dtype=torch.float32, device="cuda")
    other = torch.empty_like(block)

    def busy():                    # some 15 ms of copies
        for _ in range(40):
            other.copy_(block)

    for lo in range(0, n, m):
        busy()
        plan.add_edges_device(*(a[lo:lo + m] for a in d))
        busy()
        with pytest.raises(B.TnsError) as e:                               # older than what is stored
            plan.add_edges_device(d[0][lo:lo + m], d[1][lo:lo + m], d[2][lo:lo + m] - 100.0)
        assert e.value.status == B.TNS_EORDER
    assert plan.stats()["num_edges"] == n
    st = W.Stream(nodes, src, dst, ts, m)
    targets, t_start, t_end = W.random_queries(5, st, 3000)
    adj = oracle_lib.Adjacency(nodes, src, dst, ts, batch_rowptr=list(range(0, n + 1, m)))
    assert_same(gpu_sample(plan, targets, t_start, t_end), adj.sample(targets, t_start, t_end, 10), oracle_lib, "store")
    adj.close()
    plan.close()
