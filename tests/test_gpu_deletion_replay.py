"""A sampling call captured in a HIP graph and replayed after a deletion must not return deleted edges: the store is
changed in place, so every kernel has to read from the store itself which edges are there."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from _harness import assert_same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2311_17410_amd import binding
    binding.lib()
    return binding


def store(B, fanout, policy, tau, incl, on_device=True):
    import torch
    st = W.zipf_stream(np.random.Generator(np.random.PCG64(5)), 1 << 14, 1 << 9, 1 << 10, 1.1, "normal")    # hubs of long lists
    plan = B.Plan(st.num_nodes, fanout, policy=policy, block_threshold=tau, inclusive_end=incl, seed=21,
                  flags=B.TNS_FLAG_DEVICE_INGEST if on_device else 0)
    for lo in range(0, st.n, st.batch):
        part = [a[lo:lo + st.batch] for a in (st.src, st.dst, st.ts)]
        if on_device:
            plan.add_edges_device(*(torch.from_numpy(a).cuda() for a in part))
        else:
            B.tns_add_edges(plan.handle, 0, *part)
    plan.commit()
    # a fifth of the edges, all edges of one small node and all but the oldest of a hub
    rng = np.random.default_rng(3)
    gone = rng.random(st.n) < 0.2
    degree = np.bincount(st.src, minlength=st.num_nodes)
    gone |= st.src == np.flatnonzero(degree > 0)[np.argmin(degree[degree > 0])]
    hub = np.flatnonzero(st.src == np.argsort(degree)[-2])
    gone[hub[1:]] = True
    return st, plan, np.flatnonzero(gone).astype(np.int32), (~gone).astype(np.uint8)


def outputs(out, Q, f):
    total = int(out["rowptr"][-1].item())
    got = {n: out[n].cpu().numpy().reshape(Q, f) for n in ("nbr", "eid", "ts")}
    got.update({n: out[n].cpu().numpy() for n in ("count", "rowptr")})
    got.update({n: out[n][:total].cpu().numpy() for n in ("cmp_nbr", "cmp_eid", "cmp_ts")})
    return got


# queries: one and two of them per team of sixteen lanes, and a query per lane
@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("Q,fanout,tau,incl,on_device", [(1, 10, 48, 0, True), (701, 10, 48, 0, True), (701, 20, 8192, 1, False),
                                                         (16_385, 16, 5, 1, True), (30_001, 64, 48, 0, True), (65_536, 10, 48, 0, False),
                                                         (65_537, 10, 48, 0, True)])
def test_run_replayed_after_deletion(B, oracle_lib, policy, Q, fanout, tau, incl, on_device):
    import torch
    st, plan, victims, present = store(B, fanout, policy, tau, incl, on_device)
    targets, t_start, t_end = W.random_queries(6, st, Q)
    d = [torch.from_numpy(a).cuda() for a in (targets, t_start, t_end)]
    graphs = []
    for tb in (None, d[1]):
        out = plan.alloc_outputs(Q, compact=True)
        plan.run(d[0], tb, d[2], out=out)                       # eager once: loads the code objects
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            plan.run(d[0], tb, d[2], out=out)
        graphs.append((graph, out))
    for deleted in (False, True):
        if deleted:
            assert B.tns_delete_edges(plan.handle, 0, st.src[victims], victims) == len(victims)
            plan.commit()
        adj = oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts, present=present if deleted else None)
        for (graph, out), tb in zip(graphs, (None, t_start)):
            ref = adj.sample(targets, tb, t_end, fanout, policy=policy, inclusive_end=incl, seed=21)
            for rep in range(2):
                graph.replay()
                torch.cuda.synchronize()
                assert_same(outputs(out, Q, fanout), ref, oracle_lib, f"deleted={deleted} start={tb is not None} replay {rep}")
        adj.close()
    del graphs
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("fanouts,delta", [([10, 10], float("inf")), ([3, 17], 0.7)])
def test_khop_replayed_after_deletion(B, oracle_lib, policy, fanouts, delta):
    import torch
    from oracle import khop_oracle
    st, plan, victims, present = store(B, fanouts[0], policy, 48, 0)
    Q = 301
    targets, _, t_end = W.random_queries(6, st, Q)
    d = [torch.from_numpy(a).cuda() for a in (targets, t_end)]
    eager, _ = plan.run_khop(fanouts, d[0], None, d[1], delta=delta)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        out, ws = plan.run_khop(fanouts, d[0], None, d[1], delta=delta)
    for deleted in (False, True):
        if deleted:
            assert B.tns_delete_edges(plan.handle, 0, st.src[victims], victims) == len(victims)
            eager, _ = plan.run_khop(fanouts, d[0], None, d[1], delta=delta)
        adj = oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts, present=present if deleted else None)
        hops = khop_oracle.khop([adj], targets, None, t_end, None, fanouts, delta=delta, policy=policy, seed=21, threads=8)
        for what in ("eager", "replay", "replay again"):
            if what != "eager":
                graph.replay()
            torch.cuda.synchronize()
            for h, (got, ref) in enumerate(zip(eager if what == "eager" else out, hops)):
                n = len(ref["rowptr"]) - 1
                assert np.array_equal(got["rowptr"][:n + 1].cpu().numpy(), ref["rowptr"]), (deleted, what, h)
                total = int(ref["rowptr"][-1])
                for name in ("cmp_nbr", "cmp_eid", "cmp_ts"):
                    assert np.array_equal(got[name][:total].cpu().numpy(), ref[name]), (deleted, what, h, name)
        adj.close()
    del graph
    plan.close()
