"""Batches whose tiles tag what they publish (no cleared scan state, no tickets): sizes around the edges of that rule and of the
tiles, workspaces that hold anything, calls of other forms on the same workspace in between, and replays of a captured call."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from _harness import assert_same, build_plan, oracle_sample

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2311_17410_amd import binding
    binding.lib()
    return binding


def store(B, fanout, policy, seed=6):
    rng = np.random.default_rng(fanout)
    n, nodes = 30_000, 3000
    src = (rng.zipf(1.3, n) % nodes).astype(np.int32)
    ts = np.sort(rng.standard_normal(n)).astype(np.float32)
    st = W.Stream(nodes, src, rng.integers(0, nodes, n, dtype=np.int32), ts, 1500)
    wl = W.Workload("mixed", 0, [st], fanout=fanout, tau=48)
    return st, wl, build_plan(B, wl, policy, seed=seed)


def results(out, Q, f):
    total = int(out["rowptr"][-1].item())
    got = {n: out[n].cpu().numpy().reshape(Q, f) for n in ("nbr", "eid", "ts")}
    got.update({n: out[n].cpu().numpy() for n in ("count", "rowptr")})
    got.update({n: out[n][:total].cpu().numpy() for n in ("cmp_nbr", "cmp_eid", "cmp_ts")})
    return got


def dirty(ws, kind, seed):
    import torch
    if kind == "zeros":
        ws.zero_()
    elif kind == "ones":
        ws.fill_(255)
    else:
        g = torch.Generator(device=ws.device)
        g.manual_seed(seed)
        ws.copy_(torch.randint(0, 256, ws.shape, dtype=torch.uint8, device=ws.device, generator=g))


# one tile, its edges, both kernels around 2^15 and 2^16 queries, the last sizes without tickets (2^18, 2^17 and 2^16 with larger
# fan-outs) and the first ones with them
@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("Q,fanout", [(1, 10), (64, 10), (65, 3), (1000, 64), (1 << 15, 10), ((1 << 15) + 1, 10), (1 << 16, 5), ((1 << 16) + 1, 10),
                                      (1 << 18, 10), ((1 << 18) + 1, 10), (1 << 17, 13), ((1 << 17) + 1, 32), (1 << 16, 64), ((1 << 16) + 1, 33)])
def test_any_workspace(B, oracle_lib, policy, Q, fanout, layout):
    import torch
    st, wl, plan = store(B, fanout, policy)
    targets, _, t_end = W.random_queries(Q, st, Q)
    ref = oracle_sample(oracle_lib, wl, targets, None, t_end, None, fanout, policy, 0, 6)
    d_t, d_e = torch.from_numpy(targets).cuda(), torch.from_numpy(t_end).cuda()
    out = plan.run(d_t, None, d_e)
    assert_same(results(out, Q, fanout), ref, oracle_lib, "first call")
    for i, kind in enumerate(("zeros", "ones", "random", "as left", "as left")):
        if kind != "as left":
            dirty(out["workspace"], kind, i)
        for n in ("rowptr", "cmp_eid", "count"):
            out[n].fill_(-3)
        plan.run(d_t, None, d_e, out=out)
        torch.cuda.synchronize()
        assert not plan.status(out["workspace"]), kind
        assert_same(results(out, Q, fanout), ref, oracle_lib, kind)
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
def test_replays_between_other_calls(B, oracle_lib, policy, layout):
    # a captured call of 150 tiles, replayed with new queries; between replays the workspace serves a smaller call, one with a cleared
    # scan state, two hops, the padding removal alone, or has its head cleared
    import torch
    fanout, Q, big = 10, 9600, (1 << 18) + 300
    st, wl, plan = store(B, fanout, policy)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    targets, _, t_end = W.random_queries(1, st, big)
    d_t, d_e = d(targets[:Q]), d(t_end[:Q])
    large = plan.run(d(targets), None, d(t_end))
    hops, ws_hops = plan.run_khop([fanout, 4], d(targets[:500]), None, d(t_end[:500]))
    assert ws_hops.numel() <= large["workspace"].numel()
    ws = large["workspace"]
    out = plan.run(d_t, None, d_e)
    out["workspace"] = ws
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        plan.run(d_t, None, d_e, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        plan.run(d_t, None, d_e, out=out)
    names = [n for n, _ in B.tns_hop_buffers._fields_]
    ptrs = [{n: h[n].data_ptr() for n in names} for h in hops]

    def between(i):
        if i % 6 == 1:
            plan.run(d_t[:100], None, d_e[:100], out={**plan.run(d_t[:100], None, d_e[:100]), "workspace": ws})
        elif i % 6 == 2:
            plan.run(d(targets), None, d(t_end), out=large)
        elif i % 6 == 3:
            B.tns_run_khop(plan.handle, [fanout, 4], float("inf"), 500, d_t.data_ptr(), 0, d_e.data_ptr(), 0, 0, ptrs, ws.data_ptr(), ws.numel(),
                           torch.cuda.current_stream().cuda_stream)
        elif i % 6 == 4:
            ws[:256].zero_()
        elif i % 6 == 5:
            B.tns_compact(plan.handle, Q, *(out[n].data_ptr() for n in ("nbr", "eid", "ts", "count", "rowptr", "cmp_nbr", "cmp_eid", "cmp_ts")),
                          ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()

    for i in range(13):
        t, _, e = W.random_queries(100 + i, st, Q)
        d_t.copy_(d(t))
        d_e.copy_(d(e))
        between(i)
        out["rowptr"].fill_(-3)
        graph.replay()
        torch.cuda.synchronize()
        assert not plan.status(ws), i
        ref = oracle_sample(oracle_lib, wl, t, None, e, None, fanout, policy, 0, 6, adjs=adjs)
        assert_same(results(out, Q, fanout), ref, oracle_lib, f"replay {i}")
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("Q", [9600, 100_000])
def test_replays_over_what_an_earlier_one_left(B, oracle_lib, policy, Q, layout):
    # a captured call and a captured pair of hops, replayed with new queries: before every replay the workspace is made byte for byte
    # what the first replay left, with its tile totals (other work may put any part of it back, and leave the rest)
    import torch
    fanout, roots = 10, 700
    st, wl, plan = store(B, fanout, policy)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    targets, _, t_end = W.random_queries(1, st, Q)
    d_t, d_e = d(targets), d(t_end)
    out = plan.run(d_t, None, d_e)
    hops, ws_hops = plan.run_khop([fanout, 4], d_t[:roots], None, d_e[:roots])
    names = [n for n, _ in B.tns_hop_buffers._fields_]
    ptrs = [{n: h[n].data_ptr() for n in names} for h in hops]

    def call():
        plan.run(d_t, None, d_e, out=out)
        B.tns_run_khop(plan.handle, [fanout, 4], float("inf"), roots, d_t.data_ptr(), 0, d_e.data_ptr(), 0, 0, ptrs, ws_hops.data_ptr(), ws_hops.numel(),
                       torch.cuda.current_stream().cuda_stream)

    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    graph.replay()
    torch.cuda.synchronize()
    left = out["workspace"].clone(), ws_hops.clone()
    for i in range(6):
        t, _, e = W.random_queries(100 + i, st, Q)
        d_t.copy_(d(t))
        d_e.copy_(d(e))
        for a in (out["rowptr"], out["cmp_eid"], *(h[n] for h in hops for n in ("rowptr", "cmp_eid"))):
            a.fill_(-3)
        out["workspace"].copy_(left[0])
        ws_hops.copy_(left[1])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert not plan.status(out["workspace"]) and not plan.status(ws_hops), i
        ref = oracle_sample(oracle_lib, wl, t, None, e, None, fanout, policy, 0, 6, adjs=adjs)
        assert_same(results(out, Q, fanout), ref, oracle_lib, f"replay {i}")
        eager, _ = plan.run_khop([fanout, 4], d_t[:roots], None, d_e[:roots])
        for h, want in zip(hops, eager):
            q = roots if h is hops[0] else int(hops[0]["rowptr"][-1].item())
            assert torch.equal(h["rowptr"][:q + 1], want["rowptr"][:q + 1]), i
            rows = int(want["rowptr"][q].item())
            for n in ("cmp_nbr", "cmp_eid", "cmp_ts"):
                assert torch.equal(h[n][:rows], want[n][:rows]), (i, n)
    plan.close()


@pytest.mark.parametrize("Q", [700, 40_000, 300_000])
def test_a_tile_that_never_reports(B, Q):
    # tile 0 does not exist: the waits run out, the time-out is reported and the next sound call clears the report
    import torch
    n = max(Q, 1000)
    rng = np.random.default_rng(2)
    st = W.Stream(500, rng.integers(0, 500, n, dtype=np.int32), rng.integers(0, 500, n, dtype=np.int32), np.sort(rng.random(n)).astype(np.float32), 4096)
    wl = W.Workload("tiny", 0, [st], fanout=10, tau=48)
    lost, sound = build_plan(B, wl, flags=B.TNS_TEST_FLAG_LOST_TILE), build_plan(B, wl)
    d_t, d_e = torch.from_numpy(st.src[:Q]).cuda(), torch.from_numpy(st.ts[:Q]).cuda()
    out = lost.run(d_t, None, d_e)
    torch.cuda.synchronize()
    assert lost.status(out["workspace"]) and int(out["rowptr"][-1].item()) == 0
    total = int(sound.run(d_t, None, d_e)["rowptr"][-1].item())
    sound.run(d_t, None, d_e, out=out)
    torch.cuda.synchronize()
    assert not sound.status(out["workspace"]) and int(out["rowptr"][-1].item()) == total > 0
    lost.close()
    sound.close()


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("Q,fanout,instances", [(1, 10, 1), (130, 3, 1), (4000, 64, 1), (16_500, 10, 1), (30_001, 20, 1), (40_000, 5, 3), (100_000, 10, 1), (60_000, 64, 1),
                                                ((1 << 18) - 1, 10, 1)])
def test_tiles_that_leave_their_dense_rows_to_another(B, oracle_lib, policy, Q, fanout, instances, layout):
    # a tile that does not find the totals before it at once makes room; another one's workgroup samples it again
    import ctypes

    import torch
    rng = np.random.default_rng(Q)
    sts = []
    for _ in range(instances):
        src = (rng.zipf(1.3, 30_000) % 3000).astype(np.int32)
        sts.append(W.Stream(3000, src, rng.integers(0, 3000, 30_000, dtype=np.int32), np.sort(rng.standard_normal(30_000)).astype(np.float32), 1500))
    wl = W.Workload("mixed", 0, sts, fanout=fanout, tau=48)
    plan = build_plan(B, wl, policy, seed=6)
    defer = B.lib().tns_test_defer
    defer.argtypes, defer.restype = [ctypes.c_void_p], None
    defer(plan.handle)
    per = Q // instances
    parts = [W.random_queries(Q + i, st, per) for i, st in enumerate(sts)]
    targets, t_end = (np.concatenate([x[j] for x in parts]) for j in (0, 2))
    inst = np.arange(instances + 1, dtype=np.int64) * per if instances > 1 else None
    Q = per * instances
    ref = oracle_sample(oracle_lib, wl, targets, None, t_end, inst, fanout, policy, 0, 6)
    d = lambda a: None if a is None else torch.from_numpy(a).cuda()  # noqa: E731
    args = (d(targets), None, d(t_end), d(inst))
    out = plan.run(*args)
    for i in range(4):
        for n in ("rowptr", "cmp_eid", "count", "eid"):
            out[n].fill_(-3)
        if i == 0:
            out["workspace"][8:16].zero_()
        plan.run(*args, out=out)
        torch.cuda.synchronize()
        assert not plan.status(out["workspace"])
        assert_same(results(out, Q, fanout), ref, oracle_lib, f"call {i}")
    again = int(out["workspace"][8:16].cpu().numpy().view(np.int64)[0])      # tiles sampled again in four calls
    assert again > 0 if Q >= 30_000 else again >= 0, again
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
def test_four_streams(B, oracle_lib, policy):
    # four queues with launches that together are larger than the chip, each with its own workspace and queries, none waiting for another
    import torch
    fanout, Q, streams = 10, 200_000, [torch.cuda.Stream() for _ in range(4)]
    st, wl, plan = store(B, fanout, policy)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    queries = [W.random_queries(50 + i, st, Q) for i in range(4)]
    on_device = [(torch.from_numpy(t).cuda(), torch.from_numpy(e).cuda()) for t, _, e in queries]
    outs = [plan.run(t, None, e) for t, e in on_device]
    for o in outs:
        o["rowptr"].fill_(-3)
    torch.cuda.synchronize()
    for _ in range(20):
        for s, (t, e), o in zip(streams, on_device, outs):
            with torch.cuda.stream(s):
                plan.run(t, None, e, out=o)
    torch.cuda.synchronize()
    for (t, _, e), o in zip(queries, outs):
        assert not plan.status(o["workspace"])
        assert_same(results(o, Q, fanout), oracle_sample(oracle_lib, wl, t, None, e, None, fanout, policy, 0, 6, adjs=adjs), oracle_lib, "streams")
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
def test_small_calls_beside_large_ones(B, oracle_lib, policy, layout):
    # calls without tickets on two streams while two others keep the chip full with calls of many tiles: workgroups of the small
    # calls start late and in any order
    import torch
    fanout, streams = 10, [torch.cuda.Stream() for _ in range(4)]
    st, wl, plan = store(B, fanout, policy)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    sizes = [1 << 21, 1 << 21, 100_000, 4000]
    queries = [W.random_queries(60 + i, st, q) for i, q in enumerate(sizes)]
    on_device = [(torch.from_numpy(t).cuda(), torch.from_numpy(e).cuda()) for t, _, e in queries]
    outs = [plan.run(t, None, e) for t, e in on_device]
    torch.cuda.synchronize()
    kept = [o["cmp_eid"][:int(o["rowptr"][-1].item())].clone() for o in outs]
    for o in outs:
        for n in ("rowptr", "cmp_eid", "count"):
            o[n].fill_(-3)
    torch.cuda.synchronize()
    for _ in range(20):
        for s, (t, e), o in zip(streams, on_device, outs):
            with torch.cuda.stream(s):
                plan.run(t, None, e, out=o)
    torch.cuda.synchronize()
    for o, want in zip(outs, kept):
        assert not plan.status(o["workspace"])
        assert int(o["rowptr"][-1].item()) == want.numel() and torch.equal(o["cmp_eid"][:want.numel()], want)
    for (t, _, e), o in list(zip(queries, outs))[2:]:
        assert_same(results(o, len(t), fanout), oracle_sample(oracle_lib, wl, t, None, e, None, fanout, policy, 0, 6, adjs=adjs), oracle_lib, "small")
    plan.close()
