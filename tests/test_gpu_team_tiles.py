"""Small batches: the workgroups' sizes change with the batch and with the room the workspace has for tile states.  Both sides of
every line of that rule, with the workspace that tns_workspace asks for and with the smallest one that is accepted, against the oracle."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W

SIZES = [1, 16, 17, 512, 513, 4096, 4097, 8192, 8193, 16384, 16385, 49152, 49153]


def least(Q):
    """Bytes without room for the states of small tiles: one state per 64 queries, or the two-step form's sums."""
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    tiles = (Q + 1023) // 1024
    return max(up(4 * tiles) + up(8 * tiles) + 256, up(256 + 8 * ((Q + 63) // 64 + 1)))


@pytest.mark.gpu
@pytest.mark.parametrize("policy,fanout", [(0, 10), (1, 10), (0, 20), (1, 64)])
def test_tiles_of_small_batches(oracle_lib, policy, fanout):
    import torch
    from paper_2311_17410_amd import binding as B
    rng = np.random.default_rng(fanout + policy)
    nodes, n = 2000, 50_000
    src = (rng.zipf(1.2, n) % (nodes - 5)).astype(np.int32)
    dst = rng.integers(0, nodes, n, dtype=np.int32)
    ts = np.sort(rng.integers(0, n // 10, n)).astype(np.float32)
    plan = B.Plan(nodes, fanout, policy=policy, block_threshold=48, seed=3, flags=B.TNS_FLAG_DEVICE_INGEST)
    bounds = list(range(0, n, 2500)) + [n]
    d = [torch.from_numpy(a).cuda() for a in (src, dst, ts)]
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        plan.add_edges_device(*(a[lo:hi] for a in d))
    targets, t_start, t_end = W.random_queries(3, W.Stream(nodes, src, dst, ts, 2500), max(SIZES))
    adj = oracle_lib.Adjacency(nodes, src, dst, ts, batch_rowptr=bounds)
    ref = adj.sample(targets, t_start, t_end, fanout, policy=policy, seed=3)
    adj.close()
    dq = [torch.from_numpy(a).cuda() for a in (targets, t_start, t_end)]
    for Q in SIZES:
        part = oracle_lib.Sampled(Q, fanout)
        for name in ("nbr", "eid", "ts", "count"):
            setattr(part, name, getattr(ref, name)[:Q])
        rowptr, cn, ce, ct = oracle_lib.compact(part)
        for size in (B.tns_workspace(plan.handle, Q), least(Q)):
            out = {k: torch.full_like(t, -7 if t.dtype != torch.uint8 else 255) for k, t in plan.alloc_outputs(Q).items()}
            room = torch.full((size + 4096,), 171, dtype=torch.uint8, device="cuda")      # what lies behind the workspace stays as it is
            out["workspace"] = room[:size]
            plan.run(*(t[:Q] for t in dq), out=out)
            assert not plan.status(out["workspace"]) and bool((room[size:] == 171).all()), (Q, size)
            assert np.array_equal(out["rowptr"].cpu().numpy(), rowptr), (Q, size)
            assert np.array_equal(out["count"].cpu().numpy(), part.count), (Q, size)
            for name, want in (("cmp_nbr", cn), ("cmp_eid", ce), ("cmp_ts", ct)):
                assert np.array_equal(out[name].cpu().numpy()[:len(want)], want), (name, Q, size)
            for name in ("nbr", "eid", "ts"):
                assert np.array_equal(out[name].cpu().numpy().reshape(Q, fanout), getattr(part, name)), (name, Q, size)
        with pytest.raises(B.TnsError):
            plan.run(*(t[:Q] for t in dq), out={**out, "workspace": out["workspace"][:least(Q) - 256]})
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("policy", [0, 1])
def test_hops_with_either_workspace(oracle_lib, policy):
    # 600 and 4000 roots: the second hop's tiles are sized for the most queries it can have
    import torch
    from paper_2311_17410_amd import binding as B
    wl = W.c1()
    plan = B.Plan(wl.num_nodes, 10, policy=policy, block_threshold=wl.tau, seed=5, flags=B.TNS_FLAG_DEVICE_INGEST)
    st = wl.streams[0]
    d = [torch.from_numpy(a).cuda() for a in (st.src, st.dst, st.ts)]
    plan.add_edges_device(*d)
    for Q in (100, 600, 4000):
        t, _, e = W.random_queries(Q, st, Q)
        dt, de = torch.from_numpy(t).cuda(), torch.from_numpy(e).cuda()
        hops, ws = plan.run_khop([10, 10], dt, None, de)
        got = [{k: h[k].clone() for k in ("rowptr", "cmp_nbr", "cmp_eid", "cmp_ts")} for h in hops]
        keys = ("nbr", "eid", "ts", "count", "rowptr", "cmp_nbr", "cmp_eid", "cmp_ts")
        small = 256 + least(Q) + least(10 * Q) + (2 * 3 * 8 + 255) // 256 * 256
        assert small <= ws.numel()
        for size in (small, B.tns_workspace_khop(plan.handle, [10, 10], Q)):
            again = torch.full((size + 4096,), 171, dtype=torch.uint8, device="cuda")
            for h in hops:
                for k in keys:
                    h[k].fill_(-7)
            B.tns_run_khop(plan.handle, [10, 10], float("inf"), Q, dt.data_ptr(), 0, de.data_ptr(), 0, 0,
                           [{k: h[k].data_ptr() for k in keys} for h in hops], again.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert bool((again[size:] == 171).all()), (Q, size)
            n = Q
            for g, h in zip(got, hops):
                total = int(g["rowptr"][n])
                assert torch.equal(g["rowptr"][:n + 1], h["rowptr"][:n + 1])
                for k in ("cmp_nbr", "cmp_eid", "cmp_ts"):
                    assert torch.equal(g[k][:total], h[k][:total])
                n = total
        with pytest.raises(B.TnsError):
            B.tns_run_khop(plan.handle, [10, 10], float("inf"), Q, dt.data_ptr(), 0, de.data_ptr(), 0, 0,
                           [{k: h[k].data_ptr() for k in keys} for h in hops], again.data_ptr(), small - 256, torch.cuda.current_stream().cuda_stream)
    plan.close()
