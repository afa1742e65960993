"""The kernel with a query per lane serves batches above 2^16 queries (from there on under the recent policy and with small fan-outs): its parity at the edge of
that rule, with 64-bit positions, over instances of uneven and no size, and its bounded wait."""
import time

import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from _harness import assert_same, build_plan, gpu_sample, oracle_sample

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2311_17410_amd import binding
    binding.lib()
    return binding


def mixed_stream(seed, num_nodes, n, batch, ties):
    """Nodes of every size: none, a few edges, inline lists, and hubs of long lists."""
    rng = np.random.default_rng(seed)
    src = (rng.zipf(1.3, n) % max(num_nodes - 3, 1)).astype(np.int32)
    ts = np.sort(rng.integers(0, max(n // 10, 2), n) if ties else rng.standard_normal(n)).astype(np.float32)
    return W.Stream(num_nodes, src, rng.integers(0, num_nodes, n, dtype=np.int32), ts, batch)


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("fanout,Q", [(5, (1 << 16) - 1), (5, 1 << 16), (7, 1 << 16), (8, 1 << 16), (8, (1 << 16) + 1)])
def test_both_sides_of_the_rule(B, oracle_lib, policy, fanout, Q):
    st = mixed_stream(1, 2000, 20_000, 900, ties=False)
    wl = W.Workload("mixed", 0, [st], fanout=fanout, tau=48)
    plan = build_plan(B, wl, policy, seed=3)
    targets, t_start, t_end = W.random_queries(2, st, Q)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    for tb in (None, t_start):
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, policy, 0, 3, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, f"start={tb is not None}")
    plan.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("fanout,tau,incl,ties", [(1, 48, 0, True), (3, 16, 1, True), (10, 5, 0, False), (10, 8192, 1, True),
                                                  (16, 1, 0, True), (20, 48, 0, False), (64, 48, 1, True)])
def test_large_batches_with_64_bit_positions(B, oracle_lib, wide, policy, fanout, tau, incl, ties):
    st = mixed_stream(fanout + policy, 500, 12_000, 700, ties)
    wl = W.Workload("mixed", 0, [st], fanout=fanout, tau=tau)
    plan = build_plan(B, wl, policy, incl, seed=8, flags=B.TNS_FLAG_WIDE_POSITIONS if wide else 0)
    targets, t_start, t_end = W.random_queries(44, st, (1 << 16) + 77)
    adjs = [oracle_lib.Adjacency(st.num_nodes, st.src, st.dst, st.ts)]
    for tb in (t_start, None):
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, policy, incl, 8, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, f"start={tb is not None}")
        got = gpu_sample(plan, targets, tb, t_end, compact=False)
        assert_same(got, ref, None, f"without the padding removal, start={tb is not None}")
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("fanout", [1, 9, 10, 11, 17])
def test_degrees_around_the_line_boundaries(B, oracle_lib, policy, fanout, layout):
    # nodes of 0 to 71 edges with ties, queried at, just before and just after every time, in one large batch
    rng = np.random.default_rng(fanout)
    num_nodes = 72
    src = rng.permutation(np.repeat(np.arange(num_nodes, dtype=np.int32), np.arange(num_nodes)))
    ts = np.sort(rng.integers(0, 300, len(src))).astype(np.float32)
    st = W.Stream(num_nodes, src, rng.integers(0, num_nodes, len(src), dtype=np.int32), ts, 37)
    wl = W.Workload("degrees", 0, [st], fanout=fanout, tau=48)
    times = np.unique(ts)
    at = np.concatenate([times, np.nextafter(times, np.float32(-np.inf)), np.nextafter(times, np.float32(np.inf)), [-1.0, 1e9]]).astype(np.float32)
    targets, t_end = (a.ravel() for a in np.meshgrid(np.arange(num_nodes, dtype=np.int32), at))
    targets, t_end = (np.ascontiguousarray(np.resize(a, max(len(a), (1 << 16) + 9))) for a in (targets, t_end))
    t_start = (t_end - np.float32(40.0)).astype(np.float32)
    adjs = [oracle_lib.Adjacency(num_nodes, src, st.dst, ts)]
    for incl in (0, 1):
        plan = build_plan(B, wl, policy, incl, seed=9)
        for tb in (None, t_start):
            ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, policy, incl, 9, adjs=adjs)
            assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, f"incl={incl} start={tb is not None}")
        plan.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("policy", [0, 1])
def test_uneven_instances(B, oracle_lib, wide, policy, layout):
    rng = np.random.default_rng(5)
    I, nodes = 150, 40
    streams = [mixed_stream(100 + i, nodes, int(rng.integers(1, 400)), 64, ties=i % 2 == 0) for i in range(I)]
    wl = W.Workload("instances", 0, streams, fanout=10, tau=16)
    plan = build_plan(B, wl, policy, seed=4, flags=B.TNS_FLAG_WIDE_POSITIONS if wide else 0)
    adjs = [oracle_lib.Adjacency(s.num_nodes, s.src, s.dst, s.ts) for s in streams]
    # several instances inside a wave, none, exactly a wave, several tiles; small and large batches
    for sizes in (rng.choice([0, 1, 2, 7, 63, 64, 65, 300], I), np.where(np.arange(I) % 3 == 0, 0, rng.integers(1, 1400, I))):
        if sizes.sum() > 20_000:
            sizes[-1] += max(0, (1 << 16) + 5 - int(sizes.sum()))
        rowptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        parts = [W.random_queries(int(i), s, int(m)) for i, (s, m) in enumerate(zip(streams, sizes))]
        targets, t_start, t_end = (np.concatenate([q[k] for q in parts]) for k in range(3))
        for tb in (None, t_start):
            ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, rowptr, 10, policy, 0, 4, adjs=adjs)
            assert_same(gpu_sample(plan, targets, tb, t_end, rowptr), ref, oracle_lib, f"Q={len(targets)} start={tb is not None}")
    plan.close()


@pytest.mark.parametrize("policy", [0, 1])
def test_bounded_wait_ends(B, layout, policy):
    # as in test_gpu_parity.py: the tile tickets start at 1, so tile 0 never exists and the look-back ends by its bound
    import torch
    st = W.tiny_stream(17, 70_000, 500, 4096, ties=False)
    plan = build_plan(B, W.Workload("tiny", 0, [st], fanout=10, tau=48), policy, flags=B.TNS_TEST_FLAG_LOST_TILE)
    d_t, d_e = torch.from_numpy(st.src).cuda(), torch.from_numpy(st.ts).cuda()
    t0 = time.time()
    out = plan.run(d_t, None, d_e)
    torch.cuda.synchronize()
    assert time.time() - t0 < 60
    assert plan.status(out["workspace"]), "the time-out must be reported"
    assert int(out["rowptr"][-1].item()) == 0, "after a time-out the dense total reads 0"
    plan.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("fanout,incl", [(1, 0), (6, 1), (10, 0), (11, 0), (16, 1), (33, 0), (64, 0)])
def test_windows_inside_blocks_of_every_size(B, oracle_lib, wide, fanout, incl):
    # node v gets a block of v + 1 edges per batch (one per batch: fixed sizing would merge them), so that both window ends
    # fall into blocks of 1 to 40 slots at every position: all lanes of a wave then have two searches, 128 requests, some of
    # one slot, some of more than sixteen; times repeat
    nodes, batches = 40, 5
    rng = np.random.default_rng(fanout)
    src = np.concatenate([rng.permutation(np.repeat(np.arange(nodes, dtype=np.int32), np.arange(1, nodes + 1))) for _ in range(batches)])
    batch = len(src) // batches
    ts = np.sort(rng.integers(0, len(src) // 3, len(src))).astype(np.float32)
    st = W.Stream(nodes, src, rng.integers(0, nodes, len(src), dtype=np.int32), ts, batch)
    wl = W.Workload("blocks", 0, [st], fanout=fanout, tau=1)
    plan = build_plan(B, wl, 0, incl, flags=B.TNS_FLAG_WIDE_POSITIONS if wide else 0)
    Q = (1 << 16) + 65
    targets = (np.arange(Q) % nodes).astype(np.int32)
    t_end = rng.uniform(-2, len(src) // 3 + 2, Q).astype(np.float32)
    t_end[::3] = np.round(t_end[::3])
    t_start = np.round(t_end - rng.uniform(0, len(src) // 6, Q)).astype(np.float32)
    adjs = [oracle_lib.Adjacency(nodes, src, st.dst, ts)]
    for tb in (t_start, None):
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, 0, incl, 0, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, f"start={tb is not None}")
    plan.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("fanout", [1, 10, 20, 32, 33, 64])
def test_padded_rows_only_where_the_window_start_may_not_matter(B, oracle_lib, wide, fanout):
    # without the dense outputs; four to eight blocks of v + 1 edges per node v, queried at and around every time with windows of
    # all lengths: the blocks before the one with the window's start hold fewer than, exactly and more than the fan-out.  The
    # fan-outs give workgroups of four, three, two and one wave
    nodes = 36
    rng = np.random.default_rng(fanout)
    src = np.concatenate([rng.permutation(np.repeat(np.arange(b % 2, nodes, 1 + b % 2, dtype=np.int32), np.arange(b % 2, nodes, 1 + b % 2) + 1))
                          for b in range(8)])
    sizes = [int((np.arange(b % 2, nodes, 1 + b % 2) + 1).sum()) for b in range(8)]
    ts = np.sort(rng.integers(0, len(src) // 2, len(src))).astype(np.float32)
    dst = rng.integers(0, nodes, len(src), dtype=np.int32)
    st = W.Stream(nodes, src, dst, ts, len(src))
    wl = W.Workload("starts", 0, [st], fanout=fanout, tau=1)
    plan = B.Plan(nodes, fanout, block_threshold=1, flags=B.TNS_FLAG_WIDE_POSITIONS if wide else 0)
    lo = 0
    for m in sizes:
        plan.add_edges(src[lo:lo + m], dst[lo:lo + m], ts[lo:lo + m])
        lo += m
    plan.commit()
    Q = (1 << 17) + 65
    targets = rng.integers(0, nodes, Q, dtype=np.int32)
    t_end = ts[rng.integers(0, len(ts), Q)] + rng.integers(-1, 2, Q).astype(np.float32)
    t_start = (t_end - rng.integers(0, len(src) // 2, Q)).astype(np.float32)
    adjs = [oracle_lib.Adjacency(nodes, src, dst, ts)]
    for tb in (t_start, None):
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, 0, 0, 0, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end, compact=False), ref, None, f"start={tb is not None}")
    plan.close()
