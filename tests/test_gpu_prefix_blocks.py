"""Recent policy over the prefix layout: nodes with none to many blocks outside the prefix, window ends in every line of it."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from _harness import assert_same, gpu_sample, oracle_sample

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2311_17410_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("fanout,incl,tau", [(1, 0, 8), (7, 1, 8), (10, 0, 8), (10, 1, 48), (11, 0, 20), (40, 1, 8), (64, 0, 48)])
def test_blocks_outside_the_prefix(B, oracle_lib, wide, fanout, incl, tau):
    # node v has v edges, one per batch: with a threshold of 8 its blocks fill 32 slots of the prefix and further ones lie outside,
    # up to ten of them; times repeat, and every query time is an edge's, just before or just after one
    nodes = 112
    src = np.concatenate([np.arange(b + 1, nodes, dtype=np.int32) for b in range(nodes - 1)])
    rng = np.random.default_rng(tau)
    ts = np.repeat(np.sort(rng.integers(0, 160, nodes - 1)), np.arange(nodes - 1, 0, -1)).astype(np.float32)
    st = W.Stream(nodes, src, rng.integers(0, nodes, len(src), dtype=np.int32), ts, 1)
    wl = W.Workload("prefix", 0, [st], fanout=fanout, tau=tau)
    plan = B.Plan(nodes, fanout, block_threshold=tau, inclusive_end=incl,
                  flags=B.TNS_FLAG_PREFIX_LAYOUT | (B.TNS_FLAG_WIDE_POSITIONS if wide else 0))
    ends = np.cumsum(np.arange(nodes - 1, 0, -1))
    for lo, hi in zip(np.concatenate([[0], ends[:-1]]), ends):
        B.tns_add_edges(plan.handle, 0, st.src[lo:hi], st.dst[lo:hi], st.ts[lo:hi], None)
    plan.commit()
    times = np.unique(ts)
    at = np.concatenate([times, np.nextafter(times, np.float32(-np.inf)), np.nextafter(times, np.float32(np.inf)), [-1.0, 1e9]]).astype(np.float32)
    targets, t_end = (np.ascontiguousarray(a.ravel()) for a in np.meshgrid(np.arange(nodes, dtype=np.int32), at))
    adjs = [oracle_lib.Adjacency(nodes, src, st.dst, ts)]
    for width in (None, 3.0, 25.0, 90.0):
        tb = None if width is None else np.where(rng.random(len(t_end)) < 0.5, np.round(t_end - width), t_end - width).astype(np.float32)
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, 0, incl, 0, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, f"width {width}")
        assert_same(gpu_sample(plan, targets, tb, t_end, compact=False), ref, None, f"padded only, width {width}")
    gone = rng.random(len(src)) < 0.3
    B.tns_delete_edges(plan.handle, 0, src[gone], np.flatnonzero(gone).astype(np.int32))
    plan.commit()
    adjs = [oracle_lib.Adjacency(nodes, src, st.dst, ts, present=(~gone).astype(np.uint8))]
    for tb in (None, (t_end - np.float32(40.0)).astype(np.float32)):
        ref = oracle_sample(oracle_lib, wl, targets, tb, t_end, None, fanout, 0, incl, 0, adjs=adjs)
        assert_same(gpu_sample(plan, targets, tb, t_end), ref, oracle_lib, "deleted edges")
    plan.close()
