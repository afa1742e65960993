"""Kernels with a query per lane: their workgroups have one to sixteen waves, by the batch.  Both sides of every line of that rule: which
sizes are taken (the launched grids, without a GPU), and the results against the oracle."""
import numpy as np
import pytest

from paper_2311_17410_amd import workloads as W
from test_host_paths import run  # noqa: F401

# layout's flag, policy, fan-out, whether the padding is removed, and the lines: the first batch size beyond it, waves per workgroup on
# either side
LINES = [
    (0, 0, 10, True, [(65_537, 4, 2), (81_921, 2, 8), (131_073, 8, 4), (180_225, 4, 16), (229_377, 16, 8), (326_657, 8, 16)]),
    (0, 0, 20, True, [(65_537, 4, 2), (81_921, 2, 8), (457_729, 8, 16)]),
    (0, 0, 64, True, [(65_537, 2, 4), (228_865, 4, 8)]),
    (0, 1, 10, True, [(49_153, 1, 2), (81_921, 2, 4)]),
    (128, 0, 10, True, [(16_385, 1, 2), (32_769, 2, 4), (65_537, 4, 2), (81_921, 2, 8), (131_073, 8, 4), (180_225, 4, 16), (229_377, 16, 8), (326_657, 8, 16)]),
    (128, 1, 10, True, [(16_385, 1, 2), (32_769, 2, 4), (65_537, 4, 2), (81_921, 2, 8), (131_073, 8, 4), (180_225, 4, 8)]),
    (128, 1, 20, True, [(65_409, 1, 2), (130_817, 2, 4), (261_633, 4, 8)]),
    (0, 0, 10, False, [(65_409, 1, 2), (130_817, 2, 4)]),
    (128, 1, 20, False, [(65_409, 1, 2)]),
]


@pytest.mark.parametrize("flags,policy,fanout,dense,lines", LINES)
def test_waves_of_a_workgroup(run, flags, policy, fanout, dense, lines):  # noqa: F811
    # (the uniform policy's line at 49153 queries is where the kernel with sixteen lanes per query ends, whose last workgroups have 64 queries)
    run(f"""
p = B.Plan(1000, {fanout}, policy={policy}, flags={flags})
B.tns_commit(p.handle)
for line, before, after in {lines}:
    for Q, waves in ((line - 1, before), (line, after)):
        if {dense}: B.tns_run(p.handle, Q, 256, 0, 256, 0, 0, 256, 256, 256, 256, 256, 256, 256, 256, 256, B.tns_workspace(p.handle, Q), 0)
        else: B.tns_run(p.handle, Q, 256, 0, 256, 0, 0, 256, 256, 256, 256)
        assert fake.fake_grid() == (Q + 64 * waves - 1) // (64 * waves), (Q, waves, fake.fake_grid())
""")


@pytest.mark.gpu
@pytest.mark.parametrize("flags,policy,fanout,dense,lines", LINES)
def test_results_on_both_sides(oracle_lib, flags, policy, fanout, dense, lines):
    import torch
    from paper_2311_17410_amd import binding as B
    rng = np.random.default_rng(fanout + policy)
    nodes, n = 2000, 50_000
    src = (rng.zipf(1.2, n) % (nodes - 5)).astype(np.int32)
    dst = rng.integers(0, nodes, n, dtype=np.int32)
    ts = np.sort(rng.integers(0, n // 10, n)).astype(np.float32)
    bounds = list(range(0, n, 2500)) + [n]
    plan = B.Plan(nodes, fanout, policy=policy, block_threshold=48, seed=3, flags=flags)
    for lo, hi in zip(bounds[:-1], bounds[1:]):
        plan.add_edges(src[lo:hi], dst[lo:hi], ts[lo:hi])
    plan.commit()
    targets, t_start, t_end = W.random_queries(3, W.Stream(nodes, src, dst, ts, 2500), lines[-1][0])
    adj = oracle_lib.Adjacency(nodes, src, dst, ts, batch_rowptr=bounds)
    ref = adj.sample(targets, t_start, t_end, fanout, policy=policy, seed=3)
    adj.close()
    rowptr, *packed = oracle_lib.compact(ref)
    want = {k: torch.from_numpy(getattr(ref, k).reshape(-1)).cuda() for k in ("nbr", "eid", "ts", "count")}
    want.update(rowptr=torch.from_numpy(rowptr).cuda(), **{k: torch.from_numpy(a).cuda() for k, a in zip(("cmp_nbr", "cmp_eid", "cmp_ts"), packed)})
    dq = [torch.from_numpy(a).cuda() for a in (targets, t_start, t_end)]
    for Q in sorted({q for line, *_ in lines for q in (line - 1, line)}):
        out = plan.run(*(t[:Q] for t in dq), compact=dense)
        size = dict(count=Q, rowptr=Q + 1, nbr=Q * fanout, eid=Q * fanout, ts=Q * fanout, **dict.fromkeys(("cmp_nbr", "cmp_eid", "cmp_ts"), int(rowptr[Q])))
        for name, m in size.items():
            if dense or name in ("count", "nbr", "eid", "ts"):
                assert torch.equal(out[name].reshape(-1)[:m], want[name][:m]), (Q, name)
        assert not dense or not plan.status(out["workspace"])
    plan.close()
