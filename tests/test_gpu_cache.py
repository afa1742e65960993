"""GPU parity of the vectorised feature cache against its oracle: returned rows and hit flags,
and the whole cache state (id per slot, scores, rows, ring) after every batch, bit for bit."""
import numpy as np
import pytest

from oracle import cache_oracle as CO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def KB():
    import torch
    assert torch.cuda.is_available()
    from paper_2311_17410_amd import cache_binding
    cache_binding.lib()
    return cache_binding


def run_sequence(KB, policy, n, cap, dim, lam, batches, seed, check_state_every=1, prepare=None):
    import torch
    dev = torch.device("cuda", 0)
    store = np.random.default_rng(seed).standard_normal((n, dim)).astype(np.float32)
    d_store = torch.from_numpy(store).to(dev)
    ref = CO.VectorCache(n, cap, dim, policy, lam)
    gpu = KB.Cache(n, cap, dim, policy, lam)
    if prepare:
        prepare(gpu)
    for it, ids in enumerate(batches):
        ids = np.asarray(ids, np.int32)
        out, hit = gpu.fetch(torch.from_numpy(ids).to(dev), d_store)
        valid = (ids >= 0) & (ids < n)
        r_out, r_hit = ref.fetch(ids[valid], store)
        out, hit = out.cpu().numpy(), hit.cpu().numpy().astype(bool)
        assert np.array_equal(out[valid].view(np.int32), r_out.view(np.int32)), f"rows, batch {it}"
        assert np.all(out[~valid] == 0) and not hit[~valid].any()
        assert np.array_equal(hit[valid], r_hit), f"hit flags, batch {it}"
        if it % check_state_every == 0 or it == len(batches) - 1:
            st = gpu.save()
            assert np.array_equal(st["id_of"], ref.id_of), f"id per slot, batch {it}"
            occ = ref.id_of >= 0
            if policy != CO.FIFO:
                assert np.array_equal(st["score"], ref.score), f"scores, batch {it}"
            else:
                assert st["ring"] == ref.ring
            assert np.array_equal(st["rows"][occ].view(np.int32), ref.data[occ].view(np.int32)), f"cached rows, batch {it}"
    s = gpu.stats()
    assert (s["hits"], s["misses"], s["replaced"]) == (ref.hits, ref.misses, ref.replaced)
    return gpu, ref, store, d_store


@pytest.mark.parametrize("policy", [CO.LRU, CO.LFU, CO.FIFO])
@pytest.mark.parametrize("dim", [4, 7, 172])
def test_small_batches_every_state(KB, policy, dim):
    rng = np.random.default_rng(10 + policy)
    n, cap = 300, 37
    batches = [(rng.zipf(1.2, int(rng.integers(1, 70))) % n) for _ in range(120)]
    batches[5] = np.array([-1, 3, n, 3, 2 ** 31 - 1], np.int64)          # ids out of range return zero rows
    gpu, *_ = run_sequence(KB, policy, n, cap, dim, 0.2, batches, 1)
    gpu.close()


@pytest.mark.parametrize("policy", [CO.LRU, CO.LFU, CO.FIFO])
def test_large_batches_and_lambda_one(KB, policy):
    rng = np.random.default_rng(20 + policy)
    n, cap = 200_000, 5_000
    batches = [(rng.zipf(1.1, 40_000) % n) for _ in range(8)]
    gpu, *_ = run_sequence(KB, policy, n, cap, 16, 1.0, batches, 2)
    gpu.close()
    batches = [(rng.zipf(1.1, 30_000) % n) for _ in range(8)]
    gpu, *_ = run_sequence(KB, policy, n, cap, 16, 0.2, batches, 3)
    gpu.close()


def test_paper_scale_shapes_and_restore(KB):
    import torch
    # edge-feature shaped rows (172 floats), cache of 1 % of the ids, batches of "thousands" (section 4.3)
    rng = np.random.default_rng(30)
    n, cap = 1_000_000, 10_000
    batches = [(rng.zipf(1.05, 60_000) % n) for _ in range(6)]
    gpu, ref, store, d_store = run_sequence(KB, CO.LRU, n, cap, 172, 0.2, batches, 4, check_state_every=3)
    # restoration (section 4.3): save at the start of a round, pollute, restore: same state as saved
    saved = gpu.save()
    dev = torch.device("cuda", 0)
    for _ in range(3):
        gpu.fetch(torch.from_numpy((rng.integers(0, n, 50_000)).astype(np.int32)).to(dev), d_store)
    gpu.restore(saved)
    again = gpu.save()
    for k in ("id_of", "score", "rows"):
        assert np.array_equal(again[k], saved[k])
    ids = (rng.zipf(1.05, 20_000) % n).astype(np.int32)
    out, hit = gpu.fetch(torch.from_numpy(ids).to(dev), d_store)
    r_out, r_hit = ref.fetch(ids, store)
    assert np.array_equal(out.cpu().numpy(), r_out) and np.array_equal(hit.cpu().numpy().astype(bool), r_hit)
    gpu.close()


@pytest.mark.parametrize("seed", range(40))
def test_random_configuration(KB, seed):
    # seeded differential test over capacities, row widths, replacement caps, batch sizes and id distributions
    rng = np.random.default_rng(500 + seed)
    n = int(rng.choice([1, 5, 60, 1000, 20_000]))
    cap = int(rng.integers(1, max(2, min(n, 3000) + 1)))
    dim = int(rng.choice([1, 3, 4, 8, 33, 172]))
    lam = float(rng.choice([0.01, 0.2, 0.5, 1.0]))
    policy = int(rng.integers(0, 3))
    batches = []
    for _ in range(int(rng.integers(3, 25))):
        b = int(rng.integers(1, 3000))
        ids = (rng.zipf(1.15, b) % n) if rng.integers(0, 2) else rng.integers(0, n, b)
        if rng.integers(0, 5) == 0:
            ids = ids.astype(np.int64)
            ids[rng.integers(0, b)] = n + int(rng.integers(0, 10))      # an id outside the range
        batches.append(ids)
    gpu, *_ = run_sequence(KB, policy, n, cap, dim, lam, batches, seed)
    gpu.close()


# A fetch is three launches on the caller's stream, or (caches of more than 65536 entries under LRU and LFU, more than 2^20
# ids, more than 2^24 pieces of rows) forks its update onto a stream of the cache's own and joins it again.
@pytest.mark.parametrize("policy,n,cap,dim,b", [(CO.LRU, 5000, 400, 20, 3000), (CO.LFU, 5000, 400, 20, 3000), (CO.FIFO, 5000, 400, 20, 3000),
                                                (CO.LRU, 300_000, 70_000, 20, 30_000), (CO.LFU, 300_000, 70_000, 20, 30_000),
                                                (CO.FIFO, 60_000, 5000, 4, (1 << 20) + 1)])
def test_fetch_replayed_from_a_hip_graph(KB, policy, n, cap, dim, b):
    # captured once and replayed, every replay must behave like one more fetch of the same batch (state and rows checked
    # each time)
    import torch
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(77)
    store = rng.standard_normal((n, dim)).astype(np.float32)
    d_store = torch.from_numpy(store).to(dev)
    ids = (rng.zipf(1.1, b) % n).astype(np.int32)
    d_ids = torch.from_numpy(ids).to(dev)
    ref = CO.VectorCache(n, cap, dim, policy, 0.2)
    gpu = KB.Cache(n, cap, dim, policy, 0.2)
    out = torch.empty((len(ids), dim), dtype=torch.float32, device=dev)
    hit = torch.empty(len(ids), dtype=torch.uint8, device=dev)
    gpu.fetch(d_ids, d_store, out, hit)                     # eager once (also allocates the workspace)
    ref.fetch(ids, store)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        gpu.fetch(d_ids, d_store, out, hit)
    for rep in range(3):
        out.zero_()
        assert float(d_store.sum().item()) == float(d_store.sum().item())     # unrelated eager work and a sync
        graph.replay()
        torch.cuda.synchronize()
        r_out, r_hit = ref.fetch(ids, store)
        assert np.array_equal(out.cpu().numpy(), r_out) and np.array_equal(hit.cpu().numpy().astype(bool), r_hit), rep
        st = gpu.save()
        assert np.array_equal(st["id_of"], ref.id_of), rep
        if policy != CO.FIFO:
            assert np.array_equal(st["score"], ref.score), rep
    del graph
    gpu.close()


@pytest.mark.parametrize("policy,cap,dim,b", [
    (CO.FIFO, 3000, 4, 1 << 20), (CO.FIFO, 3000, 4, (1 << 20) + 1),       # ids on either side of the line, the ring goes round
    (CO.LRU, 3000, 4, 1 << 20), (CO.LFU, 3000, 4, (1 << 20) + 1),
    (CO.LRU, 3000, 64, 1 << 18), (CO.FIFO, 3000, 256, 1 << 18), (CO.FIFO, 3000, 256, (1 << 18) + 1),     # 2^24 pieces and one row more
    (CO.FIFO, 3000, 17, 1_000_000), (CO.LRU, 3000, 17, 986_895), (CO.LRU, 3000, 17, 986_896),           # pieces of one float
    (CO.LRU, 65_536, 8, 90_000), (CO.LRU, 65_537, 8, 90_000), (CO.LFU, 70_000, 172, 90_000), (CO.LFU, 70_000, 7, 90_000)])
def test_both_sides_of_the_lines_between_the_two_forms(KB, policy, cap, dim, b):
    rng = np.random.default_rng(cap + dim)
    n = 100_000
    batches = [rng.zipf(1.05, b) % n, rng.integers(0, n, b), rng.zipf(1.05, 1 + b // 3) % n, rng.integers(-3, n + 3, b)]
    gpu, *_ = run_sequence(KB, policy, n, cap, dim, 0.5, batches, 5)
    gpu.close()


@pytest.mark.parametrize("policy", [CO.LRU, CO.LFU])
@pytest.mark.parametrize("cap", [1, 255, 4097, 40_001, 65_535, 65_536, 65_537])
def test_victims_among_scores_of_any_size(KB, policy, cap):
    # one workgroup holds the scores of up to 65536 entries and searches for the threshold: capacities around its chunks
    # and its end, scores close together, spread over 32 bits and at their extremes, replacement of one entry up to all
    import torch
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(900 + cap)
    n, dim = 2 * cap + 10, 3
    store = rng.standard_normal((n, dim)).astype(np.float32)
    d_store = torch.from_numpy(store).to(dev)
    spreads = [(-6, 0), (0, 2 ** 20), (-(2 ** 31) + 8, 2 ** 31 - 8), (2 ** 31 - 12, 2 ** 31 - 8), (5, 6)]
    for lam in (0.2, 1.0):
        ref, gpu = CO.VectorCache(n, cap, dim, policy, lam), KB.Cache(n, cap, dim, policy, lam)
        for it, (lo, hi) in enumerate(spreads):
            ref.score[:] = rng.integers(lo, hi, cap)
            gpu.restore(dict(id_of=ref.id_of, score=ref.score, rows=ref.data, ring=0))
            for b in (1, 1500, 1024, min(2 * cap, 90_000) + 1):
                ids = rng.integers(0, n, b).astype(np.int32)
                out, hit = gpu.fetch(torch.from_numpy(ids).to(dev), d_store)
                r_out, r_hit = ref.fetch(ids, store)
                assert np.array_equal(out.cpu().numpy(), r_out) and np.array_equal(hit.cpu().numpy().astype(bool), r_hit), (lam, it, b)
                st = gpu.save()
                assert np.array_equal(st["id_of"], ref.id_of) and np.array_equal(st["score"], ref.score), (lam, it, b)
        gpu.close()


@pytest.mark.parametrize("b", [32 * 1024, 32 * 1024 + 1])
@pytest.mark.parametrize("cap,lo,hi", [(300, -3, 0), (8193, -8, 0), (40_001, -9, 0), (40_001, -2, 0), (65_536, -1, 0), (65_536, -40, 0),
                                       (65_536, 2 ** 31 - 8, 2 ** 31 - 1), (57_345, 2 ** 31 - 20, 2 ** 31 - 9), (4097, -(2 ** 31), -(2 ** 31) + 9)])
def test_values_counted_while_ids_are_awaited(KB, b, cap, lo, hi):
    # from 33 tiles of ids on the eight lowest scores are counted beforehand: thresholds inside and beyond them, one value held by
    # every entry, values so high that places beyond the last entry are next to them
    import torch
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(cap)
    n, dim = 200_000, 2
    store = rng.standard_normal((n, dim)).astype(np.float32)
    d_store = torch.from_numpy(store).to(dev)
    for lam in (0.001, 0.2, 0.9, 1.0):
        ref, gpu = CO.VectorCache(n, cap, dim, CO.LRU, lam), KB.Cache(n, cap, dim, CO.LRU, lam)
        ref.score[:] = rng.integers(lo, hi, cap)
        gpu.restore(dict(id_of=ref.id_of, score=ref.score, rows=ref.data, ring=0))
        ids = rng.integers(0, n, b).astype(np.int32)
        out, hit = gpu.fetch(torch.from_numpy(ids).to(dev), d_store)
        r_out, r_hit = ref.fetch(ids, store)
        assert np.array_equal(out.cpu().numpy(), r_out) and np.array_equal(hit.cpu().numpy().astype(bool), r_hit), lam
        st = gpu.save()
        assert np.array_equal(st["id_of"], ref.id_of) and np.array_equal(st["score"], ref.score), lam
        gpu.close()


@pytest.mark.parametrize("policy", [CO.LRU, CO.LFU, CO.FIFO])
def test_tiles_that_do_not_hear_from_one_another(KB, policy):
    # the update of a batch numbers its missed ids with a chained scan over tiles of 1024 ids; no tile of this cache waits for
    # the others, as after a wait that ran into its bound: the update must be made all the same
    import ctypes
    no_wait = KB.lib().tns_test_cache_no_wait
    no_wait.argtypes, no_wait.restype = [ctypes.c_void_p], None
    rng = np.random.default_rng(60 + policy)
    n, cap = 50_000, 9_000
    sizes = (1, 1024, 1025, 2048, 5000, 70_001)
    gpu, *_ = run_sequence(KB, policy, n, cap, 5, 0.5, [rng.integers(0, n, b) for b in sizes], 9, prepare=lambda c: no_wait(c._h))
    gpu.close()


@pytest.mark.parametrize("policy", [CO.LRU, CO.LFU, CO.FIFO])
@pytest.mark.parametrize("dim", [1, 173, 1028, 4100])
def test_rows_of_every_width_and_updates_that_fall_short(KB, policy, dim):
    # rows of one piece, of no whole number of 16-byte pieces, and of more than the insertion and the gather hold at once; updates
    # that replace as many entries as allowed, fewer (most ids cached, or a batch of a few ids repeated), one and none
    rng = np.random.default_rng(dim + policy)
    n, cap = 2000, 300
    sizes = [500, 61, 60, 59, 400, 1, 700]
    batches = [rng.integers(0, n, b) for b in sizes]
    batches += [np.concatenate([batches[-1], rng.integers(0, n, k)]) for k in (0, 1, 20)] + [np.repeat(rng.integers(0, n, 7), 40)]
    run_sequence(KB, policy, n, cap, dim, 0.2, batches, 6)[0].close()


@pytest.mark.parametrize("rows", [24384, 24385, 24386, 49000])
def test_rows_gathered_beside_lookup_and_update(KB, rows):
    # 43 pieces a row: 2^20 pieces end inside row 24385
    rng = np.random.default_rng(rows)
    run_sequence(KB, CO.LRU, 60_000, 2000, 172, 0.2, [rng.zipf(1.1, rows) % 60_000 for _ in range(3)], 8)[0].close()


@pytest.mark.parametrize("dim,b", [(1, 1), (1, 2047), (1, 2048), (1, 2049), (3, 683), (4, 2049), (8, 1025), (12, 100_001), (172, 48), (172, 5000),
                                   (2049, 3)])
def test_rows_of_a_workgroup_looked_up_once(KB, dim, b):
    # more than 65536 entries: the rows are moved by a launch of their own, 2048 pieces a workgroup, so that there are rows that fill,
    # span and share workgroups, and as many rows as pieces
    rng = np.random.default_rng(b)
    n, cap = 70_000 if dim <= 172 else 65_600, 65_537
    batches = [rng.integers(0, n, b) for _ in range(3)]
    batches[1][rng.integers(0, b, 1 + b // 9)] = rng.choice([-1, n, 2 ** 31 - 1], 1 + b // 9)
    batches[2] = batches[0]
    gpu, *_ = run_sequence(KB, CO.LRU, n, cap, dim, 0.2, batches, 4, check_state_every=3)
    gpu.close()


@pytest.mark.parametrize("dim,b", [(1, 8191), (1, 8192), (1, 8193), (1, 10_000), (1, 16_385), (3, 5462), (4, 4097), (4, 12_289), (8, 2049), (173, 95)])
def test_pieces_shared_out_evenly_beside_the_update(KB, dim, b):
    # a cache of up to 65536 entries: the rows are moved beside the update, by as few workgroups as there are thousands of pieces, eight (or
    # four of 16 bytes) a thread, and each takes as many of them as the others: batches that fill one workgroup, and a few pieces more
    rng = np.random.default_rng(b)
    for policy in (CO.LRU, CO.FIFO):
        batches = [rng.integers(0, 70_000, b) for _ in range(3)]
        batches[1][rng.integers(0, b, 5)] = [-1, 70_000, 2 ** 31 - 1, 0, 69_999]
        run_sequence(KB, policy, 70_000, 3000, dim, 0.2, batches, 4, check_state_every=3)[0].close()
