"""Host paths around the kernels, without a GPU: the library runs in a process of its own on tests/fake_hip.c (device
memory with a limit, kernels that do nothing)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_set_limit.argtypes, fake.fake_used.restype = [C.c_size_t], C.c_size_t
sys.modules["torch"] = None                     # the binding does without it; its runtime stays out of the process
sys.path.insert(0, sys.argv[2])
from paper_2311_17410_amd import binding as B, cache_binding as KB
MiB = 1 << 20
def plan_of(mib):                               # a device-built store whose node table and builder state take `mib`
    p = B.Plan(mib * MiB // 216, 10, flags=B.TNS_FLAG_DEVICE_INGEST)      # 144 bytes a node, and room to grow by half
    B.tns_commit(p.handle)
    return p
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")])

    def go(body):
        p = subprocess.run([sys.executable, "-c", PRELUDE + body, so, ROOT], capture_output=True, text=True, timeout=120)
        assert p.returncode == 0, p.stdout + p.stderr
    return go


def test_memory_kept_for_the_next_plan(run):
    run("""
p = plan_of(100); in_use = fake.fake_used(); p.close()
assert 100 * MiB <= fake.fake_used() <= in_use            # kept
n = fake.fake_allocations(); p = plan_of(100)
assert fake.fake_allocations() - n <= 1                   # and used again (the status record is not kept)
p.close()
for mib in (300, 200, 150, 250): plan_of(mib).close()
assert fake.fake_used() <= 256 * MiB                      # bounded
B.tns_destroy(None)
assert fake.fake_used() == 0                              # given back
""")


def test_kept_memory_is_given_back_to_a_cache(run):
    run("""
fake.fake_set_limit(300 * MiB)
plan_of(180).close()
assert fake.fake_used() > 150 * MiB
c = KB.Cache(1000, 400_000, 128, KB.TNS_CACHE_LRU, 0.2)   # 195 MiB of rows
""")


def test_kept_memory_is_given_back_to_a_larger_plan(run):
    run("""
fake.fake_set_limit(300 * MiB)
plan_of(180).close()
p = plan_of(200)
try:
    plan_of(200)
    raise SystemExit("200 + 200 MiB of 300")
except B.TnsError as e:
    assert e.status == B.TNS_ENOMEM
p.close()
plan_of(200)
""")


@pytest.mark.parametrize("m", [100, 5000])
def test_a_plan_that_never_reaches_the_host_is_an_error(run, m):
    # the kernels do nothing here, so the record with the batch's plan does not come; whether the queued apply phase ran
    # is then not known, and the store takes no further batch
    run(f"""
p = plan_of(1)
src = C.create_string_buffer(4 * {m})
for status, text in ((B.TNS_EHIP, "did not reach the host"), (B.TNS_ESTATE, "create a new plan")):
    try:
        B.tns_add_edges_device(p.handle, 0, C.addressof(src), C.addressof(src), C.addressof(src), None, {m}, 0)
        raise SystemExit("accepted")
    except B.TnsError as e:
        assert e.status == status and text in str(e), str(e)
assert p.stats()["num_edges"] == 0
""")


@pytest.mark.parametrize("capacity", [7, 40_000, (1 << 26) + 12])
def test_no_more_entries_are_replaced_than_the_cache_has(run, capacity):
    # lambda 1 and a capacity that rounds up to 2^26 + 16 in 32 bits: the insertion, which ends a fetch, has a wave per entry
    # that may be replaced, four a workgroup, and a workgroup for the batch
    run(f"""
c = KB.tns_cache_create(1000, {capacity}, 1, KB.TNS_CACHE_FIFO, 1.0)
KB.tns_cache_fetch(c, 100, 256, 256, 256, 0, 256, KB.tns_cache_workspace(c, 100))      # (the kernels do nothing)
assert fake.fake_grid() == ({capacity} + 3) // 4 + 1, fake.fake_grid()
KB.tns_cache_destroy(c)
""")


@pytest.mark.parametrize("queries,fanout,policy,flags", [(1, 10, 0, 0), (20_000, 10, 1, 0), (1 << 18, 10, 0, 0), (1 << 17, 20, 1, 0), (5000, 10, 0, 128),
                                                         (1 << 16, 40, 1, 128)])
def test_the_scan_state_of_a_captured_call_is_cleared(run, queries, fanout, policy, flags):
    # a captured call runs again as it is, over what the replay before left: batches that otherwise need no cleared state get a
    # launch that clears it (one for all hops)
    run(f"""
p = B.Plan(1000, {fanout}, policy={policy}, flags={flags})
B.tns_commit(p.handle)
def launches(capture):
    fake.fake_capture(capture)
    n = fake.fake_launches()
    B.tns_run(p.handle, {queries}, 256, 0, 256, 0, 0, 256, 256, 256, 256, 256, 256, 256, 256, 256, B.tns_workspace(p.handle, {queries}), 0)
    m = fake.fake_launches()
    hop = dict.fromkeys([n for n, _ in B.tns_hop_buffers._fields_], 256)
    B.tns_run_khop(p.handle, [{fanout}, 1], float("inf"), {max(1, queries // fanout)}, 256, 0, 256, 0, 0, [hop, hop], 256,
                   B.tns_workspace_khop(p.handle, [{fanout}, 1], {max(1, queries // fanout)}), 0)
    return m - n, fake.fake_launches() - m
assert launches(0) == (1, 2) and launches(1) == (2, 3) and launches(2) == (2, 3) and launches(0) == (1, 2)
""")


def test_device_addresses_are_integers(run):
    # bytes, strings, arrays and pointer objects are no device addresses: a kernel would follow them into host memory
    run("""
p = B.Plan(1000, 10)
B.tns_commit(p.handle)
hop = dict.fromkeys([n for n, _ in B.tns_hop_buffers._fields_], 256)
calls = [(B.tns_run, [p.handle, 100, 256, 0, 256, 0, 0, 256, 256, 256, 256, 256, 256, 256, 256, 256, 1 << 20, 0]),
         (B.tns_run_static, [p.handle, 100, 256, 0, 256, 0, 0, 256, 256, 256, 256, 256, 256, 256, 256, 0]),
         (B.tns_run_khop, [p.handle, [10], 1.0, 100, 256, 0, 256, 0, 0, [hop], 256, 1 << 20, 0]),
         (B.tns_compact, [p.handle, 100, 256, 256, 256, 256, 256, 256, 256, 256, 256, 1 << 20, 0]),
         (B.tns_traffic_model, [p.handle, 100, 256, 0, 256, 0, 0, 256, 0]),
         (B.tns_hbm_probe, [0, False, 256, 512, 128, 0]), (B.tns_hbm_probe_mix, [False, 256, 128, 512, 128, 0])]
for call, args in calls:
    call(*args)
    # addresses, and what may be one: not the numbers of hops and queries, the window length, nor the flag
    first = next(i for i, a in enumerate(args) if type(a) is int and a >= 256)
    for i in [i for i in range(first, len(args)) if type(args[i]) is int and args[i] in (256, 512)] + [len(args) - 1]:
        for other in (b"12345678", "12345678", C.create_string_buffer(8), C.c_void_p(256), (C.c_int64 * 2)(1, 2), 1.5):
            try:
                call(*args[:i], other, *args[i + 1:])
            except (TypeError, C.ArgumentError):
                continue
            raise SystemExit(f"{call.__name__} takes {other!r} as argument {i}")
for name in hop:
    for other in (b"12345678", "12345678", C.create_string_buffer(8)):
        try:
            B.tns_run_khop(p.handle, [10], 1.0, 100, 256, 0, 256, 0, 0, [{**hop, name: other}], 256, 1 << 20, 0)
        except TypeError:
            continue
        raise SystemExit(f"{name} takes {other!r}")
B.tns_run(p.handle, 100, 256, None, 256, None, 0, 256, 256, 256, 256, 256, 256, 256, 256, 256, 1 << 20, None)      # NULL either way
""")


@pytest.mark.parametrize("policy,fanout", [(0, 10), (1, 64)])
def test_the_workspace_holds_the_states_of_the_tiles_and_no_more(run, policy, fanout):
    # a batch's tiles are as small with the workspace that tns_workspace asks for as with any larger one; where it asks for more than
    # the least, so does some batch of that size or smaller in the same workspace, and more queries never need less
    run(f"""
p = B.Plan(1000, {fanout}, policy={policy})
B.tns_commit(p.handle)
def grid(Q, size):
    B.tns_run(p.handle, Q, 256, 0, 256, 0, 0, 256, 256, 256, 256, 256, 256, 256, 256, 256, size, 0)
    return fake.fake_grid()
def least(Q):
    up = lambda n: (n + 255) // 256 * 256
    tiles = (Q + 1023) // 1024
    return max(up(4 * tiles) + up(8 * tiles) + 256, up(256 + 8 * ((Q + 63) // 64 + 1)))
before, more = 0, 0
for Q in list(range(1, 1100)) + [m + d for m in range(2048, 40_000, 512) for d in (-1, 0, 1)]:
    size = B.tns_workspace(p.handle, Q)
    assert size >= before and size >= least(Q), Q
    before = size
    assert grid(Q, size) == grid(Q, size + (1 << 20)), Q
    if size > least(Q):
        more = Q
        assert any(grid(q, size) > grid(q, size - 256) for q in (Q, 4096) if q <= Q), Q
assert 8192 < more < 1 << 14, more
""")


def test_records_kept_for_the_next_stores(run):
    # a device-built store's page-locked record is kept when the store is closed, sixteen at most, and given back with the rest
    run("""
def stores(n): return [plan_of(1) for _ in range(n)]
first = stores(20)
assert fake.fake_host_allocations() == fake.fake_host_blocks() == 20
for p in first: p.close()
assert fake.fake_host_blocks() == 16                      # four freed
again = stores(18)
assert fake.fake_host_allocations() == 22 and fake.fake_host_blocks() == 18      # sixteen of them kept ones
again[0].close()
B.tns_destroy(None)
assert fake.fake_host_blocks() == 17                      # the kept one; those in use stay
again[0] = plan_of(1)
for p in again: p.close()
assert fake.fake_host_blocks() == 16
B.tns_destroy(None)
assert fake.fake_host_blocks() == 0 and fake.fake_used() == 0
p = plan_of(1)
fake.fake_fail_synchronize(1)                             # work that may still write to it: not kept
p.close()
fake.fake_fail_synchronize(0)
assert fake.fake_host_blocks() == 0 and fake.fake_used() == 0
""")
