"""Host code of libtg.so that only runs with a device (launch shapes, what
follows a failed allocation), on the CPU: a process per test loads the library
over the runtime of fake_hip.c, whose kernels do nothing."""
import os
import subprocess
import sys

import pytest

import paper_1312_3018_amd as tg

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys, time
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
OK, ENOMEM, EDEVICE, SYMMETRIC = 0, {enomem}, {edevice}, {symmetric}
for f, t in (("fake_thread_limit", ctypes.c_uint64), ("fake_malloc_limit", ctypes.c_size_t)):
    getattr(fake, f).argtypes = [t]
fake.fake_mark_copies.argtypes = [ctypes.c_size_t, ctypes.c_size_t]
fake.fake_most_threads.restype = ctypes.c_uint64
lib.tg_last_error.restype = ctypes.c_char_p
p64, p32 = np.ctypeslib.ndpointer(np.int64), np.ctypeslib.ndpointer(np.int32)
vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
lib.graph_load_csr.argtypes = [i64, i64, p64, p32, vp, ctypes.c_uint32, vp, ctypes.POINTER(vp)]
lib.partition_by_degree.argtypes = [vp, ctypes.c_int, ctypes.c_double, ctypes.c_uint64, ctypes.c_char_p,
                                    ctypes.POINTER(vp)]
lib.bfs.argtypes = [vp, p32, i32, vp, vp, vp]
for f in (lib.sssp, lib.bfs_batched, lib.sssp_batched, lib.bc, lib.bc_batched):
    f.argtypes = [vp, p32, i32, vp, vp]
lib.cc.argtypes = [vp, vp, vp]
lib.pagerank.argtypes = [vp, ctypes.c_float, i32, i32, vp, vp]
lib.partition_free.argtypes = [vp]
lib.server_create.argtypes = [ctypes.c_char_p, ctypes.POINTER(vp)]
lib.server_add_graph.argtypes = [vp, vp, ctypes.POINTER(i32)]
lib.server_submit.argtypes = [vp, i32, i32, i32, vp, ctypes.POINTER(ctypes.c_uint64)]
lib.server_wait.argtypes = [vp, ctypes.c_uint64, i64, vp]
lib.server_destroy.argtypes = [vp]
BUF = 4096  # an address no kernel writes to


def path(n, length, weight=300, tuning=b"{{}}", symmetric=True, share=0.0):
    "A partition of n vertices, the first `length` of them a path."
    deg = np.zeros(n + 1, dtype=np.int64)
    deg[1:length + 1] = 2
    deg[1] = deg[length] = 1
    off = np.cumsum(deg)
    i = np.arange(length)
    col = np.sort(np.stack([i - 1, i + 1], 1), 1).ravel()
    col = np.ascontiguousarray(col[(col >= 0) & (col < length)], dtype=np.int32)
    w = np.full(col.size, weight, dtype=np.int32)
    G, P = vp(), vp()
    check(lib.graph_load_csr(n, col.size, off, col, w.ctypes.data, SYMMETRIC if symmetric else 0, None,
                             ctypes.byref(G)))
    check(lib.partition_by_degree(G, 0, share, 0, tuning, ctypes.byref(P)))
    return P


def roots(k):
    return np.arange(k, dtype=np.int32)


def check(rc, want=OK):
    assert rc == want, (rc, lib.tg_last_error())
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    tg.require_native()
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", "-o", so,
                    os.path.join(HERE, "fake_hip.c")], check=True)
    prelude = PRELUDE.format(enomem=tg.TG_ENOMEM, edevice=tg.TG_EDEVICE, symmetric=tg.TG_SYMMETRIC)

    def go(script):
        r = subprocess.run([sys.executable, "-c", prelude + script, so, tg.LIB_PATH], capture_output=True, text=True,
                           timeout=110)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


# ------------------------------------------------------------ launch shapes

@pytest.mark.parametrize("symmetric", [True, False])
def test_grids_fit_every_vertex_count(run, symmetric):
    """A launch's threads are counted in 32 bits and V may be 2^31 - 1: past a
    fixed number of blocks no launch takes more than two threads per vertex
    (that number is 2^23 for the clearing of a retired slot's distances)."""
    run(f"""
n = 1 << 23
P = path(n, 100, symmetric={symmetric})
fake.fake_thread_limit(2 * n + 1)
for k in (1, 2, 64):
    check(lib.bfs_batched(P, roots(k), k, BUF, None))
    check(lib.sssp_batched(P, roots(k), k, BUF, None))
    check(lib.bfs(P, roots(k), k, BUF, None, None))
    check(lib.bfs(P, roots(k), k, BUF, BUF, None))
    check(lib.sssp(P, roots(k), k, BUF, None))
    check(lib.bc(P, roots(k), k, BUF, None))
    check(lib.bc_batched(P, roots(k), k, BUF, None))
check(lib.cc(P, BUF, None))
check(lib.pagerank(P, 0.85, 2, 0, BUF, None))
assert fake.fake_most_threads() >= n
""")


def test_grid_of_the_released_distances(run):
    """A thread per distance where 64 of them a vertex are 2^32 and more."""
    run("""
P = path((1 << 26) + 5, 100)
check(lib.sssp_batched(P, roots(2), 2, BUF, None))
assert 1 << 26 < fake.fake_most_threads() <= 1 << 31
""")


# ------------------------------------------------------------ hybrid split

def test_exchange_time_is_that_of_whole_messages(run):
    """exchange_ms of messages moved by a kernel: from the first block's start
    to the last block's end, for messages of one block and of eight."""
    run("""
import json
fake.fake_message_ticks.restype = ctypes.c_uint64
n = 60000
P = path(n, n, share=0.5)
check(lib.pagerank(P, 0.85, 10, 0, BUF, None))
buf = ctypes.create_string_buffer(4096)
lib.tg_last_stats(buf, 4096)
st = json.loads(buf.value)
ticks = fake.fake_message_ticks()
assert ticks > 10 * 800 and abs(st["exchange_ms"] - ticks / 1e5) < 1e-9, (st, ticks)
""")


# ---------------------------------------------------- errors while serving

# Copies of the engine's control block (its plan, 104 bytes, then the
# frontiers' sums) are marked, so that every slot has a frontier for ever.
SERVE = """
PLAN = 104
CONTROL = PLAN + 2 * 8 * 64 * 8
n = 1 << 16
P = path(n, 100)
S, gid, t = vp(), i32(), ctypes.c_uint64()
check(lib.server_create(None, ctypes.byref(S)))
check(lib.server_add_graph(S, P, ctypes.byref(gid)))


def submit(kind, k):
    out = []
    for r in range(k):
        check(lib.server_submit(S, gid, kind, r, BUF, ctypes.byref(t)))
        out.append(t.value)
    return out


def results(tickets):
    return [lib.server_wait(S, x, 10 * 1000 * 1000, None) for x in tickets]
"""


def test_server_query_ends_when_its_levels_find_no_room(run):
    """The rows for levels past a byte are made when a search gets there; with
    no memory for them the lane's queries end with TG_ENOMEM, and later ones
    are served."""
    run(SERVE + """
fake.fake_malloc_limit(n * 256)
fake.fake_mark_copies(CONTROL, PLAN)
assert results(submit(0, 3)) == [ENOMEM] * 3
fake.fake_mark_copies(0, 0)
assert results(submit(0, 70)) == [OK] * 70
lib.server_destroy(S)
""")


@pytest.mark.parametrize("kind", [0, 1])
def test_server_query_ends_when_a_superstep_fails(run, kind):
    run(SERVE + f"""
assert results(submit({kind}, 2)) == [OK] * 2
fake.fake_mark_copies(CONTROL, PLAN)
tickets = submit({kind}, 3)
time.sleep(0.3)  # all three in slots
fake.fake_failing_syncs(1)
assert results(tickets) == [EDEVICE] * 3
fake.fake_mark_copies(0, 0)
assert results(submit({kind}, 70)) == [OK] * 70
lib.server_destroy(S)
""")


# --------------------------------------------------- allocations that fail

@pytest.mark.parametrize("call", ["lib.bfs(P, roots(1), 1, BUF, None, None)", "lib.sssp(P, roots(1), 1, BUF, None)"])
def test_pinned_memory_that_fails_leaves_no_half_made_scratch(run, call):
    """The few-launch searches without their pinned memory: the call takes the
    next route, and the one after it finds no half-made scratch."""
    run(f"""
for k in range(4):
    P = path(1000, 100)
    fake.fake_host_mallocs(k)
    check({call})
    fake.fake_host_mallocs(-1)
    check({call})
    lib.partition_free(P)
""")


def test_workspace_that_failed_to_grow_is_made_again(run):
    """A retuned partition needs more room for hubs; wherever that fails, the
    next call must not take the buffers given back."""
    run("""
lib.partition_retune.argtypes = [vp, ctypes.c_char_p]
failed = 0
for k in range(24):
    P = path(1000, 1000)
    check(lib.cc(P, BUF, None))
    full = fake.fake_live_mallocs()
    check(lib.partition_retune(P, b'{"hub_min_deg": 2, "block_min_deg": 2, "wave_min_deg": 2, "g16_min_deg": 2, "g4_min_deg": 2}'))
    fake.fake_mallocs(k)
    failed += lib.cc(P, BUF, None) == ENOMEM
    fake.fake_mallocs(-1)
    check(lib.cc(P, BUF, None))
    assert fake.fake_live_mallocs() == full, k
    lib.partition_free(P)
assert failed > 15
""")


@pytest.mark.parametrize("part,call", [
    ("path(1000, 100)", "lib.bfs(P, roots(3), 3, BUF, BUF, None)"),  # a workgroup a root
    ("path(70000, 100)", "lib.bfs(P, roots(2), 2, BUF, None, None)"),  # the engine
    ("path(1000, 100)", "lib.sssp(P, roots(1), 1, BUF, None)"),  # rounds
    ("path(70000, 100)", "lib.sssp(P, roots(40), 40, BUF, None)"),  # the engine
    ("path(1000, 100)", "lib.bc(P, roots(2), 2, BUF, None)"),  # the chain
    ("path(1000, 100)", "lib.pagerank(P, 0.85, 2, 0, BUF, None)"),  # slices, whole
    ("path(1000, 100, tuning=b'{\"pr_whole\": 0}')", "lib.pagerank(P, 0.85, 2, 0, BUF, None)"),  # slices by class
])
def test_route_without_room_falls_back(run, part, call):
    """Whichever allocation of a route's own scratch fails, the call takes the
    route that needs less, and a later call can take the first one."""
    run(f"""
k, again = 0, []
while True:
    P = {part}
    check(lib.cc(P, BUF, None))  # the workspace every route shares
    fake.fake_mallocs(k)
    check({call})
    reached = fake.fake_mallocs_left() < 0
    fake.fake_mallocs(-1)
    check({call})
    again.append(fake.fake_live_mallocs())
    lib.partition_free(P)
    if not reached:
        break
    k += 1
assert k >= 3, k
assert min(again) >= again[-1], again  # the first route's scratch was made after all
""")


def test_buckets_without_room_fall_back(run):
    """Shared buckets (eight roots' rows at once) give way to single searches."""
    run("""
n = 100000
P = path(n, 100, weight=200, tuning=b'{"sssp_batch_roots": 64}')
fake.fake_malloc_limit(16 * n)
check(lib.sssp(P, roots(8), 8, BUF, None))
""")
