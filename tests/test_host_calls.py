"""The library's host code on a runtime without a GPU (fake_hip.c): what it launches, and what
it returns when a call into the runtime fails.  Each test runs in a process of its own, since
the library binds to the first runtime it meets."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
F.fake_launch_name.restype = C.c_char_p
F.fake_launch_arg0.restype = C.POINTER(C.c_uint64 * 8)
F.fake_fail_kernel.argtypes = [C.c_char_p]
L.vc_last_error.restype = C.c_char_p
P, u64, u32 = C.c_void_p, C.c_uint64, C.c_uint32
L.vc_trace_load.argtypes = [P, P, u64, u32, P, u32, C.POINTER(P)]
L.vc_check_small_noalloc.argtypes = [P, P, u64, u32, P, P, P, P, P]
for f in ("vc_check", "vc_sync", "vc_trace_free", "vc_ctx_destroy"):
    getattr(L, f).argtypes = [P]
def launches():
    return [(F.fake_launch_name(i).decode(), list(F.fake_launch_arg0(i).contents)) for i in range(F.fake_launches())]
def ok(rc):
    assert rc == 0, (rc, L.vc_last_error())
ctx = P()
ok(L.vc_ctx_create(0, None, C.byref(ctx)))
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = tmp_path_factory.mktemp("fake_hip") / "fake_hip.so"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), os.path.join(HERE, "fake_hip.c"),
                    "-I", os.path.join(rocm, "include")], check=True)
    return str(so)


def run(runtime, body):
    lib = os.path.join(ROOT, "paper_1910_11110_amd", "libvcheck.so")
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, runtime, lib], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_no_alloc_in_place_reads_a_copy(runtime):
    """init and final_status in one buffer: the check, whose tiles read the one and write the
    other in no order, is not handed the buffer as both; without events it stays as it is."""
    run(runtime, """
table = (C.c_uint8 * 64)(*range(64))
ev, status, viol, counts = (C.c_uint32 * 65536)(), (C.c_uint8 * 65536)(), (C.c_uint32 * 65536)(), (C.c_uint64 * 3)()
at = C.addressof(ev) + (-C.addressof(ev)) % 16
for init in (table, None):
    F.fake_reset()
    ok(L.vc_check_small_noalloc(ctx, at, 60000, 64, init, status, table, viol, counts))
    words = [a for name, a in launches() if "k_small_check" in name]
    assert len(words) == 1, launches()
    assert words[0].count(C.addressof(table)) == 1, [hex(w) for w in words[0]]
assert list(table) == list(range(64))  # (the copy is the library's own; kernels do not run here)
ok(L.vc_check_small_noalloc(ctx, at, 0, 64, table, status, table, viol, counts))
other = (C.c_uint8 * 64)()
ok(L.vc_check_small_noalloc(ctx, at, 0, 64, table, status, other, viol, counts))
assert list(table) == list(other) == list(range(64))
""")


@pytest.mark.parametrize("n,words,fuel,steps", [(2048, 240, 32, False), (2048, 240, 128, True), (2048, 64, 4, False),
                                                (2048, 64, 4096, True), (1 << 17, 240, 128, False),
                                                (1 << 17, 240, 512, True), (1 << 17, 24, 16, True),
                                                (300, 600, 4096, False), (300, 1, 0, False), (300, 0, 0, True)])
def test_programs_with_little_fuel_are_walked_in_place(runtime, n, words, fuel, steps):
    """Making the steps of all words is not worth it for programs that take few reductions."""
    run(runtime, f"""
import numpy as np
off = np.arange({n} + 1, dtype=np.uint64) * {words}
w = np.full(max({n} * {words}, 1), 4 << 24, np.uint32)
L.vc_run_programs.argtypes = [P, P, u64, P, u32, P, P, u64, C.POINTER(P)]
h = P()
ok(L.vc_run_programs(ctx, off.ctypes.data, {n}, w.ctypes.data, 1, None, None, {fuel}, C.byref(h)))
names = [name for name, _ in launches() if "k_run_" in name]
assert len(names) == 1 and ("k_run_steps" in names[0]) == {steps}, names
""")


@pytest.mark.parametrize("sizes,walks", [
    (((40000, 1000 * 1536), (20000, 24 * 1024)), 1),
    (((40000, 1000 * 1536), (20000, 24 * 1024 + 1)), 2),
    (((20000, 1000),), 1),
    (((65536, 1), (32768, 1), (16384, 1), (8192, 1)), 1),
    (((65536, 1), (300, 10 ** 6)), 2),
    (((65536, 1), (16384, 0), (300, 10 ** 6)), 2)])
def test_batch_classes_share_launches(runtime, sizes, walks):
    """A batch that leaves the device idle is walked by one launch for several classes of ids:
    while the device holds all their chunks (1,024 of more than 32,768 ids) at once."""
    run(runtime, f"""
import os
os.environ["VC_NO_AUTOTUNE"] = "1"
L.vc_batch_check.argtypes = [P, C.POINTER(P), u32]
traces = []
for ids, n in {sizes}:
    ev, t = (C.c_uint32 * max(n, 1))(), P()
    ok(L.vc_trace_load(ctx, ev, n, ids, None, 0, C.byref(t)))
    traces.append(t)
F.fake_reset()
ok(L.vc_batch_check(ctx, (P * len(traces))(*traces), len(traces)))
names = [n for n, _ in launches()]
for walk in ("k_dense_fold", "k_dense_apply"):
    assert len([n for n in names if walk in n]) == {walks}, names
""")


CHECKED = """
ev = (C.c_uint32 * 5000)()
t = P()
ok(L.vc_trace_load(ctx, ev, 5000, 100, None, 0, C.byref(t)))
ok(L.vc_check(t))
F.fake_reset()
"""


def test_sync_reports_a_collection_that_was_not_launched(runtime):
    """What vc_sync takes of a trace comes from the launch behind its work: without it, from no
    launch of that call.  The next synchronization collects the trace."""
    run(runtime, CHECKED + """
F.fake_fail_kernel(b"k_collect")
assert L.vc_sync(ctx) == -3, L.vc_last_error()
assert F.fake_syncs() >= 1
F.fake_fail_kernel(b"")
L.vc_sync(ctx)
assert [n for n, _ in launches() if "k_collect" in n]
ok(L.vc_check(t))
""")


def test_sync_waits_without_pinned_memory(runtime):
    run(runtime, CHECKED + """
F.fake_fail_pinned(1)
assert L.vc_sync(ctx) == -2, L.vc_last_error()
assert F.fake_syncs() >= 1
F.fake_fail_pinned(0)
ok(L.vc_check(t))
""")


@pytest.mark.parametrize("name,at", [("small", 3 << 21), ("compact", 1 << 22)])
def test_scratch_holds_every_shorter_trace(runtime, name, at):
    """A work space sized for n events serves every shorter trace, also where the layout changes."""
    run(runtime, f"""
size = getattr(L, "_ZN2vc{len(name) + 14}{name}_scratch_bytesEm")
size.argtypes, size.restype = [u64], C.c_size_t
sizes = [size(n) for n in list(range(0, 40_000, 997)) + list(range({at} - 50_000, {at} + 900_000, 4_093)) + [1 << 24, 1 << 30]]
assert sizes == sorted(sizes)
""")
