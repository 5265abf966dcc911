"""CPU: the library's host code with a stand-in for the HIP runtime (tests/_hip_stub.c) whose calls fail on demand: the marks
and flags of knowledge-graph steps that update rows in place."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
def var(name, t): return t.in_dll(stub, name)
K, E, dim, ns, no = 100_000, 99_000, 16, 2, 2
h = C.c_void_p()
assert lib.ps_create(C.c_int64(K), C.c_int32(4 * dim), C.c_int32(2), C.byref(h)) == 0
x = C.c_void_p(C.addressof(C.create_string_buffer(1 << 16)))
def step(batch):
    return lib.kge_sgd_step(h, C.c_int32(-1), C.c_int64(E), C.c_int32(dim), C.c_int64(batch), x, x, x, C.c_int32(ns), x, C.c_int32(no), x,
                            C.c_float(.1), C.c_float(1e-10), None, None)
C.memmove(C.addressof(var("stub_watch", C.c_char * 64)), b"k_kge_keys\0", 11)
var("stub_watch_arg", C.c_int).value = 3            # where the marks are
seen = 8 * K
def flags(batch): return 8 * batch * (3 + ns + no)
def get(*names): return [var("stub_" + n, C.c_int).value for n in names]
exec(sys.argv[3])
"""

STEPS = {
    # the marks: no memory, ever - asked for once, and every step does without them
    "no memory for the marks": """
var("stub_fail_alloc_bytes", C.c_size_t).value = seen
assert [step(400) for _ in range(3)] == [0, 0, 0]
assert get("watched", "watched_null") == [3, 3]
assert get("allocs_of_size") == [1], get("allocs_of_size")
""",
    # the marks cannot be cleared: never used uncleared, also not by the next step
    "marks not cleared": """
var("stub_fail_zero_bytes", C.c_size_t).value = seen
var("stub_fail_zero_times", C.c_int).value = 1
assert [step(400) for _ in range(3)] == [0, 0, 0]
assert get("watched_uncleared") == [0], get("watched_uncleared")
assert get("watched", "watched_null") == [3, 1]
""",
    "no memory for the flags": """
var("stub_fail_alloc_bytes", C.c_size_t).value = flags(600)
assert [step(n) for n in (400, 600, 600, 700, 400, 500)] == [0] * 6
assert get("allocs_of_size") == [1], get("allocs_of_size")
var("stub_watch_arg", C.c_int).value = 4            # where the flags are
var("stub_watched_null", C.c_int).value = 0
assert step(500) == 0 and get("watched_null", "watched_uncleared") == [0, 0]
""",
    "flags not cleared": """
var("stub_watch_arg", C.c_int).value = 4
var("stub_fail_zero_bytes", C.c_size_t).value = flags(400)
var("stub_fail_zero_times", C.c_int).value = 1
assert [step(400) for _ in range(3)] == [0, 0, 0]
assert get("watched_uncleared") == [0]
""",
    # what the header says: a step's own memory waits for the stream, not for the device
    "waits": """
before = get("device_syncs")
assert step(400) == 0
assert get("device_syncs") == before, get("device_syncs")
""",
}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = tmp_path_factory.mktemp("stub") / "hip_stub.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "_hip_stub.c"), "-o", str(so)])
    return str(so)


@pytest.mark.parametrize("what", sorted(STEPS))
def test_marks_and_flags_of_in_place_steps(stub, what):
    lib = os.path.join(ROOT, "paper_2002_00655_amd", "libdpaps.so")
    r = subprocess.run([sys.executable, "-c", PROGRAM, stub, lib, STEPS[what]], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-1500:]
