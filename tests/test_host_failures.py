"""CPU: the library's host code with a stand-in for the HIP runtime (tests/_hip_stub.c) whose calls fail on demand: the marks
and flags of knowledge-graph steps that update rows in place, the two sets of sorted pairs of an epoch, and what
is set up per device."""
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
lib.ps_last_error.restype = C.c_char_p
def epoch(n, batch, h=h):
    part = (C.c_int64 * 3)(0, n // 2, n)
    return lib.kge_sgd_epoch(h, C.c_int64(E), C.c_int32(dim), C.c_int64(n), x, x, x, C.c_int32(ns), x, C.c_int32(no), x, part, C.c_int32(2),
                             C.c_int64(batch), C.c_int32(1), C.c_float(.1), C.c_float(1e-10), None, None)
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
    # an epoch's second set of sorted pairs: no memory, ever - asked for once, without an error's text; the scratch that is there is kept, and
    # an epoch of a size seen before neither waits nor allocates
    "no memory for two sets of pairs": """
asked = (C.c_size_t * 4096).in_dll(stub, "stub_alloc_bytes")
def server():
    p = C.c_void_p()
    assert lib.ps_create(C.c_int64(K), C.c_int32(4 * dim), C.c_int32(2), C.byref(p)) == 0
    return p
sizes = []
for batch in (500, 700):                             # what two sets take: a new server's epoch allocates its own scratch, then these
    other = server()
    at = get("allocs")[0]
    assert epoch(4 * batch, batch, other) == 0
    new = [s for s in asked[at:get("allocs")[0]] if s not in (seen, flags(batch))]
    assert len(new) == 2, new
    sizes.append(new[1])
var("stub_fail_alloc_bytes", C.c_size_t).value = sizes[0]
for i in range(3):
    before = get("device_syncs", "stream_syncs", "frees", "allocs")
    assert epoch(2000, 500) == 0 and lib.ps_last_error(h) == b"", (i, lib.ps_last_error(h))
    assert get("allocs_of_size") == [1], (i, get("allocs_of_size"))
    if i > 0: assert get("device_syncs", "stream_syncs", "frees", "allocs") == before, (i, before)
var("stub_fail_alloc_bytes", C.c_size_t).value = sizes[1]
at = get("allocs")[0]
assert epoch(2800, 700) == 0 and sizes[1] not in asked[at:get("allocs")[0]]      # nor is more than what was refused
# scratch that one set fits into stays where it is
other = server()
assert lib.ps_push(other, C.c_int32(0), x, C.c_int64(500 * (3 + ns + no)), x, None) == 0
var("stub_fail_alloc_bytes", C.c_size_t).value = sizes[0]
var("stub_allocs_of_size", C.c_int).value = 0
before = get("device_syncs", "frees")
assert epoch(2000, 500, other) == 0 and get("device_syncs", "frees") == before and get("allocs_of_size") == [1]
""",
    # kernels with more than 64 KB of dynamic LDS: allowed on the device of the handle, once per handle
    "LDS on a second device": """
handles = []
for device in (0, 1):
    var("stub_device", C.c_int).value = device
    p = C.c_void_p()
    assert lib.ps_create(C.c_int64(K), C.c_int32(256), C.c_int32(2), C.byref(p)) == 0
    handles.append(p)
    for i in range(2):
        if i: before = get("lds_calls")
        assert lib.ps_push(p, C.c_int32(0), x, C.c_int64(300_000), x, None) == 0
        assert lib.kge_sgd_step(p, C.c_int32(-1), C.c_int64(E), C.c_int32(64), C.c_int64(8), x, x, x, C.c_int32(2), x, C.c_int32(3), x,
                                C.c_float(.1), C.c_float(1e-10), None, None) == 0
    assert get("lds_calls") == before, device
    assert get("lds_refused") == [0], (device, get("lds_refused"))
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
