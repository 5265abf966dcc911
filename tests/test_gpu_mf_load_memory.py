"""What mf_load_ratings allocates, seen through a hook on hipMalloc in a process of its own: the schedule by levels is made
only for data that the SGD kernels process by levels, and data loads without it where its memory is refused."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import ctypes as C, sys
hook = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import numpy as np, torch
from paper_2002_00655_amd import ps as P, workloads as wl
from oracle.oracle import mf_block_ratings
armed, count, fail_at = (C.c_int.in_dll(hook, "hook_" + n) for n in ("armed", "count", "fail_at"))
SCHEDULE = 7                    # the tables of a schedule and its scratch

def data(m, n, nnz, d, rank=16):
    w = wl.make_mf("tiny", seed=3, m=m, n=n, nnz=nnz, rank=rank, planted=4)
    rb, cb = wl.equal_bounds(m, d), wl.equal_bounds(n, d)
    br, bc, bv, bp = mf_block_ratings(m, n, w.rows, w.cols, w.vals, rb, cb)
    return w, rb, cb, [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (br, bc, bv)], bp

def load(srv, x, fail=-1):
    # -> allocations of the load, the error
    w, rb, cb, t, bp = x
    count.value, fail_at.value, armed.value = 0, fail, 1
    try:
        srv.mf_load_ratings(w.m, w.n, *t, rb, cb, bp)
        return count.value, 0
    except P.PSError as e:
        return count.value, e.code
    finally:
        armed.value, fail_at.value = 0, -1

def server(x):
    w = x[0]
    srv = P.ParameterServer(w.m + w.n, w.rank, len(x[1]) - 1)
    srv.push(torch.arange(w.m + w.n, device="cuda"), torch.from_numpy(np.concatenate([w.W0, w.H0])).cuda())
    return srv

def epoch(srv, x):
    w = x[0]
    srv.mf_sgd_epoch(wl.cyclic_schedule(len(x[1]) - 1), w.lr, w.lam)
    out = srv.pull(torch.arange(w.m + w.n, device="cuda")).cpu().numpy()
    srv.status()
    return out

levels = data(400, 300, 20_000, 4)                  # rows of a dozen entries per block
exec(sys.argv[3])
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = tmp_path_factory.mktemp("hook") / "malloc_hook.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "_malloc_hook.c"), "-o", str(so), "-ldl"])

    def go(body):
        r = subprocess.run([sys.executable, "-u", "-c", PROGRAM, str(so), ROOT, body], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stdout[-500:] + r.stderr[-1500:]
        print(r.stdout, flush=True)
    return go


def test_a_schedule_is_made_only_where_it_is_used(run):
    run(r"""
single = data(6000, 300, 8_000, 4)                  # rows of mostly one entry per block
long_runs = data(6000, 8, 40_000, 2)                # columns of thousands of entries per block
a = load(server(levels), levels)
for x in (single, long_runs):
    b = load(server(x), x)
    print(a, b, flush=True)
    assert a[1] == b[1] == 0 and b[0] <= a[0] - SCHEDULE
""")


def test_a_load_survives_a_refused_schedule(run):
    """Every allocation of a load refused in turn: the load reports it and the handle takes the next load, or - for the
    schedule's - goes on without, and an epoch gives the same factors up to the forms' rounding (1e-5, the small cases' bar)."""
    run(r"""
srv = server(levels)
total, rc = load(srv, levels)
assert rc == 0
want = epoch(srv, levels)
went_on = 0
for i in range(total):
    srv = server(levels)
    n, rc = load(srv, levels, i)
    assert n >= i + 1 and rc in (0, -5), (i, n, rc)
    if rc:
        assert load(srv, levels) == (total, 0)
    else:
        went_on += 1
    assert np.abs(epoch(srv, levels) - want).max() <= 1e-5, i
print("allocations", total, "without", went_on, flush=True)
assert went_on == SCHEDULE
""")
