"""CPU: the workgroup-wide decisions of csrc/together.h, compiled for the host: a thread per device thread, a barrier that
counts only the threads still running, and an error flag that one thread sees set and another does not, as when another
workgroup of the launch sets it in between.  (The form in which every thread first looks at the flag by itself and leaves is
run as well: it lets a bad key pass.)"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODEL = r"""
#include <atomic>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>
#define __device__
#define __forceinline__ inline
#define volatile
struct Dim { unsigned x; };
static thread_local Dim threadIdx;
static Dim blockDim;
// the barrier of a workgroup: threads that have left are not waited for
static std::mutex m; static std::condition_variable cv;
static int running, arrived, phase, acc, result;
static void release() { if (arrived > 0 && arrived == running) { result = acc; acc = 0; arrived = 0; ++phase; cv.notify_all(); } }
static int __syncthreads_or(int p) {
    std::unique_lock<std::mutex> l(m);
    acc |= p; ++arrived;
    const int mine = phase;
    release();
    cv.wait(l, [&] { return phase != mine; });
    return result;
}
static void leave() { std::unique_lock<std::mutex> l(m); --running; release(); }
static std::atomic<int> sets{0};
static int atomicExch(int *p, int v) { sets = v; return 0; }
#include "together.h"

int main(int argc, char **argv) {
    // argv: old form (1), not (0), or one thread's look for all (2); number of keys; the bad one's place (-1: none); the flag as the threads see it, bit by bit
    const int form = atoi(argv[1]), n = atoi(argv[2]), bad = atoi(argv[3]); const char *sees = argv[4];
    const int T = 8;
    blockDim.x = T; running = T;
    std::vector<int64_t> keys(n, 5);
    if (bad >= 0) keys[bad] = 1000;
    std::vector<int> went_on(T, 0);
    std::vector<std::thread> ts;
    for (int t = 0; t < T; ++t) ts.emplace_back([&, t] {
        threadIdx.x = t;
        int32_t flag = sees[t] == '1' ? -10 : 0, clear = 0;
        if (form == 2) { static int word; look_for_all(&flag, &word); __syncthreads_or(0); went_on[t] = word == 0; }
        else if (form == 1) { if (!flag) went_on[t] = !few_keys_off(keys.data(), n, 10, &clear); }
        else went_on[t] = !few_keys_off(keys.data(), n, 10, &flag);
        leave();
    });
    for (auto &t : ts) t.join();
    int on = 0;
    for (int x : went_on) on += x;
    printf("%d %d\n", on, (int)sets);
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("together")
    src = d / "model.cpp"
    src.write_text(MODEL)
    exe = d / "model"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_2002_00655_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])

    def run(old, n, bad, sees):
        on, err = subprocess.check_output([str(exe), str(int(old)), str(n), str(bad), sees], timeout=20).split()
        return int(on), int(err)
    return run


@pytest.mark.parametrize("n", [1, 7, 8, 9, 20])
def test_a_call_of_few_keys_goes_on_with_all_threads_or_none(model, n):
    assert model(False, n, -1, "00000000") == (8, 0)
    for bad in range(n):
        # whoever sees the flag of another workgroup already: nobody goes on
        for sees in ("00000000", "01100000", "11111110", "00000001", "10000000", "11111111"):
            on, err = model(False, n, bad, sees)
            assert on == 0
            assert err == (-2 if sees[0] == "0" else 0)        # the error is set where it did not stand
    # an earlier error: every thread sees it, nothing is done and it is kept
    assert model(False, n, -1, "11111111") == (0, 0)


@pytest.mark.parametrize("sees", ["00000000", "01100000", "10000000", "11111110", "11111111"])
def test_one_look_at_the_flag_holds_for_all(model, sees):
    assert model(2, 0, -1, sees)[0] == (8 if sees[0] == "0" else 0)


def test_leaving_one_by_one_would_let_a_bad_key_pass(model):
    assert model(True, 8, 2, "00100000")[0] == 7
