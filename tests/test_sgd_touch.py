"""CPU: which words of the store are fetched ahead of a block's second part (csrc/sgd_touch.h, compiled for the host).  Where
column factors pass from workgroup to workgroup inside a launch (an epoch with hand-over) they are read and written past
the die's cache, and an ordinary load must not bring their lines into it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODEL = r"""
#define __device__
#define __forceinline__ inline
#include <cstdio>
#include <cstdlib>
#include "sgd_touch.h"
int main(int argc, char **argv) {
    const bool loop = atoi(argv[1]) != 0;
    const int L = atoi(argv[2]), by = atoi(argv[3]);
    const int32_t rows[] = {0, 3, 4}, cols[] = {1, 5};
    auto load = [](int64_t i) { printf("%lld\n", (long long)i); };
    for (int first = 0; first < by; ++first) {
        if (loop) touch_factors<true>(first, by, 3, 2, rows, cols, 10, L, load);
        else touch_factors<false>(first, by, 3, 2, rows, cols, 10, L, load);
    }
}
"""


@pytest.fixture(scope="module")
def touched(tmp_path_factory):
    d = tmp_path_factory.mktemp("touch")
    (d / "model.cpp").write_text(MODEL)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2002_00655_amd", "csrc"), str(d / "model.cpp"), "-o", str(d / "model")])
    return lambda *args: [int(x) for x in subprocess.check_output([str(d / "model"), *map(str, args)], timeout=20).split()]


@pytest.mark.parametrize("L", [1, 16, 32, 33, 100, 128])
@pytest.mark.parametrize("by", [1, 2, 64])
@pytest.mark.parametrize("loop", [0, 1])
def test_columns_that_are_handed_over_are_left_alone(touched, loop, L, by):
    keys = [0, 3, 4] if loop else [0, 3, 4, 11, 15]
    assert sorted(touched(loop, L, by)) == [k * L + i for k in keys for i in range(0, L, 32)]
