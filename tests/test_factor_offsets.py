"""CPU: the byte offsets of the grouped SGD kernel's accesses to a block's factors (csrc/factor_offsets.h, compiled for the host), in
the largest block that is taken and in blocks a little smaller: what exists is where it lies, and what does not - an entry past a group's
end, a component past the rank - is past the end of the buffer, where an access reads zero and writes nothing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MODEL = r"""
#define __device__
#define __forceinline__ inline
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "factor_offsets.h"
int main(int argc, char **argv) {
    const int64_t L = atoll(argv[1]), limit = (1ll << 31) - 4096;     // what a block's factors may span
    const int64_t most = (limit - 1) / (4 * L);
    if (!dpaps_span_ok(most, L) || dpaps_span_ok(most + 1, L)) { puts("another limit"); return 1; }
    // rows in a block; the rows looked at: the first, the last, and what lies around the offset that stands for "nowhere"
    for (int64_t rows : {most, most - 1, (int64_t)DPAPS_PAST_END / (4 * L), (int64_t)0x7F000000 / (4 * L) + 2, (int64_t)1000}) {
        if (rows > most) continue;
        const int64_t span = rows * L * 4;
        for (int64_t row : {(int64_t)0, (int64_t)1, rows / 2, (int64_t)0x7F000000 / (4 * L), rows - 2, rows - 1}) {
            if (row >= rows) continue;
            for (int k = 0; k < 128; ++k)                              // a wavefront's lanes, one or two components each
                for (int there = 0; there < 2; ++there) {
                    const uint64_t at = (uint32_t)past_end_sum(row_start(there != 0, (int)row, (int)L), component_at(k, (int)L));
                    const bool exists = there && k < L;
                    if (exists ? at != (uint64_t)((row * L + k) * 4) : at < (uint64_t)span || at + 8 > 1ull << 32) {
                        printf("rows %lld row %lld there %d component %d: %llu of %lld\n", (long long)rows, (long long)row, there, k, (unsigned long long)at, (long long)span);
                        return 1;
                    }
                }
        }
    }
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    (d / "model.cpp").write_text(MODEL)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2002_00655_amd", "csrc"), str(d / "model.cpp"), "-o", str(d / "model")])
    return str(d / "model")


@pytest.mark.parametrize("L", [1, 2, 3, 16, 49, 50, 64, 65, 99, 100, 127, 128])
def test_what_does_not_exist_is_past_the_end(model, L):
    r = subprocess.run([model, str(L)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
