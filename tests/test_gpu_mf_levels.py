"""The grouped SGD kernel's second part by levels: every number of lanes per entry, ranks that are and are not multiples
of 4 and of 2, one and many chunks per block, records kept for the block and fetched with a chunk, levels with more
entries than places, cells revealed several times, workgroups of 1 to 16 wavefronts, both launch forms.  Against the
fp32 oracle within the bar that the small cases of this kernel have (1e-5: a few roundings of O(1) values per update)."""
import numpy as np
import pytest

from paper_2002_00655_amd import workloads as wl
from _util import oracle_epochs, gpu_epochs, compare_state, check_handoff_order, replay_schedule

pytestmark = pytest.mark.gpu

OPT_CACHE, OPT_WAVES, OPT_HEAVY_LEN = 2, 3, 6


def _workload(m, n, nnz, rank, seed, repeat=0):
    w = wl.make_mf("tiny", seed=seed, m=m, n=n, nnz=nnz, rank=rank, planted=4)
    if repeat:                                              # the same few cells again and again
        rng = np.random.default_rng(seed)
        extra = rng.integers(0, 40, repeat)
        w.rows = np.concatenate([w.rows, w.rows[extra]]); w.cols = np.concatenate([w.cols, w.cols[extra]])
        w.vals = np.concatenate([w.vals, rng.standard_normal(repeat).astype(np.float32)])
    return w


# m, n, entries, d: one block of many rows (several chunks; 700 x 40: records beside them, 4000 x 60: with each chunk), a
# dense block (levels of up to 300 entries), blocks with a handful of entries, a single row and a single column
SHAPES = [(700, 40, 3000, 1), (4000, 60, 30000, 1), (300, 300, 30000, 1), (60, 50, 400, 4), (1, 200, 90, 1), (200, 1, 90, 1)]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("rank,waves", [(1, 16), (3, 16), (16, 16), (17, 5), (30, 12), (50, 16), (64, 16), (65, 1), (100, 16), (128, 16), (127, 12)])
def test_levels_match_the_oracle(shape, rank, waves):
    from oracle.oracle import mf_block_ratings
    m, n, nnz, d = SHAPES[shape]
    for heavy_len, repeat in ((10 ** 6, 0), (48, 200)):     # all entries by levels; long runs in groups first
        print(f"case {SHAPES[shape]} rank={rank} waves={waves} heavy_len={heavy_len} repeat={repeat}", flush=True)
        w = _workload(m, n, nnz, rank, 7 + shape, repeat)
        rb, cb = wl.equal_bounds(m, d), wl.equal_bounds(n, d)
        blocked = mf_block_ratings(m, n, w.rows, w.cols, w.vals, rb, cb)
        sched = wl.cyclic_schedule(d)
        orc = oracle_epochs("f32", w, rb, cb, blocked, sched)
        options = [(OPT_WAVES, waves), (OPT_HEAVY_LEN, heavy_len)]
        srv = gpu_epochs(w, rb, cb, blocked, sched, options=options)
        compare_state(orc, srv, exact=False, atol=1e-5)
        if shape == 0 and rank in (17, 100):                # the variant without a schedule (a bound on the factors in LDS)
            compare_state(orc, gpu_epochs(w, rb, cb, blocked, sched, options=options + [(OPT_CACHE, 1 << 20)]), exact=False, atol=1e-5)


@pytest.mark.parametrize("rank", [16, 50, 100])
def test_levels_with_handoff(rank):
    """Column blocks handed from worker to worker between levels' blocks; the reported order replayed on the oracle."""
    from oracle.oracle import mf_block_ratings
    w = _workload(900, 200, 20000, rank, 3)
    d = 4
    rb, cb = wl.equal_bounds(w.m, d), wl.equal_bounds(w.n, d)
    blocked = mf_block_ratings(w.m, w.n, w.rows, w.cols, w.vals, rb, cb)
    print(f"case hand-over rank={rank}", flush=True)
    srv = gpu_epochs(w, rb, cb, blocked, wl.cyclic_schedule(d), epochs=0)
    order = srv.mf_sgd_epoch_handoff(w.lr, w.lam)
    srv.status()
    check_handoff_order(order)
    orc = oracle_epochs("f32", w, rb, cb, blocked, replay_schedule(order))
    compare_state(orc, srv, exact=False, atol=1e-5)


@pytest.mark.parametrize("rows", [63, 2047, 2048, 2049, 2200])
def test_levels_of_blocks_around_the_rows_that_lds_counts(rows):
    """Blocks whose row runs are counted in LDS, and in memory (from 2,049 rows), columns of more than 64 entries and cells
    revealed several times."""
    from oracle.oracle import mf_block_ratings
    m, n = rows, 40
    w = _workload(m, n, m * n // 3, 16, 5, 100)
    rb, cb = wl.equal_bounds(m, 1), wl.equal_bounds(n, 1)
    blocked = mf_block_ratings(m, n, w.rows, w.cols, w.vals, rb, cb)
    print(f"case {rows} rows, {np.unique(w.rows).size} with entries", flush=True)
    sched = wl.cyclic_schedule(1)
    orc = oracle_epochs("f32", w, rb, cb, blocked, sched)
    srv = gpu_epochs(w, rb, cb, blocked, sched, options=[(OPT_HEAVY_LEN, 10 ** 6)])
    compare_state(orc, srv, exact=False, atol=1e-5)
