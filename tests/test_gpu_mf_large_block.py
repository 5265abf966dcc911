"""A row block whose factors span nearly 2 GiB, the most that the grouped SGD kernel takes: its accesses of rows past a group's end and of
components past the rank must not reach rows of the block (rank 100: lanes past the rank; 127: the same, component by component; 128:
only rows past a group's end; 15 and 16: four rows in one access), against the entry-by-entry kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,m,waves", [(100, 5_340_000, 16), (100, 5_368_698, 12), (127, 4_210_000, 16), (128, 4_194_295, 16),
                                          (15, 35_600_000, 16), (16, 33_554_367, 16)])
def test_a_row_block_of_nearly_two_gib(rank, m, waves):
    import torch
    from paper_2002_00655_amd import ps as P
    assert 0x7F000000 + 4096 < m * rank * 4 < 2 ** 31 - 4096
    rng = np.random.default_rng(rank)
    # the rows with entries: the first, the last, and those around 0x7F000000 bytes
    mid = 0x7F000000 // (4 * rank)
    ids = np.concatenate([np.arange(20), np.arange(mid - 10, mid + 10), np.arange(m - 20, m)])
    runs = [46, 31, 16, 15, 14, 5, 1]                       # entries of a column: groups of 15, fewer, and one more
    n = len(runs)
    cols = np.repeat(np.arange(n, dtype=np.int32), runs)
    rows = np.concatenate([np.sort(rng.choice(ids, r, replace=False)) for r in runs]).astype(np.int32)
    vals = rng.standard_normal(rows.size).astype(np.float32)
    keys = torch.from_numpy(np.concatenate([ids, m + np.arange(n)])).cuda()
    init = torch.from_numpy((rng.standard_normal((len(keys), rank)) * rank ** -0.5).astype(np.float32)).cuda()
    srv = []
    for grouped in (0, 1):
        print(f"case rank={rank} m={m} waves={waves} grouped={grouped}", flush=True)
        s = P.ParameterServer(m + n, rank, 1)
        s.set_option(P.OPT_MF_GROUPED, grouped)
        s.set_option(P.OPT_MF_HEAVY_LEN, 4)
        s.set_option(P.OPT_MF_WAVES, waves)
        s.push(keys, init)
        s.mf_load_ratings(m, n, *(torch.from_numpy(x).cuda() for x in (rows, cols, vals)), [0, m], [0, n], [0, rows.size])
        for _ in range(2):
            s.mf_sgd_epoch([np.array([[0, 0, 0]], np.int32)], 0.05, 0.05)
        s.status()
        srv.append(s)
    assert srv[0].stats() == srv[1].stats()
    written = torch.zeros(m + n, dtype=torch.bool, device="cuda")
    written[keys] = True
    for a in range(0, m + n, 1 << 20):
        k = torch.arange(a, min(a + (1 << 20), m + n), device="cuda")
        want, got = srv[0].pull(k), srv[1].pull(k)
        # (1e-5: as in the other comparisons of the two kernels)
        assert float((want - got).abs().max()) <= 1e-5, a
        assert not got[~written[k]].any(), a
