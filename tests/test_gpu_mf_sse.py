"""mf_train_sse against the same sum in numpy float64: every width of a row piece (16, 8 and 4 bytes), every number of
pieces per lane, entry counts around a wavefront's 64 and around the eight shares of the entries."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [1, 2, 3, 4, 15, 16, 17, 32, 33, 50, 62, 64, 66, 100, 126, 127, 128, 129, 130, 145, 146, 161, 162, 178, 191, 193, 200, 210, 225,
                                  226, 242, 250, 254, 255, 256])
def test_train_sse_sums_in_double(rank):
    import torch
    from paper_2002_00655_amd import ps as P
    rng = np.random.default_rng(rank)
    m, n = 37, 23
    dev = torch.device("cuda")
    val = rng.standard_normal((m + n, rank)).astype(np.float32)
    for nnz in (1, 63, 64, 65, 511, 513, 5000):
        print(f"case rank={rank} nnz={nnz}", flush=True)
        cell = np.sort(rng.integers(0, m * n, size=nnz))                      # one block; cells may be revealed twice
        cols, rows = (cell // m).astype(np.int32), (cell % m).astype(np.int32)
        vals = rng.standard_normal(nnz).astype(np.float32)
        srv = P.ParameterServer(m + n, rank, 1)
        srv.push(torch.arange(m + n, device=dev), torch.from_numpy(val).to(dev))
        srv.mf_load_ratings(m, n, *(torch.from_numpy(x).to(dev) for x in (rows, cols, vals)), [0, m], [0, n], [0, nnz])
        got = srv.mf_train_sse()
        v = val.astype(np.float64)
        dot = (v[rows] * v[m + cols]).sum(1)
        want = float(((vals.astype(np.float64) - dot) ** 2).sum())
        # an inner product of `rank` terms is off by at most rank 2^-53 sum |w h|, its square and the sum by the same order
        size = np.abs(v[rows] * v[m + cols]).sum(1) + np.abs(vals)
        bound = float((2 * np.abs(vals - dot) * size * (rank + 2)).sum() + nnz * want) * 2.0 ** -53
        assert abs(got - want) <= 2 * bound, (got, want, bound)


@pytest.mark.parametrize("nnz", [2047, 2048, 2049, 4097, 131071, 131072, 131073, 524288, 524289, 700001])
def test_train_sse_at_numbers_of_workgroups(nnz):
    """Entry counts at which the launch gets more workgroups, and the most it gets; the bound as above."""
    import torch
    from paper_2002_00655_amd import ps as P
    rng = np.random.default_rng(nnz)
    m, n, rank = 900, 800, 4
    dev = torch.device("cuda")
    val = rng.standard_normal((m + n, rank)).astype(np.float32)
    cell = np.sort(rng.integers(0, m * n, size=nnz))
    cols, rows = (cell // m).astype(np.int32), (cell % m).astype(np.int32)
    vals = rng.standard_normal(nnz).astype(np.float32)
    srv = P.ParameterServer(m + n, rank, 1)
    srv.push(torch.arange(m + n, device=dev), torch.from_numpy(val).to(dev))
    srv.mf_load_ratings(m, n, *(torch.from_numpy(x).to(dev) for x in (rows, cols, vals)), [0, m], [0, n], [0, nnz])
    print(f"case nnz={nnz}", flush=True)
    got = srv.mf_train_sse()
    v = val.astype(np.float64)
    e = vals - (v[rows] * v[m + cols]).sum(1)
    want = float((e ** 2).sum())
    size = np.abs(v[rows] * v[m + cols]).sum(1) + np.abs(vals)
    bound = float((2 * np.abs(e) * size * (rank + 2)).sum() + nnz * want) * 2.0 ** -53
    assert abs(got - want) <= 2 * bound, (got, want, bound)
