"""A push of 65 to 2,048 keys, which is one launch, or a sort and the sums where rows are long: bit for bit the sums that the
interface describes - the pairs ordered by key, in ranges of 64, a key's terms inside a range one after the other, its ranges'
sums in order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _push(val, keys, d):
    order = np.argsort(keys, kind="stable")
    k = keys[order]
    at = 0
    while at < k.size:
        end = at + int((k[at:] == k[at]).sum())
        total = val[k[at]].copy()
        lo = at
        while lo < end:
            hi = min(end, (lo // 64 + 1) * 64)
            s = total if lo == at else np.zeros_like(total)
            for p in order[lo:hi]:
                s = s + d[p]
            total = s if lo == at else total + s
            lo = hi
        val[k[at]] = total
        at = end


# distinct keys; one key only; two keys that end inside a range; eight keys one after the other; frequent keys among others
@pytest.mark.parametrize("kind", ["distinct", "one", "two", "eight", "mixed"])
@pytest.mark.parametrize("L", [1, 6, 64, 65, 100, 128, 130, 260, 400])
def test_push_of_few_keys_is_what_the_interface_says(kind, L):
    _check(kind, L, (65, 127, 128, 129, 333, 1023, 1025, 2047, 2048))


# long rows: around the numbers of workgroups up to which it is one launch (768 up to 1,024 keys, then 448, or 512 of one value per piece)
@pytest.mark.parametrize("kind", ["distinct", "mixed"])
@pytest.mark.parametrize("L,sizes", [(1023, (768, 769, 1024, 1025, 2048)), (1022, (1024, 1025, 1500)), (1000, (1024, 1025, 1792, 1793, 2048)),
                                     (255, (2047, 2048)), (257, (1632, 1633, 2048))])
def test_push_of_few_long_rows(kind, L, sizes):
    _check(kind, L, sizes)


def _check(kind, L, sizes):
    import torch
    from oracle.oracle import Oracle
    from paper_2002_00655_amd import ps as P
    K, W = 5000, 256
    rng = np.random.default_rng(L)
    srv, orc = P.ParameterServer(K, L, W), Oracle("f32", K, L, W)
    val = np.zeros((K, L), np.float32)
    for n in sizes:
        print(f"case kind={kind} L={L} n={n}", flush=True)
        if kind == "distinct":
            keys = rng.permutation(K)[:n]
        elif kind == "one":
            keys = np.full(n, int(rng.integers(0, K)))
        elif kind == "two":
            keys = np.where(rng.random(n) < 0.4, 17, 4000)
        elif kind == "eight":
            keys = np.arange(n) * 8 // n
        else:
            keys = rng.integers(0, K, n)
            for _ in range(9):
                keys[rng.random(n) < 0.1] = rng.integers(0, K)
        d = (rng.standard_normal((n, L)) * 10.0 ** rng.integers(-3, 4, size=(n, 1))).astype(np.float32)
        worker = int(rng.integers(-1, W))
        srv.push(torch.from_numpy(keys).cuda(), torch.from_numpy(d).cuda(), worker)
        orc.push(keys, d, worker)                            # (for the statistics)
        _push(val, keys, d)
        assert np.array_equal(srv.pull(torch.arange(K, device="cuda")).cpu().numpy().view(np.uint32), val.view(np.uint32)), n
    assert srv.stats() == orc.stats()
