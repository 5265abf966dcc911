"""The order that a push brings its pairs into, at the sizes where the sort's way changes (tiles of 1,024, 2,048 and 8,192 pairs, and
1,024 and 4,096 with four launches per digit), by sums that depend on it: bit for bit what the interface describes - the pairs ordered by
key, equal keys by position, in ranges of 64, a key's terms inside a range one after the other, its ranges' sums in order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _push(val, keys, d):
    order = np.argsort(keys, kind="stable")
    k = keys[order]
    n = k.size
    at = np.flatnonzero(np.concatenate([[True], (k[1:] != k[:-1]) | (np.arange(1, n) % 64 == 0)]))      # where a key's share of a range starts
    size = np.diff(np.append(at, n))
    key = k[at]
    first = np.concatenate([[True], key[1:] != key[:-1]])
    sums = np.where(first[:, None], val[key], np.float32(0))
    for j in range(64):
        s = np.flatnonzero(size > j)
        sums[s] += d[order[at[s] + j]]
    head = np.flatnonzero(first)
    shares = np.diff(np.append(head, at.size))
    total = sums[head]
    by_shares = np.argsort(-shares, kind="stable")                          # those with more than j shares come first
    more = shares[by_shares]
    for j in range(1, int(shares.max())):
        s = by_shares[:np.searchsorted(-more, -j)]
        total[s] += sums[head[s] + j]
    val[key[head]] = total


@pytest.mark.parametrize("K,kind", [(1, "one"), (700, "uniform"), (5000, "ordered"), (5000, "mixed"), ((1 << 20) + 7, "uniform"), ((1 << 20) + 7, "one")])
@pytest.mark.parametrize("n", [2049, 32768, 32769, 131072, 131073, 262144, 262145, 270337, 2097152, 2097153])
def test_pairs_keep_their_order(K, kind, n):
    import torch
    from paper_2002_00655_amd import ps as P
    L = 2
    rng = np.random.default_rng(n + K)
    print(f"case K={K} kind={kind} n={n}", flush=True)
    keys = rng.integers(0, K, n)
    if kind == "one":
        keys[:] = K - 1
    elif kind == "ordered":
        keys.sort()
    elif kind == "mixed":                                                    # a third of the keys is one
        keys[rng.random(n) < 0.3] = 4321
    d = (rng.standard_normal((n, L)) * 10.0 ** rng.integers(-3, 4, size=(n, 1))).astype(np.float32)
    val = np.zeros((K, L), np.float32)
    srv = P.ParameterServer(K, L, 3)
    kt, dt = torch.from_numpy(keys).cuda(), torch.from_numpy(d).cuda()
    for _ in range(2):                                                       # (the second onto values, in scratch that has been used)
        srv.push(kt, dt, 1)
        _push(val, keys, d)
    assert np.array_equal(srv.pull(torch.arange(K, device="cuda")).cpu().numpy().view(np.uint32), val.view(np.uint32))
    srv.status()
