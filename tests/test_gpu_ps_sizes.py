"""The parameter-server calls at the sizes where their launches change (64 keys: a push in one launch; 2,048: few keys,
checked by the call's own kernel, sorted in one workgroup; 131,072: the sort's large tiles; 128 MB: a pull's result
written past the caches), at row lengths and alignments read in 16, 8 and 4 bytes, against the fp32 oracle: values bit for bit where every key's terms lie in one range or are integers,
owner map and every counter exact; a key out of range changes nothing.  Knowledge-graph steps that update rows of keys
named once in place: against the same step with the sums of the push only."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 127, 128, 129, 255, 257, 2047, 2048, 2049, 4096, 4097, 131072, 131073]


@pytest.mark.parametrize("K,L,W", [(5000, 4, 3), (300_000, 6, 256), (1 << 20, 3, 7), ((1 << 21) + 5, 1, 300), (700, 130, 1), (40_000, 100, 5),
                                    (9000, 260, 4)])
def test_calls_at_every_size(K, L, W):
    import torch
    from oracle.oracle import Oracle
    from paper_2002_00655_amd import ps as P
    rng = np.random.default_rng(K + L)
    orc, srv = Oracle("f32", K, L, W), P.ParameterServer(K, L, W)
    dev = torch.device("cuda")
    for i, n in enumerate(SIZES):
        print(f"case K={K} L={L} W={W} n={n}", flush=True)
        worker = int(rng.integers(0, W))
        keys = rng.integers(0, K, size=n)
        keys[rng.random(n) < 0.3] = rng.integers(0, K)                      # one key often: over many ranges
        d = rng.integers(-8, 9, size=(n, L)).astype(np.float32)             # sums of small integers are exact in any order
        kt, dt = torch.from_numpy(keys).to(dev), torch.empty(n * L + 2, device=dev)[i % 3:][:n * L].reshape(n, L)
        dt.copy_(torch.from_numpy(d))                                       # from 4, 8 and 16 bytes on
        srv.localize(kt, worker); orc.localize(keys, worker)
        other = int(rng.integers(-1, W))
        srv.push(kt, dt, other); orc.push(keys, d, other)
        assert np.array_equal(srv.pull(kt, worker).cpu().numpy(), orc.pull(keys, worker)), n
        out = torch.empty(n * L + 1, device=dev)[1:].reshape(n, L)          # a result that starts on 4 bytes only
        assert np.array_equal(srv.pull(kt, other, out=out).cpu().numpy(), orc.pull(keys, other)), n
        assert np.array_equal(srv.owner(kt).cpu().numpy(), orc.owner()[keys]), n
        if n <= P_NOALLOC and -(-n // 64) * L <= 1 << 20:
            srv.push_noalloc(kt, dt, other); orc.push(keys, d, other)
        assert srv.stats() == orc.stats(), n
    assert np.array_equal(srv.pull(torch.arange(K, device=dev)).cpu().numpy(), orc.pull(np.arange(K)))
    assert np.array_equal(srv.owner().cpu().numpy(), orc.owner())


P_NOALLOC = 262144


def test_push_of_up_to_64_keys_adds_in_argument_order():
    import torch
    from oracle.oracle import Oracle
    from paper_2002_00655_amd import ps as P
    rng = np.random.default_rng(9)
    K, L = 50, 100
    orc, srv = Oracle("f32", K, L, 2), P.ParameterServer(K, L, 2)
    for n in (1, 13, 16, 17, 63, 64):
        keys = rng.integers(0, 7, size=n)
        d = (rng.standard_normal((n, L)) * 10.0 ** rng.integers(-3, 4, size=(n, 1))).astype(np.float32)
        orc.push(keys, d, 0); srv.push(torch.from_numpy(keys).cuda(), torch.from_numpy(d).cuda(), 0)
    assert np.array_equal(srv.pull(torch.arange(K, device="cuda")).cpu().numpy().view(np.uint32), orc.pull(np.arange(K)).view(np.uint32))
    assert srv.stats() == orc.stats()


@pytest.mark.parametrize("n", [1, 64, 65, 2048, 2049, 140_000, 270_337, 2_100_000])
@pytest.mark.parametrize("bad", [-1, 1000, 1 << 40])
def test_a_bad_key_changes_nothing(n, bad):
    import torch
    from paper_2002_00655_amd import ps as P
    K, L = 1000, 8
    srv = P.ParameterServer(K, L, 4)
    rng = np.random.default_rng(n)
    allk = torch.arange(K, device="cuda")
    srv.push(allk, torch.from_numpy(rng.standard_normal((K, L)).astype(np.float32)).cuda(), 1)
    before, owner, stats = srv.pull(allk).cpu().numpy(), srv.owner().cpu().numpy(), srv.stats()
    keys = rng.integers(0, K, size=n)
    keys[int(rng.integers(0, n)) if n < 270_000 else n - 1] = bad            # (of the largest sorts' tiles the last, a partial one)
    kt = torch.from_numpy(keys).cuda()
    out = torch.full((n, L), 7.0, device="cuda")
    own = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    calls = [lambda: srv.pull(kt, 2, out=out), lambda: srv.push(kt, torch.ones((n, L), device="cuda"), 2), lambda: srv.localize(kt, 2), lambda: srv.owner(kt)]
    for call in calls:
        print(f"case n={n} bad={bad}", flush=True)
        call()
        with pytest.raises(P.PSError) as e:
            srv.status()
        assert e.value.code == P.PS_EKEY
    assert (out == 7.0).all() and (own == 7).all()
    assert np.array_equal(srv.pull(allk).cpu().numpy(), before) and np.array_equal(srv.owner().cpu().numpy(), owner) and srv.stats() == stats


@pytest.mark.parametrize("dim,ns,no,batch,stray", [(8, 4, 4, 300, False), (100, 5, 5, 600, False), (100, 3, 0, 900, True), (70, 0, 7, 400, True), (200, 2, 2, 700, True)])
def test_rows_named_once_are_updated_in_place(dim, ns, no, batch, stray):
    """Two steps and an epoch, with the push's sums only (its sequential order) and as they are: the same bits for every
    key whose terms lie in one range of the push, i.e. here all that are not frequent; the rest within a few roundings."""
    import torch
    from paper_2002_00655_amd import ps as P
    E, R = 30_000, 40
    rng = np.random.default_rng(dim + batch)
    K, L = E + R, 4 * dim
    subj, obj = rng.integers(0, 2000, size=batch), rng.integers(0, E, size=batch)
    rel = rng.integers(0, R, size=batch)
    negs, nego = rng.integers(0, E, size=(batch, ns)), rng.integers(0, E, size=(batch, no))
    neg = negs if ns else nego
    neg[0, 0], neg[1, 0] = subj[2], neg[3, 0]                               # a subject elsewhere; the same negative twice
    neg[5, 0] = subj[5]                                                     # the data point's own subject
    if stray:
        neg[7, 0] = E + int(rel[8])                                         # a number that is a relation's key
    init = np.concatenate([rng.standard_normal((K, 2 * dim)) * 0.1, np.full((K, 2 * dim), 0.01)], 1).astype(np.float32)
    t = [torch.from_numpy(np.ascontiguousarray(x.astype(np.int32))).cuda() for x in (subj, rel, obj, negs, nego)]
    got = []
    for sequential in (1, 0):
        print(f"case dim={dim} negatives={ns}+{no} batch={batch} sequential={sequential}", flush=True)
        srv = P.ParameterServer(K, L, 3)
        srv.set_option(P.OPT_PUSH_SEQUENTIAL, 1)
        srv.push(torch.arange(K, device="cuda"), torch.from_numpy(init).cuda())
        srv.set_option(P.OPT_PUSH_SEQUENTIAL, sequential)
        one = srv.kge_sgd_step(E, dim, *t, 0.1, 1e-10, 1)
        a = srv.pull(torch.arange(K, device="cuda")).cpu().numpy()
        two = srv.kge_sgd_step(E, dim, *t, 0.1, 1e-10, 1)
        part = [0, batch // 3, batch]
        loss = None if stray else srv.kge_sgd_epoch(E, dim, *t, np.array(part), max(1, batch // 2 - 1), 1, 0.1, 1e-10)
        srv.status()
        got.append((a, srv.pull(torch.arange(K, device="cuda")).cpu().numpy(), one, two, loss, srv.stats()))
    (a1, b1, *l1, s1), (a0, b0, *l0, s0) = got
    terms = np.bincount(np.concatenate([subj, rel + E, obj, negs.ravel(), nego.ravel()]), minlength=K)
    rare = terms <= 1
    assert np.array_equal(a1[rare].view(np.uint32), a0[rare].view(np.uint32))
    # a key of n terms in more than one range: n additions in another order, each off by 2^-24 of the partial sum
    assert np.abs(a1 - a0).max() <= terms.max() * 2.0 ** -24 * np.abs(a1).max()
    assert np.abs(b1 - b0).max() <= 2e-5 and s1 == s0
    for x, y in zip(l1, l0):
        assert x is None or abs(x - y) <= 1e-6 * abs(x)


@pytest.mark.parametrize("n", [300, 2048])
def test_a_bad_key_is_seen_by_every_workgroup_of_a_call(n):
    """Calls of few keys in hundreds of workgroups, which set the error while others start: none may miss the bad key."""
    import torch
    from paper_2002_00655_amd import ps as P
    K, L = 3000, 1024
    srv = P.ParameterServer(K, L, 300)
    rng = np.random.default_rng(n)
    good = rng.integers(0, K, size=n)
    before = srv.stats()
    out, own = torch.full((n, L), 7.0, device="cuda"), torch.full((n,), 7, dtype=torch.int32, device="cuda")
    for place in (0, 63, 64, 200, n - 1):
        print(f"case n={n} place={place}", flush=True)
        keys = good.copy()
        keys[place] = K
        kt = torch.from_numpy(keys).cuda()
        for call in (lambda: srv.pull(kt, 2, out=out), lambda: srv.localize(kt, 2), lambda: srv.owner(kt)):
            call()
            with pytest.raises(P.PSError) as e:
                srv.status()
            assert e.value.code == P.PS_EKEY
    assert (out == 7.0).all() and srv.stats() == before
    kt = torch.from_numpy(good).cuda()
    srv.pull(kt, 2, out=out)
    assert (out == 0.0).all() and np.array_equal(srv.owner(kt).cpu().numpy(), good // (K // 300))


def test_a_relation_number_below_zero_shares_an_entity_key():
    """Only the key as a whole has to be in range: a relation number -j names entity E - j.  A negative elsewhere that names
    it is not alone.  Two steps against the same steps with the push's sums only (its sequential order): same bits, since no key
    has more than two terms, and (value + a) + b is what both orders add."""
    import torch
    from paper_2002_00655_amd import ps as P
    E, R, dim, ns, no, batch = 30_000, 200, 40, 4, 4, 400
    rng = np.random.default_rng(21)
    K = E + R
    ids = rng.permutation(E)[:batch * (2 + ns + no)].reshape(batch, -1)     # every entity once
    subj, obj, negs, nego = ids[:, 0], ids[:, 1], ids[:, 2:2 + ns].copy(), ids[:, 2 + ns:].copy()
    rel = np.arange(batch) % R
    rel[:200] = negs[200:, 0] - E                                           # keys of negatives of other data points
    init = np.concatenate([rng.standard_normal((K, 2 * dim)) * 0.1, np.full((K, 2 * dim), 0.01)], 1).astype(np.float32)
    t = [torch.from_numpy(np.ascontiguousarray(x.astype(np.int32))).cuda() for x in (subj, rel, obj, negs, nego)]
    got = []
    for sequential in (1, 0):
        print(f"case sequential={sequential}", flush=True)
        srv = P.ParameterServer(K, 4 * dim, 3)
        srv.push(torch.arange(K, device="cuda"), torch.from_numpy(init).cuda())
        srv.set_option(P.OPT_PUSH_SEQUENTIAL, sequential)
        losses = [srv.kge_sgd_step(E, dim, *t, 0.1, 1e-10, 1) for _ in range(2)]
        srv.status()
        got.append((srv.pull(torch.arange(K, device="cuda")).cpu().numpy()[:E], losses, srv.stats()))
    assert np.array_equal(got[0][0].view(np.uint32), got[1][0].view(np.uint32)) and got[0][1:] == got[1][1:]


@pytest.mark.parametrize("K,L,W", [(3000, 4, 5), (200_000, 2, 256), (200_000, 2, 257), (100_000, 1, 2048)])
def test_statistics_at_the_sizes_where_workgroups_are_added(K, L, W):
    """512 keys: one workgroup counts a call's statistics; 8,192: localize and owner check their keys themselves, and up to 32
    workgroups are counted on one word, more on 16; 131,072: the most workgroups; more than
    256 nodes: pairs by stamps.  Owners are spread by localize calls first; some calls name few destinations many times."""
    import torch
    from oracle.oracle import Oracle
    from paper_2002_00655_amd import ps as P
    rng = np.random.default_rng(W)
    orc, srv = Oracle("f32", K, L, W), P.ParameterServer(K, L, W)
    for n in (1, 256, 257, 511, 512, 513, 2047, 2048, 2049, 8191, 8192, 8193, 8449, 12_288, 30_000, 131_073):
        for same in (False, True):
            print(f"case K={K} W={W} n={n} same={same}", flush=True)
            keys = rng.integers(0, K, size=n) if not same else rng.integers(0, 3, size=n) * (K // 3)
            kt, worker, other = torch.from_numpy(keys).cuda(), int(rng.integers(0, W)), int(rng.integers(0, W))
            d = rng.integers(-4, 5, size=(n, L)).astype(np.float32)
            srv.pull(kt, worker); orc.pull(keys, worker)
            srv.push(kt, torch.from_numpy(d).cuda(), other); orc.push(keys, d, other)
            srv.localize(kt, worker); orc.localize(keys, worker)
            assert np.array_equal(srv.owner(kt).cpu().numpy(), orc.owner()[keys]), n
            srv.pull(kt, other); orc.pull(keys, other)
            assert srv.stats() == orc.stats(), n
    assert np.array_equal(srv.owner().cpu().numpy(), orc.owner())
