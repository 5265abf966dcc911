"""Knowledge-graph steps of a few data points, which are one launch: the same bits, losses and counters as the step that sorts its
keys and adds them strictly in order (PS_OPT_PUSH_SEQUENTIAL takes it), whose arithmetic and order are the same - and steps of
one slot more than fit, and of value lengths around what fits in LDS."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,ns,no,batch", [(1, 1, 1, 1), (10, 5, 5, 4), (10, 5, 5, 5), (64, 0, 0, 21), (65, 0, 3, 2), (100, 5, 5, 1), (100, 5, 5, 3),
                                             (100, 3, 0, 10), (128, 5, 5, 2), (150, 10, 10, 1), (256, 0, 13, 1), (256, 14, 0, 1), (20, 30, 31, 1), (20, 30, 32, 1)])
def test_steps_of_a_few_data_points(dim, ns, no, batch):
    import torch
    from paper_2002_00655_amd import ps as P
    E, R, W = 300, 7, 256
    K, L = E + R, 4 * dim
    rng = np.random.default_rng(dim + 7 * batch)
    init = np.concatenate([rng.standard_normal((K, 2 * dim)) * 0.3, rng.random((K, 2 * dim)) * 0.02], 1).astype(np.float32)
    steps = []
    for i in range(4):
        subj, obj, rel = rng.integers(0, E, batch), rng.integers(0, E, batch), rng.integers(0, R, batch)
        negs, nego = rng.integers(0, E, (batch, ns)), rng.integers(0, E, (batch, no))
        if i == 1:                                                          # keys in several slots
            obj[0] = subj[0]
            negs[:, : ns // 2] = subj[0]
            nego[:, no // 2:] = obj[-1]
        steps.append([torch.from_numpy(np.ascontiguousarray(x.astype(np.int32))).cuda() for x in (subj, rel, obj, negs, nego)])
    got = []
    for sequential in (1, 0):
        srv = P.ParameterServer(K, L, W)
        srv.push(torch.arange(K, device="cuda"), torch.from_numpy(init).cuda())
        srv.set_option(P.OPT_PUSH_SEQUENTIAL, sequential)
        losses = []
        for i, t in enumerate(steps):
            print(f"case dim={dim} ns={ns} no={no} batch={batch} sequential={sequential} step={i}", flush=True)
            losses.append(srv.kge_sgd_step(E, dim, *t, 0.1, 1e-10, i if i < 3 else -1, want_loss=i != 2))
        got.append((srv.pull(torch.arange(K, device="cuda")).cpu().numpy().view(np.uint32), losses, srv.stats()))
    assert np.array_equal(got[0][0], got[1][0])
    assert got[0][1] == got[1][1] and got[0][2] == got[1][2]


@pytest.mark.parametrize("bad", [-1, 10 ** 6])
def test_a_bad_index_changes_nothing(bad):
    import torch
    from paper_2002_00655_amd import ps as P
    E, R, dim = 100, 4, 10
    srv = P.ParameterServer(E + R, 4 * dim, 3)
    srv.push(torch.arange(E + R, device="cuda"), torch.ones(E + R, 4 * dim, device="cuda"), 0)
    stats = srv.stats()
    t = [torch.zeros(2, dtype=torch.int32, device="cuda") for _ in range(3)] + [torch.zeros(2, 3, dtype=torch.int32, device="cuda") for _ in range(2)]
    t[4][1, 2] = bad
    print(f"case bad={bad}", flush=True)
    srv.kge_sgd_step(E, dim, *t, 0.1, 1e-10, 1, want_loss=False)
    with pytest.raises(P.PSError) as e:
        srv.status()
    assert e.value.code == P.PS_EKEY
    assert (srv.pull(torch.arange(E + R, device="cuda")) == 1.0).all() and srv.stats() == stats
