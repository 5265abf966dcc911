"""What the performance of this framework is measured on: the work that a program using it has it do, through the
public entry points of ``paper_2002_00655_amd.ps``.

Five kinds of pass:

``pull``    a worker reads the values of a batch of keys;
``update``  a worker pushes one update row per key and reads the keys back, as the next step of its program does;
``move``    a worker localizes the keys of its next batch, reads them, pushes its updates and looks where they live;
``mf``      one epoch of blocked matrix-factorization SGD, its training error, and the factors read out;
``kge``     one mini-batch step of knowledge-graph-embedding training and the rows of its keys read back (``parts`` = 0),
            or one epoch over that many workers with its loss, and the model read out (``parts`` > 0).

Sizes are those of the framework's own configurations (``workloads.MF_CONFIGS``, ``workloads.make_kge``, the benchmark's
stores), and those between and below them.
"""
import math

import numpy as np
import torch

from paper_2002_00655_amd import workloads as wl

DEV = "cuda"
LR, LAM = 0.01, 0.05                    # matrix factorization
KGE_LR, KGE_EPS = 0.1, 1e-10            # knowledge-graph embeddings


# ---- the cases ----------------------------------------------------------------------------------------------------
def listed():
    big = dict(keys=497_959, length=100, workers=256)                       # the store of a 480,189 x 17,770 matrix at rank 100
    return [
        # the keys of a handful of data points: what a program that goes point by point pays per call
        dict(name="pull_small", kind="pull", n=100, skew=1.0, **big),
        # a large batch, or a checkpoint of the model: bound by memory
        dict(name="pull_bulk", kind="pull", n=1_000_003, skew=1.0, **big),
        # the terms of a few data points pushed and read back
        dict(name="update_small", kind="update", n=333, skew=1.0, **big),
        # as many terms as a large mini-batch has, frequent keys among them thousands of times
        dict(name="update_bulk", kind="update", n=1_000_003, skew=1.0, **big),
        # parameters that move between a few workers, at a rank whose rows do not start on 16 bytes
        dict(name="move_mid", kind="move", n=20_001, skew=0.0, keys=110_000, length=50, workers=8),
        # MF_CONFIGS["tiny"]: 16 small blocks, launches count
        dict(name="mf_tiny", kind="mf", m=1000, n=1000, nnz=100_000, row_skew=0.0, col_skew=0.0, rank=16, d=4, cost=8.0),
        # MF_CONFIGS["medium"]: fewer blocks in flight than the chip has compute units, rank 50
        dict(name="mf_medium", kind="mf", m=100_000, n=10_000, nnz=10_000_000, row_skew=1.0, col_skew=1.0, rank=50, d=64, cost=8.0),
        # MF_CONFIGS["large"]
        dict(name="mf_large", kind="mf", m=480_189, n=17_770, nnz=100_000_000, row_skew=1.0, col_skew=1.0, rank=100, d=256, cost=8.0),
        # MF_CONFIGS["wide"] at a fifth in every direction: mostly one entry per row and block, columns with a million
        dict(name="mf_wide", kind="mf", m=2_000_000, n=200_000, nnz=100_000_000, row_skew=0.0, col_skew=1.1, rank=100, d=256, cost=3.0),
        # one data point per step, the access pattern the method's experiments describe
        dict(name="kge_point", kind="kge", entities=500_000, relations=600, dim=100, triples=1, ns=5, no=5, batch=1, parts=0, ahead=False),
        # the batch of the ComplEx benchmark
        dict(name="kge_batch", kind="kge", entities=500_000, relations=600, dim=100, triples=8192, ns=5, no=5, batch=8192, parts=0, ahead=False),
        # an epoch over four workers with pre-localization, batches of 1,024
        dict(name="kge_epoch", kind="kge", entities=500_000, relations=600, dim=100, triples=32_768, ns=5, no=5, batch=1024, parts=4, ahead=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pull", "update", "move", "mf", "mf", "kge", "kge"])
    if kind in ("pull", "update", "move"):
        length = rng.choice([16, 50, 64, 100, 128, 400, rng.randint(1, 255)])
        return dict(kind=kind, n=_log_int(rng, 1, 1_000_000), skew=rng.choice([0.0, 1.0]), keys=_log_int(rng, 2000, 500_000), length=length,
                    workers=rng.choice([1, 2, 4, 8, 64, 256]))
    if kind == "mf":
        m, n, d = _log_int(rng, 400, 60_000), _log_int(rng, 300, 20_000), rng.choice([4, 8, 16, 32, 64])
        d = max(d, 8) if m > 20_000 else d
        nnz = min(_log_int(rng, 5_000, 8_000_000), m * n // 8, 150_000 * d)
        return dict(kind="mf", m=m, n=n, nnz=nnz, row_skew=rng.choice([0.0, 1.0]), col_skew=rng.choice([0.0, 1.0, 1.1]),
                    rank=rng.choice([8, 16, 32, 50, 64, 100, 128, rng.randint(1, 128)]), d=d, cost=8.0)
    dim = rng.choice([10, 50, 64, 100, 128, rng.randint(1, 150)])
    parts = rng.choice([0, 0, 0, 1, 2, 4, 8])
    triples = _log_int(rng, 2_000, 30_000) if parts else _log_int(rng, 1, 8192)
    batch = _log_int(rng, 200, 2048) if parts else triples
    return dict(kind="kge", entities=_log_int(rng, 1000, 500_000), relations=_log_int(rng, 5, 600), dim=dim, triples=triples,
                ns=rng.randint(0, 10), no=rng.randint(0, 10), batch=batch, parts=parts, ahead=bool(parts) and rng.random() < 0.7)


# ---- inputs -------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, device=DEV, generator=g)


def _probs(size, skew, cap, g):
    """rank^-skew, none above cap, dealt to the ids by a random permutation."""
    p = torch.arange(1, size + 1, dtype=torch.float64, device=DEV) ** -skew
    p = p / p.sum()
    cap = max(cap, 1.5 / size)
    for _ in range(30):
        over = p >= cap
        rest = 1.0 - cap * int(over.sum())
        p = torch.where(over, cap, p * (rest / p[~over].sum()))
        if float(p.max()) <= cap * (1 + 1e-9):
            break
    return p[torch.randperm(size, device=DEV, generator=g)]


def _ids(size, count, cdf, g):
    if cdf is None:
        return torch.randint(0, size, (count,), device=DEV, generator=g)
    u = torch.rand(count, device=DEV, generator=g, dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=size - 1)


def _cdf(size, skew, cap, g):
    return None if skew == 0.0 else torch.cumsum(_probs(size, skew, cap, g), 0)


def _store(c, seed):
    """keys of one batch, update rows, initial values"""
    g = _gen(seed)
    keys = _ids(c["keys"], c["n"], _cdf(c["keys"], c["skew"], 0.02, g), g)
    values = (_rand(g, c["keys"], c["length"]) - 0.5) * 0.2
    deltas = (_rand(g, c["n"], c["length"]) - 0.5) * 0.02
    return keys, values, deltas


def _ratings(c, seed):
    """rows, columns, values of the revealed cells, initial factors"""
    g = _gen(seed)
    m, n, nnz = c["m"], c["n"], c["nnz"]
    cdf_r, cdf_c = _cdf(m, c["row_skew"], 0.5 * n / nnz, g), _cdf(n, c["col_skew"], 0.5 * m / nnz, g)
    have = torch.empty(0, dtype=torch.int64, device=DEV)
    while have.numel() < nnz:
        count = int((nnz - have.numel()) * 1.1) + 1024
        have = torch.unique(torch.cat([have, _ids(m, count, cdf_r, g) * n + _ids(n, count, cdf_c, g)]))
    if have.numel() > nnz:                                     # drop random ones
        keep = torch.ones(have.numel(), dtype=torch.bool, device=DEV)
        keep[torch.randperm(have.numel(), device=DEV, generator=g)[: have.numel() - nnz]] = False
        have = have[keep]
    rows, cols = (have // n).to(torch.int32), (have % n).to(torch.int32)
    del have
    k = 16                                                     # a planted model plus noise
    U, V = torch.randn(m, k, device=DEV, generator=g) * k ** -0.5, torch.randn(n, k, device=DEV, generator=g) * k ** -0.5
    vals = torch.empty(nnz, device=DEV)
    for a in range(0, nnz, 1 << 22):
        vals[a:a + (1 << 22)] = (U[rows[a:a + (1 << 22)].long()] * V[cols[a:a + (1 << 22)].long()]).sum(1)
    vals += 0.1 * torch.randn(nnz, device=DEV, generator=g)
    init = (_rand(g, m + n, c["rank"]) - 0.5) * c["rank"] ** -0.5
    return rows, cols, vals, init


def _bounds(ids, size, d, per_id):
    """d ranges of about equal weight (an index weighs its entries + per_id); an index with more entries than an
    average range is a range of its own."""
    count = torch.bincount(ids, minlength=size).cpu().numpy().astype(np.float64)
    heavy = np.flatnonzero(count > count.sum() / d)
    heavy = heavy if 2 * heavy.size < d else heavy[:0]
    light = count + per_id
    light[heavy] = 0.0
    cum = np.cumsum(light)
    cuts = d - 1 - 2 * heavy.size
    inner = np.searchsorted(cum, cum[-1] * np.arange(1, cuts + 1) / (cuts + 1)) + 1
    inner = np.sort(np.concatenate([inner, heavy, heavy + 1]))
    return np.concatenate([[0], np.clip(inner, 0, size), [size]]).astype(np.int64)


def _triples(c, seed):
    """triples with their negatives, grouped by worker (all triples of a relation with one worker), initial values and accumulators"""
    g = _gen(seed)
    T, E, R = c["triples"], c["entities"], c["relations"]
    cdf_e, cdf_r = _cdf(E, 1.0, 0.02 + 4.0 / E, g), _cdf(R, 1.0, 0.2 + 4.0 / R, g)
    subj, obj, rel = _ids(E, T, cdf_e, g), _ids(E, T, cdf_e, g), _ids(R, T, cdf_r, g)
    negs, nego = torch.randint(0, E, (T, c["ns"]), device=DEV, generator=g), torch.randint(0, E, (T, c["no"]), device=DEV, generator=g)
    part_ptr = None
    if c["parts"]:
        part = rel % c["parts"]
        order = torch.argsort(part, stable=True)
        subj, obj, rel, negs, nego = subj[order], obj[order], rel[order], negs[order], nego[order]
        part_ptr = np.concatenate([[0], np.cumsum(torch.bincount(part, minlength=c["parts"]).cpu().numpy())]).astype(np.int64)
    init = torch.cat([0.1 * torch.randn(E + R, 2 * c["dim"], device=DEV, generator=g),
                      0.01 + 0.02 * _rand(g, E + R, 2 * c["dim"])], 1)      # after some training: the accumulators are not zero
    return [x.to(torch.int32) for x in (subj, rel, obj, negs, nego)], part_ptr, init


def _slots(c, t):
    """the keys a knowledge-graph step touches, one per slot of a data point"""
    subj, rel, obj, negs, nego = (x.long() for x in t)
    return torch.cat([subj[:, None], rel[:, None] + c["entities"], obj[:, None], negs, nego], 1)


def _read(c, t):
    """the keys read after a pass: a step's own, or the whole model"""
    return torch.arange(c["entities"] + c["relations"], device=DEV) if c["parts"] else _slots(c, t).reshape(-1)


# ---- a pass -------------------------------------------------------------------------------------------------------
def _server(K, L, W, init):
    from paper_2002_00655_amd import ps as P
    srv = P.ParameterServer(K, L, W)
    for lo in range(0, K, 1 << 18):
        hi = min(K, lo + (1 << 18))
        srv.push(torch.arange(lo, hi, device=DEV), init[lo:hi])
    return srv


def prepare(case, seed):
    c = case
    if c["kind"] == "mf":
        from paper_2002_00655_amd import ps as P
        rows, cols, vals, init = _ratings(c, seed)
        m, n, d = c["m"], c["n"], c["d"]
        rb, cb = _bounds(rows, m, d, 0.0), _bounds(cols, n, d, c["cost"] * d)
        br, bc, bv, bp = P.mf_block_ratings(m, n, rows, cols, vals, rb, cb)
        srv = _server(m + n, c["rank"], d, init)
        srv.mf_load_ratings(m, n, br, bc, bv, rb, cb, bp)
        tasks = np.ascontiguousarray(wl.cyclic_schedule(d).reshape(-1, 3))
        return dict(c=c, srv=srv, tasks=tasks, sptr=(np.arange(d + 1) * d).astype(np.int32), all=torch.arange(m + n, device=DEV))
    if c["kind"] == "kge":
        t, part_ptr, init = _triples(c, seed)
        srv = _server(c["entities"] + c["relations"], 4 * c["dim"], max(1, c["parts"]), init)
        return dict(c=c, srv=srv, t=t, part_ptr=part_ptr, read=_read(c, t))
    keys, values, deltas = _store(c, seed)
    srv = _server(c["keys"], c["length"], c["workers"], values)
    return dict(c=c, srv=srv, keys=keys, deltas=deltas, worker=c["workers"] // 2)


def run(state):
    c, srv = state["c"], state["srv"]
    if c["kind"] == "pull":
        return srv.pull(state["keys"], worker=state["worker"])
    if c["kind"] == "update":
        srv.push(state["keys"], state["deltas"], worker=state["worker"])
        return srv.pull(state["keys"], worker=state["worker"])
    if c["kind"] == "move":
        state["worker"] = (state["worker"] + 1) % c["workers"]                 # the keys move on every pass
        srv.localize(state["keys"], state["worker"])
        before = srv.pull(state["keys"], worker=state["worker"])
        srv.push(state["keys"], state["deltas"], worker=state["worker"])
        return dict(before=before, after=srv.pull(state["keys"], worker=state["worker"]), owner=srv.owner(state["keys"]))
    if c["kind"] == "mf":
        srv.mf_sgd_epoch_raw(state["tasks"], state["sptr"], LR, LAM)
        sse = srv.mf_train_sse()
        return dict(factors=srv.pull(state["all"]), sse=sse)
    t = state["t"]
    if c["parts"]:
        loss = srv.kge_sgd_epoch(c["entities"], c["dim"], *t, state["part_ptr"], c["batch"], c["ahead"], KGE_LR, KGE_EPS)
        return dict(rows=srv.pull(state["read"]), loss=loss)
    srv.kge_sgd_step(c["entities"], c["dim"], *t, KGE_LR, KGE_EPS, worker=0, want_loss=False)
    return srv.pull(state["read"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _distinct(size, count, skew, cap):
    """expected number of different ids among `count` drawn ones"""
    if skew == 0.0:
        return size * -math.expm1(count * math.log1p(-1.0 / size)) if size > 1 else 1.0
    p = np.arange(1, size + 1, dtype=np.float64) ** -skew
    p = np.minimum(p / p.sum(), max(cap, 1.5 / size))
    return float((1 - np.exp(-count * p)).sum())


def work(case):
    c = case
    if c["kind"] == "mf":
        factors = 4.0 * (c["m"] + c["n"]) * c["rank"]
        # factors read, written and read out, entries read; per entry an inner product, two updated rows, and the error's inner product
        return dict(bytes=3 * factors + 12.0 * c["nnz"], flops=10.0 * c["rank"] * c["nnz"])
    if c["kind"] == "kge":
        row, per, slots = 16.0 * c["dim"], 1 + c["ns"] + c["no"], 3 + c["ns"] + c["no"]
        batches = max(1, -(-c["triples"] // c["batch"]))
        B = c["triples"] / batches
        E, R = c["entities"], c["relations"]

        def rows(T):
            return _distinct(E, 2 * T, 1.0, 0.02 + 4.0 / E) + _distinct(R, T, 1.0, 0.2 + 4.0 / R) + _distinct(E, (c["ns"] + c["no"]) * T, 0.0, 1.0)
        # every step reads and writes the rows it touches; then the rows of a step, or of the model, are read out
        out = row * ((E + R) if c["parts"] else slots * c["triples"])
        return dict(bytes=2 * row * rows(B) * batches + out + 4.0 * slots * c["triples"],
                    flops=c["triples"] * c["dim"] * (30.0 * per + 12.0 * slots))
    n, row = c["n"], 4.0 * c["length"]
    rows = _distinct(c["keys"], n, c["skew"], 0.02)
    pulled = rows * row + n * (row + 8.0)                       # stored rows read, the result written
    pushed = n * (row + 8.0) + 2 * rows * row                   # update rows read, stored rows read and written
    if c["kind"] == "pull":
        return dict(bytes=pulled, flops=0.0)
    if c["kind"] == "update":
        return dict(bytes=n * (row + 8.0) + 2 * rows * row + n * row, flops=float(n) * c["length"])
    return dict(bytes=pulled + pushed + n * row + n * 12.0, flops=float(n) * c["length"])


def tolerance(case):
    """About four times what two correct orders of the same sums differ by: the default path against the checking modes
    (a key's terms one after the other; entry by entry; scores summed in index order), measured on the listed cases:
    rel / max 2.3e-6 / 1.5e-5 (update), 7.0e-7 / 8.5e-6 (mf), 4.1e-7 / 8.4e-6 (kge)."""
    if case["kind"] == "pull":
        return "exact"
    return {"mf": {"rel": 4e-6, "max": 6e-5}, "kge": {"rel": 2e-6, "max": 4e-5}}.get(case["kind"], {"rel": 1e-5, "max": 6e-5})


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------
def _blocked(rows, cols, rb, cb):
    """entries block by block (row-block major), a block's columns by decreasing count, a column's entries by row; block pointers"""
    d, n = rb.size - 1, int(cb[-1])
    br = torch.searchsorted(torch.from_numpy(rb).to(DEV), rows.long(), right=True) - 1
    bc = torch.searchsorted(torch.from_numpy(cb).to(DEV), cols.long(), right=True) - 1
    count = torch.bincount(br * n + cols, minlength=d * n)[br * n + cols]
    order = torch.argsort(rows, stable=True)
    for key in (cols, -count, br * d + bc):
        order = order[torch.argsort(key[order], stable=True)]
    ptr = torch.cumsum(torch.bincount(br * d + bc, minlength=d * d), 0).cpu().numpy()
    return order, np.concatenate([[0], ptr])


def _exact_mf(c, seed):
    d, m = c["d"], c["m"]
    rows, cols, vals, init = _ratings(c, seed)
    rb, cb = _bounds(rows, m, d, 0.0), _bounds(cols, c["n"], d, c["cost"] * d)
    order, ptr = _blocked(rows, cols, rb, cb)
    r, q, v = (x[order].cpu().numpy() for x in (rows.long(), cols.long() + m, vals.double()))
    length = np.diff(ptr).reshape(d, d)
    b = np.arange(d)
    steps = sum(int(length[b, (b + s) % d].max()) for s in range(d))
    if steps * (20e-6 + 6e-9 * d * c["rank"]) > 15:
        return None
    val = init.double().cpu().numpy()
    for s in range(d):                                      # the tasks of a stratum share neither rows nor columns: side by side
        cb_s = (b + s) % d
        start, size = ptr[:-1].reshape(d, d)[b, cb_s], length[b, cb_s]
        by_size = np.argsort(-size, kind="stable")
        start, size = start[by_size], size[by_size]
        for t in range(int(size[0]) if d else 0):
            p = start[: int(np.searchsorted(-size, -t))] + t
            i, j = r[p], q[p]
            w, h = val[i], val[j]
            e = (v[p] - np.einsum("ij,ij->i", w, h))[:, None]
            val[i] = w + LR * (e * h - LAM * w)
            val[j] = h + LR * (e * w - LAM * h)
    e = v - np.einsum("ij,ij->i", val[r], val[q])
    return dict(factors=val, sse=float((e * e).sum()))


def _exact_kge_step(c, val, t):
    D, B = c["dim"], t[0].numel()
    slot = _slots(c, t)
    x = val[slot]                                           # [B, slots, 4 D]
    z, G = torch.complex(x[..., :D].contiguous(), x[..., D:2 * D].contiguous()), x[..., 2 * D:]
    s, r, o, ns, no = z[:, 0:1], z[:, 1:2], z[:, 2:3], z[:, 3:3 + c["ns"]], z[:, 3 + c["ns"]:]
    loss, grads = 0.0, [torch.zeros_like(a) for a in (s, r, o)]
    own = []
    for a, w, label in ((s, o, 1.0), (ns, o, -1.0), (s, no, -1.0)):
        k = max(a.shape[1], w.shape[1]) if min(a.shape[1], w.shape[1]) else 0
        if k == 0:
            own.append(a[:, :0])
            continue
        score = (a * r * w.conj()).real.sum(-1, keepdim=True)
        loss += float(torch.nn.functional.softplus(-label * score).sum())
        dl = -label * torch.sigmoid(-label * score)
        ga, gr, gw = dl * r.conj() * w, dl * a.conj() * w, dl * a * r
        grads[1] = grads[1] + gr.sum(1, keepdim=True)
        if a is ns:
            own.append(ga)
        else:
            grads[0] = grads[0] + ga.sum(1, keepdim=True)
        if w is no:
            own.append(gw)
        else:
            grads[2] = grads[2] + gw.sum(1, keepdim=True)
    g = torch.cat(grads + own, 1)
    g = torch.cat([g.real, g.imag], -1)
    step = torch.cat([-KGE_LR * g / torch.sqrt(G + g * g + KGE_EPS), g * g], -1)
    val.index_add_(0, slot.reshape(-1), step.reshape(B * slot.shape[1], 4 * D))
    return loss


def exact(case, seed):
    c = case
    if c["kind"] == "mf":
        return _exact_mf(c, seed)
    if c["kind"] == "kge":
        t, part_ptr, init = _triples(c, seed)
        val = init.double()
        if not c["parts"]:
            _exact_kge_step(c, val, t)
            return val[_read(c, t)]
        loss = 0.0
        for at in range(0, int(np.diff(part_ptr).max()), c["batch"]):         # the workers take turns
            for w in range(c["parts"]):
                lo, hi = int(part_ptr[w]) + at, min(int(part_ptr[w]) + at + c["batch"], int(part_ptr[w + 1]))
                if lo < hi:
                    loss += _exact_kge_step(c, val, [x[lo:hi] for x in t])
        return dict(rows=val[_read(c, t)], loss=loss)
    keys, values, deltas = _store(c, seed)
    val = values.double()
    before = val[keys]
    if c["kind"] == "pull":
        return before
    val.index_add_(0, keys, deltas.double())
    return val[keys] if c["kind"] == "update" else dict(before=before, after=val[keys], owner=None)
