"""The measured cases: what a user of this library has it do, through the entry
points of ``paper_1508_00703_amd.native``, with inputs shaped like the
repository's own workloads (``datagen.CONFIGS`` / ``DENSE``), drawn on the GPU.

A case's ``op`` is the call that one pass makes:

  schedule    pdb_schedule: levels, grouping and previous writers of a CSR
  epoch       pdb_sgd_epoch on a schedule the program keeps
  step        pdb_schedule, then pdb_sgd_epoch (or pdb_mf_epoch)
  mb_epoch    pdb_batch_epoch on a batch schedule the program keeps
  mb_step     pdb_batch_schedule, then pdb_batch_epoch
  delay       pdb_stale_epoch
  dense       pdb_dense_gd

The other fields give the input: ``n`` examples over ``d`` features, ``lo`` to
``hi`` entries per example (uniform, or Poisson with mean ``mean``), feature ids
Zipf(``alpha``) or uniform (``alpha`` 0), stored values ``val`` ("ones",
"normal", "lognormal"), the loss ("logistic" or "squared") and its step size.
"""
import math

import numpy as np
import torch

from paper_1508_00703_amd import native

RANK = 32


# ---------------------------------------------------------------------------
# the cases

def _sparse(name, op, n, d, lo, hi, alpha, val, loss, lr, mean=0.0, **more):
    return dict(name=name, op=op, n=n, d=d, lo=lo, hi=hi, mean=mean, alpha=alpha, val=val,
                loss=loss, lr=lr, **more)


def listed():
    return [
        # the smallest training job of the benchmark, whole: a schedule and an
        # epoch on ten thousand short examples, where launches, host waits and
        # the latency of a dependent chain are all there is
        _sparse("step-small", "step", 10_000, 1_000, 10, 10, 1.0, "normal", "logistic", 0.1),
        # scheduling a large click-log-like set: binary, Zipf-hot features, every
        # example in conflict with the one before it
        _sparse("schedule-zipf", "schedule", 2_000_000, 1_000_000, 50, 50, 1.2, "ones",
                "logistic", 0.01),
        # training on it: one dependent chain through the hot features
        _sparse("epoch-zipf", "epoch", 1_000_000, 1_000_000, 50, 50, 1.2, "ones", "logistic",
                0.01),
        # real-valued features, ragged rows of an odd count, still chain-like
        _sparse("epoch-ragged", "epoch", 200_003, 100_000, 20, 40, 1.1, "lognormal", "logistic",
                0.05),
        # scheduling where conflicts are rare (uniform features): wide levels
        _sparse("schedule-uniform", "schedule", 1_000_000, 2_000_000, 1, 400, 0.0, "normal",
                "squared", 0.001, mean=80.0),
        # training there: examples of many levels in flight over the whole chip
        _sparse("epoch-uniform", "epoch", 1_000_000, 2_000_000, 1, 400, 0.0, "normal", "squared",
                0.001, mean=80.0),
        # matrix completion, schedule and epoch: Zipf users and items
        dict(name="step-mf", op="step", mf=True, n=4_000_000, users=1_000_000, items=200_000,
             lr=0.005, reg=0.02),
        # mini-batches of 100 (the paper's size) on rare conflicts, batch
        # schedule and epoch
        _sparse("minibatch-uniform", "mb_step", 500_000, 2_000_000, 1, 400, 0.0, "normal",
                "squared", 0.00001, mean=80.0, batch=100),
        # mini-batches of 100 where hot features are in every example, one of
        # many epochs on a kept schedule
        _sparse("minibatch-zipf", "mb_epoch", 500_000, 1_000_000, 50, 50, 1.2, "ones", "logistic",
                0.0001, batch=100),
        # bounded delay on a chain-like set (the paper's asynchronous reads)
        _sparse("delay-ragged", "delay", 200_000, 100_000, 20, 40, 1.1, "lognormal", "logistic",
                0.05, delay=8),
        # dense linear regression of the paper's first experiment: the matrix
        # fits on chip, iterations are short
        dict(name="dense-resident", op="dense", n=5_000, d=960, iters=200, loss="squared",
             lr=1e-4),
        # and the widest of its feature sweep: the matrix streams from memory
        dict(name="dense-streamed", op="dense", n=500, d=1_000_000, iters=50, loss="squared",
             lr=1e-6),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["zipf", "zipf", "uniform", "uniform", "mf", "mb", "mb", "delay", "dense",
                       "dense"])
    if kind == "zipf":
        op = rng.choice(["schedule", "epoch", "step"])
        lo = rng.randint(5, 50)
        return _sparse_drawn(op, _log(rng, 10_000, 1_000_000 if op != "schedule" else 2_000_000),
                             _log(rng, 1_000, 1_000_000), lo, rng.choice([lo, min(60, 2 * lo)]),
                             rng.choice([1.0, 1.1, 1.2]), rng)
    if kind == "uniform":
        op = rng.choice(["schedule", "epoch", "step"])
        d = _log(rng, 200_000, 2_000_000)
        return _sparse_drawn(op, _log(rng, 20_000, 1_000_000), d, 1, 400, 0.0, rng,
                             mean=float(rng.randint(20, 80)))
    if kind == "mf":
        return dict(op=rng.choice(["schedule", "epoch", "step"]), mf=True,
                    n=_log(rng, 50_000, 4_000_000), users=_log(rng, 20_000, 1_000_000),
                    items=_log(rng, 5_000, 200_000), lr=0.005, reg=0.02)
    if kind == "mb":
        zipf = rng.random() < 0.5
        batch = rng.choice([32, 50, 100, 128, 200])
        return _sparse_drawn(rng.choice(["mb_epoch", "mb_step"]), _log(rng, 20_000, 500_000),
                             _log(rng, 200_000, 2_000_000), 30 if zipf else 1, 50 if zipf else 400,
                             1.2 if zipf else 0.0, rng, mean=0.0 if zipf else 80.0, batch=batch)
    if kind == "delay":
        zipf = rng.random() < 0.7
        return _sparse_drawn("delay", _log(rng, 10_000, 200_000),
                             _log(rng, 10_000, 200_000) if zipf else _log(rng, 200_000, 2_000_000),
                             20 if zipf else 1, 40 if zipf else 400, 1.1 if zipf else 0.0, rng,
                             mean=0.0 if zipf else 80.0, delay=rng.choice([1, 4, 8, 15, 31]))
    if rng.random() < 0.5:
        n, d = _log(rng, 500, 5_000), _log(rng, 200, 1_500)
        return dict(op="dense", n=n, d=d, iters=rng.randint(50, 200),
                    loss=rng.choice(["squared", "logistic"]),
                    lr=0.5 / (math.sqrt(n) + math.sqrt(d)) ** 2)
    n, d = rng.randint(200, 1_000), _log(rng, 100_000, 1_000_000) // 2
    return dict(op="dense", n=n, d=d, iters=rng.randint(10, 50),
                loss=rng.choice(["squared", "logistic"]),
                lr=0.5 / (math.sqrt(n) + math.sqrt(d)) ** 2)


def _sparse_drawn(op, n, d, lo, hi, alpha, rng, mean=0.0, **more):
    if alpha == 0.0:
        val, loss, lr = rng.choice(["normal", "ones"]), "squared", 0.001
    else:
        val, loss = rng.choice(["ones", "normal", "lognormal"]), "logistic"
        lr = 0.01 if val == "ones" else 0.05
    if "batch" in more:
        lr /= more["batch"]
    c = _sparse("", op, n, d, lo, hi, alpha, val, loss, lr, mean=mean, **more)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs

DEV = "cuda"


def _zipf_cdf(d, alpha):
    p = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow_(-alpha)
    c = torch.cumsum(p.cpu(), 0)  # on the host: the same sums every time
    return (c / c[-1]).to(DEV)


def _ids(shape, d, cdf, g):
    if cdf is None:
        return torch.randint(0, d, shape, generator=g, device=DEV)
    u = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=d - 1)


def _csr(case, seed):
    """row_ptr, col, val, labels.  Each example's ids are its first m distinct
    draws, in ascending order; the entry counts m depend on the case alone, so
    that every seed gives arrays of the same sizes."""
    g = torch.Generator(device=DEV).manual_seed(seed * 2 + 1)
    n, d, lo, hi = case["n"], case["d"], case["lo"], case["hi"]
    cdf = _zipf_cdf(d, case["alpha"]) if case["alpha"] else None
    wstar = torch.randn(d, generator=g, device=DEV, dtype=torch.float64)
    gm = torch.Generator(device=DEV).manual_seed(n)
    rows = 1 << 17
    counts, cols, vals, ys = [], [], [], []
    for r0 in range(0, n, rows):
        R = min(rows, n - r0)
        if case["mean"]:
            m = torch.poisson(torch.full((R,), case["mean"], device=DEV), generator=gm)
            m = m.long().clamp_(lo, hi)
        else:
            m = torch.randint(lo, hi + 1, (R,), generator=gm, device=DEV)
        most = int(m.max())
        if cdf is None:
            ids = _ids((R, most + 8), d, None, g)
        else:  # where the draws hold fewer than m distinct ids, the hottest complete them
            hot = torch.arange(most, device=DEV).expand(R, most)
            ids = torch.cat([_ids((R, 4 * most), d, cdf, g), hot], 1)
        D = ids.shape[1]
        ids, at = ids.sort(dim=1, stable=True)
        first = torch.ones_like(ids, dtype=torch.bool)
        first[:, 1:] = ids[:, 1:] != ids[:, :-1]
        drawn = torch.zeros_like(first).scatter_(1, at, first)  # a new id, in draw order
        taken = drawn & (drawn.to(torch.int32).cumsum(1) <= m[:, None])
        keep = taken.gather(1, at)
        if case["val"] == "ones":
            x = None
            margin = (wstar[ids] * keep).sum(1)
        else:
            x = torch.randn((R, D), generator=g, device=DEV)
            if case["val"] == "lognormal":
                sign = torch.randint(0, 2, (R, D), generator=g, device=DEV) * 2 - 1
                x = sign * torch.exp(0.5 * x)
            margin = (wstar[ids] * x * keep).sum(1)
            vals.append(x[keep])
        if case["loss"] == "logistic":
            flip = torch.rand(R, generator=g, device=DEV) < 0.05
            ys.append(torch.where((margin >= 0) != flip, 1.0, -1.0))
        else:
            ys.append((margin + 0.1 * torch.randn(R, generator=g, device=DEV)).float())
        counts.append(keep.sum(1))
        cols.append(ids[keep].to(torch.int32))
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cat(counts).cumsum(0)
    return (row_ptr, torch.cat(cols), torch.cat(vals) if vals else None,
            torch.cat(ys).float().contiguous())


def _ratings(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed * 2 + 1)
    n, nu, ni = case["n"], case["users"], case["items"]
    user = _ids((n,), nu, _zipf_cdf(nu, 1.0), g)
    item = _ids((n,), ni, _zipf_cdf(ni, 1.0), g)
    sd = RANK ** -0.5
    us = torch.randn((nu, RANK), generator=g, device=DEV) * sd
    vs = torch.randn((ni, RANK), generator=g, device=DEV) * sd
    r = (us[user].double() * vs[item].double()).sum(1) + 0.5 * torch.randn(n, generator=g,
                                                                          device=DEV)
    U = torch.randn((nu, RANK), generator=g, device=DEV) * sd
    V = torch.randn((ni, RANK), generator=g, device=DEV) * sd
    return user.to(torch.int32), item.to(torch.int32), r.float(), U, V


def _dense(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed * 2 + 1)
    n, d = case["n"], case["d"]
    X = torch.empty((n, d), device=DEV)
    margin = torch.empty(n, dtype=torch.float64, device=DEV)
    wstar = torch.randn(d, generator=g, device=DEV, dtype=torch.float64)
    for i in range(0, n, 64):  # in slabs: the double-precision products stay small
        X[i:i + 64].normal_(generator=g)
        margin[i:i + 64] = (X[i:i + 64].double() * wstar).sum(1) / math.sqrt(d)
    noise = torch.randn(n, generator=g, device=DEV)
    if case["loss"] == "logistic":
        y = torch.where(margin >= 0, 1.0, -1.0)
    else:
        y = margin + 0.1 * noise
    return X, y.float().contiguous()


def _loss(case):
    return native.PDB_LOGISTIC if case["loss"] == "logistic" else native.PDB_SQUARED


def prepare(case, seed):
    op = case["op"]
    s = dict(case=case, op=op)
    if op == "dense":
        s["X"], s["y"] = _dense(case, seed)
        s["w"] = torch.zeros(case["d"], device=DEV)
        s["blocks"] = native.pdb_dense_plan(case["n"], case["d"])
        s["ws"] = native.workspace(
            native.pdb_dense_workspace_bytes(case["n"], case["d"], *s["blocks"]), DEV)
        return s
    n = case["n"]
    if case.get("mf"):
        s["user"], s["item"], s["r"], s["U"], s["V"] = _ratings(case, seed)
        d = case["users"] + case["items"]
        col = torch.stack([s["user"], s["item"] + case["users"]], 1).reshape(-1).contiguous()
        row_ptr = torch.arange(0, 2 * n + 1, 2, dtype=torch.int64, device=DEV)
        s["csr"] = native.Csr(row_ptr, col, None)
        words = d * RANK
    else:
        row_ptr, col, val, s["y"] = _csr(case, seed)
        s["csr"] = native.Csr(row_ptr, col, val)
        d = words = case["d"]
        s["w"] = torch.zeros(d, device=DEV)
    s["d"] = d
    nnz = s["csr"].nnz
    if op in ("mb_epoch", "mb_step"):
        s["bt"] = native.Batches(n, nnz, case["batch"], DEV)
        s["lv"] = native.Levels(s["bt"].nb, nnz, DEV)
        for t in (s["bt"].ucol, s["bt"].uptr):
            t.fill_(-1)
    else:
        s["lv"] = native.Levels(n, nnz, DEV)
    # the arrays hold the most levels (unions) there can be; -1 where a schedule has none
    for t in (s["lv"].level_ptr, s["lv"].prev_nz):
        t.fill_(-1)
    s["sws"] = native.workspace(native.pdb_schedule_workspace_bytes(n, d, nnz), DEV)
    s["ws"] = native.workspace(native.pdb_stale_workspace_bytes(nnz) if op == "delay" else
                               native.pdb_epoch_workspace_bytes(words), DEV)
    if op in ("epoch", "delay"):
        native.pdb_schedule(s["csr"], None, n, d, s["lv"], ws=s["sws"])
    elif op == "mb_epoch":
        native.pdb_batch_schedule(s["csr"], n, d, s["bt"], s["lv"], ws=s["sws"])
    return s


# ---------------------------------------------------------------------------
# one pass

def run(s):
    case, op = s["case"], s["op"]
    n = case["n"]
    if op == "dense":
        native.pdb_dense_gd(s["X"], s["y"], s["w"], case["lr"], _loss(case), case["iters"],
                            *s["blocks"], ws=s["ws"])
        return s["w"]
    csr, lv, d = s["csr"], s["lv"], s["d"]
    out = ()
    if op in ("schedule", "step"):
        native.pdb_schedule(csr, None, n, d, lv, ws=s["sws"])
        out = (lv.level, lv.perm, lv.level_ptr, lv.prev_nz)
    elif op == "mb_step":
        native.pdb_batch_schedule(csr, n, d, s["bt"], lv, ws=s["sws"])
        bt = s["bt"]
        out = (lv.level, lv.perm, lv.level_ptr, lv.prev_nz, bt.bptr, bt.ucol, bt.uptr, bt.occ)
    if op in ("epoch", "step"):
        if case.get("mf"):
            native.pdb_mf_epoch(s["user"], s["item"], s["r"], n, s["U"], case["users"], s["V"],
                                case["items"], RANK, case["lr"], case["reg"], lv, ws=s["ws"])
            out += (s["U"], s["V"])
        else:
            native.pdb_sgd_epoch(csr, s["y"], n, d, s["w"], case["lr"], _loss(case), lv,
                                 ws=s["ws"])
            out += (s["w"],)
    elif op in ("mb_epoch", "mb_step"):
        native.pdb_batch_epoch(csr, s["y"], n, d, s["w"], case["lr"], _loss(case), s["bt"], lv,
                               ws=s["ws"])
        out += (s["w"],)
    elif op == "delay":
        native.pdb_stale_epoch(csr, s["y"], n, d, s["w"], case["lr"], _loss(case), case["delay"],
                               lv, ws=s["ws"])
        out = (s["w"],)
    return out


def work(case):
    op = case["op"]
    n, d = case["n"], case.get("d", 0)
    if op == "dense":
        # the matrix once on chip, else once per iteration; labels, weights
        fits = n * d * 4 <= 32 << 20
        return {"bytes": 4 * n * d * (1 if fits else case["iters"]) + 4 * n + 8 * d,
                "flops": 4 * n * d * case["iters"]}
    b = f = 0
    if case.get("mf"):
        nnz = 2 * n
        b_epoch = 20 * n + 2 * 4 * RANK * min(2 * n, case["users"] + case["items"])
        f_epoch = 10 * RANK * n
    else:
        per = case["mean"] if case["mean"] else 0.5 * (case["lo"] + case["hi"])
        nnz = int(per * n)
        b_epoch = nnz * (4 if case["val"] == "ones" else 8) + 12 * n + 8 * d
        f_epoch = 4 * nnz + 30 * n
    if op in ("schedule", "step"):
        b += 8 * n + 4 * nnz + 4 * nnz + 8 * n  # bounds, columns; previous writers, levels
    elif op == "mb_step":
        # bounds, columns; union lists and occurrences (about one per entry)
        b += 8 * n + 4 * nnz + 24 * nnz
    if op != "schedule":
        b += b_epoch
        f += f_epoch
    return {"bytes": b, "flops": f}


def tolerance(case):
    # every sum's order is part of the interface (pdb.h states the arithmetic
    # of an example, of a batch and of a dense iteration bit for bit), and the
    # schedule is whole numbers: a correct implementation gives the same bits
    return "exact"


# ---------------------------------------------------------------------------
# the same in 64 bits, one example after another

def _scale(case, z, y):
    lr = float(np.float32(case["lr"]))
    if case["loss"] == "logistic":
        return lr * (1.0 / (1.0 + np.exp(np.minimum(-z, 700.0))) - (y > 0))
    return lr * (z - y)


def _padded(a, size):
    return np.concatenate([a, np.full(size - len(a), -1, np.int64)])


def _levels(bounds, col, d):
    n = len(bounds) - 1
    last = np.zeros(max(d, 1), np.int64)
    level = np.ones(n, np.int64)
    for i in range(n):
        c = col[bounds[i]:bounds[i + 1]]
        if len(c):
            level[i] = l = last[c].max() + 1
            last[c] = l
    perm = np.argsort(level, kind="stable")
    ptr = np.cumsum(np.bincount(level))
    return level, perm, _padded(ptr, n + 1)


def _previous(col):
    order = np.argsort(col, kind="stable")
    prev = np.full(len(col), -1, np.int64)
    same = col[order[1:]] == col[order[:-1]]
    prev[order[1:][same]] = order[:-1][same]
    return prev


def _exact_mf(case, seed):
    user, item, r, U, V = [t.cpu().numpy() for t in _ratings(case, seed)]
    out = ()
    if case["op"] in ("schedule", "step"):
        col = np.stack([user, item.astype(np.int64) + case["users"]], 1).reshape(-1)
        out = _levels(np.arange(0, 2 * case["n"] + 1, 2), col, case["users"] + case["items"])
        out += (_previous(col),)
    if case["op"] in ("epoch", "step"):
        U, V = U.astype(np.float64), V.astype(np.float64)
        lr, reg = float(np.float32(case["lr"])), float(np.float32(case["reg"]))
        for a, b, t in zip(user.tolist(), item.tolist(), r.tolist()):
            u, v = U[a], V[b]
            e = t - u @ v
            du, dv = lr * (e * v - reg * u), lr * (e * u - reg * v)
            u += du
            v += dv
        out += (U, V)
    return out


def _exact_dense(case, seed):
    X, y = _dense(case, seed)
    w = torch.zeros(case["d"], dtype=torch.float64, device=DEV)
    y = y.double()
    lr = float(np.float32(case["lr"]))
    X = X.double()
    for _ in range(case["iters"]):
        z = X @ w
        g = torch.sigmoid(z) - (y > 0).double() if case["loss"] == "logistic" else z - y
        w = w - lr * (g @ X)
    return w.cpu().numpy()


def _exact_batches(case, col, rows, d):
    """Union lists of every batch: entries by (batch, feature, index)."""
    batch = rows // case["batch"]
    order = np.lexsort((col, batch))  # stable: entries of a group stay in order
    cb, bb = col[order], batch[order]
    head = np.ones(len(col), bool)
    head[1:] = (cb[1:] != cb[:-1]) | (bb[1:] != bb[:-1])
    at = np.flatnonzero(head)
    ucol = cb[at].astype(np.int64)
    nb = -(-case["n"] // case["batch"])
    bptr = np.searchsorted(bb[at], np.arange(nb + 1))
    level, perm, ptr = _levels(bptr, ucol, d)
    nnz = len(col)
    return (level, perm, ptr, _padded(_previous(ucol), nnz), bptr, _padded(ucol, nnz),
            _padded(np.append(at, nnz), nnz + 1), order)


def exact(case, seed):
    op = case["op"]
    if op == "dense":
        return _exact_dense(case, seed)
    if case["n"] > 2_000_000 or (case.get("mf") and op != "schedule" and case["n"] > 1_000_000):
        return None
    if case.get("mf"):
        return _exact_mf(case, seed)
    row_ptr, col, val, y = [None if t is None else t.cpu().numpy() for t in _csr(case, seed)]
    n, d = case["n"], case["d"]
    out = ()
    if op in ("schedule", "step"):
        out = _levels(row_ptr, col, d) + (_previous(col),)
        if op == "schedule":
            return out
    y = y.astype(np.float64)
    x = np.ones(len(col)) if val is None else val.astype(np.float64)
    w = np.zeros(d)
    if op in ("mb_epoch", "mb_step"):
        rows = np.repeat(np.arange(n), np.diff(row_ptr))
        if op == "mb_step":
            out = _exact_batches(case, col, rows, d)
        for i in range(0, n, case["batch"]):
            j = min(n, i + case["batch"])
            b, e = row_ptr[i], row_ptr[j]
            c, xv, rr = col[b:e], x[b:e], rows[b:e] - i
            z = np.bincount(rr, w[c] * xv, minlength=j - i)
            np.subtract.at(w, c, _scale(case, z, y[i:j])[rr] * xv)
        return out + (w,)
    rp = row_ptr.tolist()
    delay = case.get("delay", 0)
    late = []  # updates that are made but not yet read
    for i in range(n):
        c, xv = col[rp[i]:rp[i + 1]], x[rp[i]:rp[i + 1]]
        s = _scale(case, w[c] @ xv, y[i])
        late.append((c, s * xv))
        if len(late) > delay:
            c, u = late.pop(0)
            w[c] -= u
    for c, u in late:
        w[c] -= u
    return out + (w,)
