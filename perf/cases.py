"""The work that users of the solver have it do, as a list of cases: training passes of every engine (the
asynchronous epoch in the primal and in the dual form, the exact group sweeps of one-hot data resident and
streamed from pinned host memory, the exact tile sweeps of dense ridge regression), resuming from a saved model,
and decision values for new rows.

A training case is what a program does between two looks at the model: some epochs, the objective with its dual
value (the stopping test), and the weights.  The asynchronous cases start each time from the zero model (a fit), because
the work of an epoch depends on how far the model is; an epoch of the sweeps costs the same at every model, so
these carry on with the training they have begun.
"""
import math

import numpy as np
import torch

import paper_1803_06333_amd as snap

NUMERIC_FIELDS, CATEGORICAL_FIELDS, BINS = 13, 26, 64      # the fields of a click-log row
TILE = 128                                                 # columns per tile of the dense sweeps (include/snap.h)
DEVICE = "cuda"


def listed():
    return [
        # the smallest training call: a text-classification sized problem, where latency and launches count
        dict(name="fit_logistic_small", kind="fit", loss="logistic", n=10_000, d=1_000, k=20, lam=1e-3, lam1=0.0, epochs=5),
        # elastic-net regression on sparse features of odd sizes
        dict(name="fit_elastic_net", kind="fit", loss="ridge", n=300_007, d=20_011, k=31, lam=1e-3, lam1=1e-5, epochs=4),
        # SVM on a corpus with popular words, examples as coordinates: 50 M nonzeros
        dict(name="fit_svm_large", kind="fit", loss="hinge", n=1_000_000, d=100_000, k=50, lam=1e-4, lam1=0.0, epochs=5),
        # logistic regression in the dual form on a corpus of ordinary size
        dict(name="fit_dual_logistic", kind="fit", loss="dual_logistic", n=60_013, d=5_003, k=23, lam=1e-3, lam1=0.0, epochs=10),
        # dense ridge regression, large and of a small odd size
        dict(name="dense_ridge_large", kind="dense", n=400_000, d=2_000, lam=1e-4, epochs=3),
        dict(name="dense_ridge_odd", kind="dense", n=30_011, d=333, lam=1e-4, epochs=5),
        # click-log regression (39 one-hot fields per row): a day's log, ...
        dict(name="onehot_large", kind="onehot", loss="logistic", n=45_840_617, d=1_000_000, lam=1e-6, values=False, resume=False,
             streamed=False, epochs=2),
        # ... a sample of it, resumed from a saved model, ...
        dict(name="onehot_resume", kind="onehot", loss="logistic", n=1_000_003, d=100_000, lam=1e-5, values=False, resume=True,
             streamed=False, epochs=5),
        # ... a small regression with weighted indicators, ...
        dict(name="onehot_ridge_small", kind="onehot", loss="ridge", n=40_009, d=4_001, lam=1e-3, values=True, resume=False,
             streamed=False, epochs=5),
        # ... and data that stay in host memory
        dict(name="onehot_streamed", kind="onehot", loss="logistic", n=3_000_017, d=200_000, lam=1e-6, values=False, resume=False,
             streamed=True, epochs=3),
        # scoring: a batch of click-log rows, and a small dense request
        dict(name="predict_csr", kind="predict", layout="csr", rows=1_000_000, d=1_000_000, k=39),
        dict(name="predict_dense_small", kind="predict", layout="dense_rowmajor", rows=1_023, d=2_000, k=2_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fit", "fit", "dense", "onehot", "onehot", "predict"])
    if kind == "fit":
        loss = rng.choice(["logistic", "ridge", "hinge", "dual_logistic"])
        k = rng.randint(10, 50)
        if loss in ("logistic", "ridge"):
            n = _log(rng, 10_000, 300_000)
            d = max(k + 1, min(n // 8, _log(rng, 500, 20_000)))
            return dict(kind="fit", loss=loss, n=n, d=d, k=k, lam=1e-3, lam1=rng.choice([0.0, 1e-5]), epochs=rng.randint(3, 5))
        n = _log(rng, 20_000, 500_000)
        d = max(2_000, min(n // 10, _log(rng, 2_000, 50_000)))
        return dict(kind="fit", loss=loss, n=n, d=d, k=k, lam=60.0 / n, lam1=0.0, epochs=6 if loss == "hinge" else 10)
    if kind == "dense":
        n = _log(rng, 5_000, 400_000)
        return dict(kind="dense", n=n, d=min(_log(rng, 40, 2_000), 800_000_000 // n), lam=1e-4, epochs=rng.randint(2, 5))
    if kind == "onehot":
        n = _log(rng, 30_000, 10_000_000)
        d = max(2_000, min(1_000_000, n // rng.randint(8, 60)))
        streamed = rng.random() < 0.25
        loss = rng.choice(["logistic", "logistic", "ridge"])
        return dict(kind="onehot", loss=loss, n=n, d=d, lam=max(1e-6, 0.5 / n), values=not streamed and rng.random() < 0.3,
                    resume=not streamed and rng.random() < 0.3, streamed=streamed, epochs=rng.randint(2, 5))
    layout = rng.choice(["csr", "csc", "dense_rowmajor", "dense_colmajor"])
    if layout.startswith("dense"):
        rows, d = _log(rng, 64, 200_000), _log(rng, 100, 4_000)
        return dict(kind="predict", layout=layout, rows=rows, d=d, k=d)
    d = _log(rng, 10_000, 1_000_000)
    return dict(kind="predict", layout=layout, rows=_log(rng, 500, 1_000_000), d=d, k=rng.randint(8, 120))


# ---- inputs ---------------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _zipf_cdf(size, s):
    p = torch.arange(1, size + 1, dtype=torch.float64, device=DEVICE) ** (-s)
    return torch.cumsum(p / p.sum(), 0)


def _bin_cdf():
    """64 bins of a count with a bell-shaped logarithm."""
    z = (torch.arange(BINS, dtype=torch.float64, device=DEVICE) - 14.0) / 9.0
    p = torch.exp(-0.5 * z * z)
    return torch.cumsum(p / p.sum(), 0)


def _sample(cdf, count, g):
    u = torch.rand(count, generator=g, device=DEVICE, dtype=torch.float64)
    return torch.searchsorted(cdf, u).clamp_(max=cdf.numel() - 1)


def _labels(margin, g):
    """+1 for about a quarter of the rows, more likely where the margin is large."""
    p = torch.sigmoid(margin - margin.mean() - 1.2)
    return torch.where(torch.rand(margin.numel(), generator=g, device=DEVICE, dtype=torch.float64) < p, 1.0, -1.0).to(torch.float32)


def _sorted_rows(cat, size):
    """Rows by category (ascending inside a category), and the number of rows of every category."""
    by_cat, rows = torch.sort(cat.to(torch.int32), stable=True)
    first = torch.searchsorted(by_cat, torch.arange(size + 1, dtype=torch.int32, device=DEVICE))
    return rows.to(torch.int32), first[1:] - first[:-1]


def _sparse(case, seed):
    """Rows of about k distinct columns: uniform columns (primal) or Zipf(1.1) popularity (dual); CSR triple, values, labels."""
    n, d, k, g = case["n"], case["d"], case["k"], _generator(seed)
    dual = case["loss"] in ("hinge", "dual_logistic")
    if dual:
        cols = _sample(_zipf_cdf(d, 1.1), n * k, g).view(n, k)
    else:
        cols = torch.randint(0, d, (n, k), generator=g, device=DEVICE)
    cols = torch.sort(cols, dim=1).values
    first = torch.ones_like(cols, dtype=torch.bool)
    first[:, 1:] = cols[:, 1:] != cols[:, :-1]             # a column that was drawn twice counts once: ragged rows
    val = torch.ones(n, k, device=DEVICE, dtype=torch.float64)
    if dual or case["loss"] == "ridge":
        val = torch.randn(n, k, generator=g, device=DEVICE, dtype=torch.float64).abs_() + 0.05
    val = torch.where(first, val, torch.zeros_like(val))
    if dual:
        val = val / val.norm(dim=1, keepdim=True)
    w = torch.randn(d, generator=g, device=DEVICE, dtype=torch.float64)
    margin = (val * w[cols]).sum(1)
    noise = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64)
    if case["loss"] == "ridge":
        y = (margin / math.sqrt(k) + 0.1 * noise).to(torch.float32)
    else:
        y = torch.where(margin + 0.1 * margin.std() * noise >= 0, 1.0, -1.0).to(torch.float32)
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    ptr[1:] = torch.cumsum(first.sum(1), 0)
    return ptr, cols[first], val[first].to(torch.float32), y


def _dense(case, seed):
    """A[j] = column j (unit rows), labels of a planted model."""
    n, d, g = case["n"], case["d"], _generator(seed)
    A = torch.randn(d, n, generator=g, device=DEVICE, dtype=torch.float32)
    A /= A.norm(dim=0, keepdim=True)
    w = torch.randn(d, generator=g, device=DEVICE, dtype=torch.float32) / math.sqrt(d)
    y = w @ A + 0.01 * torch.randn(n, generator=g, device=DEVICE, dtype=torch.float32)
    return A, y


def _fields(d):
    """Column range of every field: small numeric ones first, the categorical ones share the rest."""
    rest = d - NUMERIC_FIELDS * BINS
    sizes = [BINS] * NUMERIC_FIELDS + [rest // CATEGORICAL_FIELDS + (f < rest % CATEGORICAL_FIELDS) for f in range(CATEGORICAL_FIELDS)]
    return sizes, np.concatenate([[0], np.cumsum(sizes)]).tolist()


def _categories(case, seed):
    """Yields per field: its categories, one per row, its values (None: all 1) and the planted weights of its columns."""
    g = _generator(seed)
    bins, cdfs = _bin_cdf(), {}
    for size in _fields(case["d"])[0]:
        cdf = bins if size == BINS else cdfs.setdefault(size, _zipf_cdf(size, 1.2))
        cat = _sample(cdf, case["n"], g)
        val = 0.5 + torch.rand(case["n"], generator=g, device=DEVICE) if case["values"] else None
        yield cat, val, torch.randn(size, generator=g, device=DEVICE, dtype=torch.float64) / math.sqrt(39.0)


def _onehot_labels(case, seed, margin):
    g = _generator(seed + 77_777)
    if case["loss"] == "ridge":
        return (margin + 0.3 * torch.randn(margin.numel(), generator=g, device=DEVICE, dtype=torch.float64)).to(torch.float32)
    return _labels(margin, g)


def _saved_model(case, seed):
    g = _generator(seed + 55_555)
    return (0.1 * torch.randn(case["d"], generator=g, device=DEVICE)).cpu().numpy()


def _onehot(case, seed):
    n, d = case["n"], case["d"]
    sizes, bounds = _fields(d)
    idx = torch.empty(39 * n, dtype=torch.int32, device=DEVICE)
    val = torch.empty(39 * n, dtype=torch.float32, device=DEVICE) if case["values"] else None
    ptr = torch.zeros(d + 1, dtype=torch.int64, device=DEVICE)
    margin = torch.zeros(n, dtype=torch.float64, device=DEVICE)
    for f, (cat, a, w) in enumerate(_categories(case, seed)):
        rows, counts = _sorted_rows(cat, sizes[f])
        idx[f * n:(f + 1) * n] = rows
        if a is not None:
            val[f * n:(f + 1) * n] = a[rows.long()]
        margin += w[cat] if a is None else w[cat] * a
        ptr[bounds[f] + 1:bounds[f + 1] + 1] = counts
    return torch.cumsum(ptr, 0), idx, val, _onehot_labels(case, seed, margin), bounds


def _request(case, seed):
    """New rows for a model of d weights: the arrays of the layout, and the matrix's nonzeros by row for exact()."""
    rows, d, k, g = case["rows"], case["d"], case["k"], _generator(seed)
    w = torch.randn(d, generator=g, device=DEVICE)
    if case["layout"].startswith("dense"):
        X = torch.randn(rows, d, generator=g, device=DEVICE)
        flat = X if case["layout"] == "dense_rowmajor" else X.t()
        return w, None, None, flat.contiguous().view(-1), X
    length = torch.randint(max(1, k // 2), k + k // 2 + 1, (rows,), generator=g, device=DEVICE)
    ptr = torch.zeros(rows + 1, dtype=torch.int64, device=DEVICE)
    ptr[1:] = torch.cumsum(length, 0)
    nnz = int(ptr[-1])
    cols = _sample(_zipf_cdf(d, 1.1), nnz, g)              # (a column may come twice in a row: its entries add up)
    val = torch.randn(nnz, generator=g, device=DEVICE)
    row = torch.repeat_interleave(torch.arange(rows, device=DEVICE), length)
    if case["layout"] == "csr":
        return w, ptr, cols.to(torch.int32), val, (row, cols, val)
    order, counts = _sorted_rows(cols, d)
    cptr = torch.zeros(d + 1, dtype=torch.int64, device=DEVICE)
    cptr[1:] = torch.cumsum(counts, 0)
    order = order.long()
    return w, cptr, row[order].to(torch.int32), val[order], (row, cols, val)


def _pinned(t):
    out = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    out.copy_(t)
    return out


# ---- the calls ------------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "predict":
        w, ptr, idx, val, _ = _request(case, seed)
        # a handle that holds the model: a few training rows are enough
        d = case["d"]
        tptr = torch.arange(d + 1, dtype=torch.int64, device=DEVICE)
        tidx = (torch.arange(d, device=DEVICE) % 64).to(torch.int32)
        y = torch.ones(64, device=DEVICE)
        torch.cuda.synchronize()
        s = snap.Solver("csc", 64, d, tptr, tidx, torch.ones(d, device=DEVICE), y, "ridge", 1e-3, auto_groups=False)
        s.set_model(w.cpu().numpy())
        return dict(case=case, solver=s, ptr=ptr, idx=idx, val=val)
    if kind == "fit":
        ptr, cols, val, y = _sparse(case, seed)
        n, d = case["n"], case["d"]
        dual = case["loss"] in ("hinge", "dual_logistic")
        if dual:
            layout, idx, start = "csr", cols.to(torch.int32), np.full(n, 0.0 if case["loss"] == "hinge" else 0.5, dtype=np.float32)
        else:
            row = torch.repeat_interleave(torch.arange(n, device=DEVICE), ptr[1:] - ptr[:-1])
            order, counts = _sorted_rows(cols, d)
            order = order.long()
            ptr = torch.zeros(d + 1, dtype=torch.int64, device=DEVICE)
            ptr[1:] = torch.cumsum(counts, 0)
            layout, idx, val, start = "csc", row[order].to(torch.int32), val[order], np.zeros(d, dtype=np.float32)
        torch.cuda.synchronize()
        s = snap.Solver(layout, n, d, ptr, idx, val, y, "logistic" if case["loss"] == "dual_logistic" else case["loss"], case["lam"],
                        lam1=case["lam1"], auto_groups=None if dual else False)
        return dict(case=case, solver=s, start=start, epoch=0)
    if kind == "dense":
        A, y = _dense(case, seed)
        torch.cuda.synchronize()
        s = snap.Solver("dense_colmajor", case["n"], case["d"], None, None, A.view(-1), y, "ridge", case["lam"])
        return dict(case=case, solver=s, start=None, epoch=0)
    ptr, idx, val, y, bounds = _onehot(case, seed)
    options = dict(group_bounds=bounds)
    if case["streamed"]:
        nnz = int(idx.numel())
        options.update(device_budget_bytes=2 * nnz, chunk_bytes=max(1 << 20, 2 * nnz))
        ptr, idx, y = _pinned(ptr), _pinned(idx), _pinned(y)
    torch.cuda.synchronize()
    s = snap.Solver("csc", case["n"], case["d"], ptr, idx, val, y, case["loss"], case["lam"], **options)
    return dict(case=case, solver=s, start=_saved_model(case, seed) if case["resume"] else None, epoch=0)


def run(state):
    case, s = state["case"], state["solver"]
    if case["kind"] == "predict":
        return s.predict(case["layout"], case["rows"], state["ptr"], state["idx"], state["val"])
    first = state["epoch"]
    if state["start"] is not None:
        s.set_model(state["start"])
        first = 0
    for e in range(first, first + case["epochs"]):
        s.epoch(e)
    state["epoch"] = first + case["epochs"]
    primal, dual = s.objective(want_dual=True)
    return {"w": s.model()[0], "primal": primal, "dual": dual}


def work(case):
    """Per epoch the matrix once in the form the engine needs it (index and value per nonzero; dense: the value; one-hot:
    two bytes of category per field and row, and the value where it is not 1), the shared vector and the labels; the
    objective with its dual value reads the matrix once more.  Scoring: the matrix and the weights once."""
    kind = case["kind"]
    if kind == "predict":
        rows, d, k = case["rows"], case["d"], case["k"]
        matrix = 4 * rows * d if case["layout"].startswith("dense") else 8 * rows * k + 8 * rows
        return {"bytes": matrix + 4 * d + 4 * rows, "flops": 2 * rows * k}
    n, d = case["n"], case["d"]
    passes = case["epochs"] + 1
    if kind == "dense":
        return {"bytes": passes * (4 * n * d + 12 * n + 8 * d), "flops": passes * 4 * n * d}
    if kind == "fit":
        nnz = n * case["k"]
        return {"bytes": passes * (8 * nnz + 12 * (n + d)), "flops": passes * nnz * (4 if case["loss"] in ("ridge", "hinge") else 20)}
    per = 39 * n * (6 if case["values"] else 2) + 12 * n + 12 * d
    return {"bytes": passes * per, "flops": passes * 39 * n * (4 if case["loss"] == "ridge" else 20)}


def tolerance(case):
    if case["kind"] == "fit":
        # the asynchronous engine: which updates a step sees differs from run to run (measured, weights of two runs
        # on the same inputs: 4e-3 for the dual forms, 5e-4 logistic, 7e-5 ridge)
        return {"logistic": {"rel": 2e-3}, "ridge": {"rel": 3e-4}}.get(case["loss"], {"rel": 1.6e-2, "max": 0.5})
    if case["kind"] == "predict":
        return {"rel": 1e-7, "max": 3e-7}                  # fp64 sums rounded once (against exact(): 2.5e-8, 6e-8)
    if case["kind"] == "dense" or case["loss"] == "ridge":
        return {"rel": 1e-6}                               # (against exact(): 1.7e-7 ... 4e-7)
    return {"rel": 6e-6}                                   # (against exact(): 1.6e-6)


# ---- the results in 64 bits -------------------------------------------------------------------------------------
_M = (1 << 64) - 1


def _mix(z):
    z = (z + 0x9E3779B97F4A7C15) & _M
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M
    return z ^ (z >> 31)


def _order(seed, chunk, count):
    """The permutation of Section 3.2: indices sorted by their 32-bit xorshift keys (chunk: the id that enters the key)."""
    base = _mix(seed ^ _mix((chunk + 0x632BE59BD9B4E019) & _M))
    keys = []
    for c in range(count):
        z = _mix((base + c * 0x9E3779B97F4A7C15) & _M)
        x = (z ^ (z >> 32)) & 0xFFFFFFFF or 0x6C078965
        for _ in range(4):
            x ^= (x << 13) & 0xFFFFFFFF
            x ^= x >> 17
            x ^= (x << 5) & 0xFFFFFFFF
        keys.append((x, c))
    return [c for _, c in sorted(keys)]


_BLOCKS = 0xFFFFFFFF                                       # chunk id of the order of the fields and of the tiles


def _exact_dense(case, seed):
    A, y = _dense(case, seed)
    n, d, lam = case["n"], case["d"], case["lam"]
    y = y.double()
    r = -y                                                 # v - y at the zero model
    x = torch.zeros(d, dtype=torch.float64, device=DEVICE)
    norms = torch.stack([A[j].double().square().sum() for j in range(d)]) / n
    for e in range(case["epochs"]):
        for t in _order(e, _BLOCKS, (d + TILE - 1) // TILE):
            for c in _order(e, t, min(TILE, d - t * TILE)):
                j = t * TILE + c
                a = A[j].double()
                step = -(torch.dot(a, r) / n + lam * x[j]) / (norms[j] + lam)
                x[j] += step
                r += step * a
    grad = torch.stack([torch.dot(A[j].double(), r) for j in range(d)]) / n + lam * x
    primal = 0.5 * float(r.square().mean()) + 0.5 * lam * float(x.square().sum())
    return {"w": x.cpu().numpy(), "primal": primal, "dual": primal - float(grad.square().sum()) / (2 * lam)}


def _exact_onehot(case, seed):
    n, d, lam = case["n"], case["d"], case["lam"]
    sizes, bounds = _fields(d)
    fields, margin = [], torch.zeros(n, dtype=torch.float64, device=DEVICE)
    for f, (cat, a, w) in enumerate(_categories(case, seed)):
        margin += w[cat] if a is None else w[cat] * a
        rows, counts = _sorted_rows(cat, sizes[f])
        ends = torch.zeros(sizes[f] + 1, dtype=torch.int64, device=DEVICE)
        ends[1:] = torch.cumsum(counts, 0)
        fields.append((cat.to(torch.int32), a, rows, ends))
    y = _onehot_labels(case, seed, margin).double()
    del margin
    start = torch.from_numpy(_saved_model(case, seed)).to(DEVICE).double() if case["resume"] else torch.zeros(d, dtype=torch.float64, device=DEVICE)
    x = [start[bounds[f]:bounds[f + 1]].clone() for f in range(39)]

    def spread(f, delta):                                  # A_f delta
        t = delta[fields[f][0].long()]
        return t if fields[f][1] is None else t * fields[f][1].double()

    def gather(f, u, power=1):                             # sum of a^power u per column
        a = fields[f][1]
        u = u if a is None else u * a.double() ** power
        total = torch.zeros(n + 1, dtype=torch.float64, device=DEVICE)
        torch.cumsum(u[fields[f][2].long()], 0, out=total[1:])
        total = total[fields[f][3]]
        return total[1:] - total[:-1]

    def slope(v):
        return v - y if case["loss"] == "ridge" else -y * torch.sigmoid(-y * v)

    def bend(v):
        if case["loss"] == "ridge":
            return torch.ones_like(v)
        p = torch.sigmoid(-y * v)
        return p * (1 - p)

    v = torch.zeros(n, dtype=torch.float64, device=DEVICE)
    for f in range(39):
        v += spread(f, x[f])
    for e in range(case["epochs"]):
        for f in _order(e, _BLOCKS, 39):
            g, h = gather(f, slope(v)) / n, gather(f, bend(v), 2) / n
            step = -(g + lam * x[f]) / (h + lam)
            x[f] += step
            v += spread(f, step)
    u = slope(v)
    gap = sum(float((gather(f, u) / n + lam * x[f]).square().sum()) for f in range(39)) / (2 * lam)
    w = torch.cat(x)
    loss = 0.5 * (v - y).square() if case["loss"] == "ridge" else torch.nn.functional.softplus(-y * v)
    primal = float(loss.mean()) + 0.5 * lam * float(w.square().sum())
    return {"w": w.cpu().numpy(), "primal": primal, "dual": primal - gap}


def exact(case, seed):
    if case["kind"] == "predict":
        w, _, _, _, X = _request(case, seed)
        if case["layout"].startswith("dense"):
            return torch.cat([X[i:i + 8192].double() @ w.double() for i in range(0, case["rows"], 8192)])
        row, cols, val = X
        return torch.zeros(case["rows"], dtype=torch.float64, device=DEVICE).index_add_(0, row, val.double() * w.double()[cols])
    if case["kind"] == "dense":
        return _exact_dense(case, seed)
    if case["kind"] == "onehot":
        return _exact_onehot(case, seed)
    return None                                            # asynchronous epochs: which updates a step sees is not determined
