"""GPU: kernels and dispatch branches that serve a range of sizes, at the edges of that range, against the oracle
or a plain fp64 computation of the same quantity."""
import numpy as np
import pytest
import torch

import oracle
import paper_1803_06333_amd as snap

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def zipf_rows(lengths, d, seed, s=1.1):
    """CSR arrays: row i holds lengths[i] distinct columns of popularity rank^-s, unit rows."""
    rng = np.random.default_rng(seed)
    p = np.arange(1, d + 1, dtype=np.float64) ** -s
    p /= p.sum()
    name = rng.permutation(d)                              # every second row: popularity does not follow the column number
    cols, ptr = [], np.zeros(len(lengths) + 1, dtype=np.int64)
    for i, k in enumerate(lengths):
        c = rng.choice(d, size=min(d, 2 * k + 8), p=p)
        c = np.unique(c)[:k] if k else c[:0]
        cols.append(np.sort(name[c] if i % 2 else c))
        ptr[i + 1] = ptr[i] + cols[-1].size
    idx = np.concatenate(cols).astype(np.int32)
    val = (np.abs(rng.standard_normal(idx.size)) + 0.05).astype(np.float32)
    for i in range(len(lengths)):
        v = val[ptr[i]:ptr[i + 1]]
        if v.size:
            v /= np.linalg.norm(v)
    return ptr, idx, val


def row_lengths(kind, n, rng):
    if kind == "to32":
        return rng.integers(1, 33, n)
    if kind == "to64":
        return rng.integers(20, 65, n)
    if kind == "tails64":                                  # a few rows longer than the places of a row, and empty ones
        k = rng.integers(8, 60, n)
        k[::97], k[5::211] = rng.integers(65, 400, k[::97].size), 0
        return k
    k = rng.integers(65, 257, n)                           # "tails256"
    k[::101] = rng.integers(257, 700, k[::101].size)
    return k


@pytest.mark.parametrize("loss", ["hinge", "logistic"])
@pytest.mark.parametrize("kind,n", [("to32", 4096), ("to64", 4103), ("tails64", 5001), ("tails256", 4099)])
@pytest.mark.parametrize("in_flight", [100, 300])          # four and eight rows per wavefront
def test_rows_with_popular_features_keep_the_shared_vector_and_reach_the_optimum(kind, n, loss, in_flight):
    d, lam = 6_000, 60.0 / n
    rng = np.random.default_rng(11)
    ptr, idx, val = zipf_rows(row_lengths(kind, n, rng), d, 12)
    w = rng.standard_normal(d)
    y = np.where([(val[a:b] * w[idx[a:b]]).sum() >= 0 for a, b in zip(ptr, ptr[1:])], 1.0, -1.0).astype(np.float32)
    nnz = int(ptr[-1])
    s = snap.Solver("csr", n, d, ptr, idx, val, y, loss, lam, max_inflight_nnz=in_flight * nnz // n)
    A = np.zeros(d)
    for e in range(40):
        s.epoch(e)
        if e in (0, 1, 5):
            alpha = s.model()[1].astype(np.float64)
            assert alpha.min() >= 0.0 and alpha.max() <= 1.0
            A[:] = 0.0
            np.add.at(A, idx, val.astype(np.float64) * np.repeat(y * alpha, np.diff(ptr)))
            assert np.linalg.norm(s.shared() - A) <= 1e-4 * np.linalg.norm(A)
    o = oracle.Solver(oracle.Matrix("csr", n, d, ptr, idx, val), y, loss, lam)
    for e in range(40):
        o.epoch(e)
    P, D = s.objective(want_dual=True)
    assert P - D >= -1e-6 * abs(P)
    assert abs(D - o.dual()) <= 1e-3 * abs(o.dual()), (D, o.dual())


def one_hot_columns(n, sizes, seed, missing, weighted):
    """CSC arrays of one-hot fields (a share of the rows without a category), group bounds."""
    rng = np.random.default_rng(seed)
    cols, rows = [], []
    bounds = np.concatenate([[0], np.cumsum(sizes)])
    for f, size in enumerate(sizes):
        cat = np.minimum((size * rng.random(n) ** 3).astype(np.int64), size - 1)
        r = np.nonzero(rng.random(n) >= (missing if size else 2.0))[0]
        cols.append(bounds[f] + cat[r])
        rows.append(r)
    cols, rows = np.concatenate(cols), np.concatenate(rows)
    order = np.lexsort((rows, cols))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=bounds[-1]))]).astype(np.int64)
    val = (0.5 + rng.random(rows.size)).astype(np.float32) if weighted else np.ones(rows.size, dtype=np.float32)
    return ptr, rows[order].astype(np.int32), val, bounds.tolist()


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,sizes", [(1, [1]), (7, [3, 1]), (2049, [300, 0, 17, 64]), (5003, [1, 255, 256, 40, 9]), (70_001, [66_000, 30])])
def test_shared_vector_of_a_saved_model_from_the_row_maps(n, sizes, weighted):
    ptr, idx, val, bounds = one_hot_columns(n, sizes, 5, 0.1, weighted)
    d, rng = bounds[-1], np.random.default_rng(6)
    s = snap.Solver("csc", n, d, ptr, idx, val, rng.standard_normal(n).astype(np.float32), "ridge", 1e-2, group_bounds=bounds)
    for scale in (1.0, 1e-3):
        x = (scale * rng.standard_normal(d)).astype(np.float32)
        s.set_model(x)
        want = np.zeros(n)
        np.add.at(want, idx, val.astype(np.float64) * np.repeat(x.astype(np.float64), np.diff(ptr)))
        np.testing.assert_allclose(s.shared(), want, rtol=1.2e-7, atol=1e-12)     # fp64 sums rounded once: half an ulp


@pytest.mark.parametrize("d,n", [(1, 50), (700, 5000), (4096, 3000), (30_011, 9001)])      # around the 4096 table slots
def test_shared_vector_of_a_dual_model_with_popular_features(d, n):
    rng = np.random.default_rng(7)
    ptr, idx, val = zipf_rows(rng.integers(0, min(d, 40) + 1, n), d, 8)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    s = snap.Solver("csr", n, d, ptr, idx, val, y, "hinge", 1e-2)
    alpha = rng.random(n).astype(np.float32)
    s.set_model(alpha)
    want = np.zeros(d)
    np.add.at(want, idx, val.astype(np.float64) * np.repeat((y * alpha).astype(np.float64), np.diff(ptr)))
    np.testing.assert_allclose(s.shared(), want, rtol=1.2e-7, atol=1e-9)


def model_handle(w, loss="ridge"):
    d = w.size
    s = snap.Solver("csc", 4, d, np.arange(d + 1, dtype=np.int64), (np.arange(d) % 4).astype(np.int32), np.ones(d, dtype=np.float32),
                    np.ones(4, dtype=np.float32), loss, 1e-3, auto_groups=False)
    s.set_model(w)
    return s


@pytest.mark.parametrize("offset", [0, 1])                 # rows on 16 bytes, and not
@pytest.mark.parametrize("rows,d", [(1, 1), (3, 255), (65, 256), (64, 1023), (130, 4096), (1000, 129)])
def test_dense_requests_of_every_shape(rows, d, offset):
    rng = np.random.default_rng(rows * d)
    w, X = rng.standard_normal(d).astype(np.float32), rng.standard_normal((rows, d)).astype(np.float32)
    s = model_handle(w)
    want = X.astype(np.float64) @ w.astype(np.float64)
    bound = 1.2e-7 * np.abs(want) + 1e-13 * (np.abs(X) @ np.abs(w).astype(np.float64))      # fp64 sums rounded once
    for layout, flat in (("dense_rowmajor", X), ("dense_colmajor", X.T)):
        buf = torch.empty(rows * d + offset, device=DEV)
        buf[offset:] = torch.from_numpy(np.ascontiguousarray(flat).ravel())
        got = s.predict(layout, rows, None, None, buf[offset:]).cpu().numpy()
        assert (np.abs(got - want) <= bound).all()


@pytest.mark.parametrize("top", [1, 17, 70, 150, 700])     # lanes per row 8, 8, 16 ... 64; rows shorter and longer than a step
def test_sparse_rows_of_every_length_and_a_refused_matrix(top):
    rng = np.random.default_rng(top)
    rows, d = 501, 900
    k = rng.integers(0, top + 1, rows)
    k[-1] = 2 * top
    ptr = np.concatenate([[0], np.cumsum(k)]).astype(np.int64)
    idx, val = rng.integers(0, d, ptr[-1]).astype(np.int32), rng.standard_normal(ptr[-1]).astype(np.float32)
    w = rng.standard_normal(d).astype(np.float32)
    s = model_handle(w)
    want = np.zeros(rows)
    np.add.at(want, np.repeat(np.arange(rows), k), val.astype(np.float64) * w[idx])
    for _ in range(2):
        np.testing.assert_allclose(s.predict("csr", rows, ptr, idx, val), want, rtol=1.2e-7, atol=1e-9)
        bad = idx.copy()
        bad[-1] = d
        with pytest.raises(snap.SnapError):
            s.predict("csr", rows, ptr, bad, val)          # refused, and the next call is not


@pytest.mark.parametrize("loss", ["ridge", "logistic"])
@pytest.mark.parametrize("n,d", [(5, 1), (255, 9), (1024, 8), (16_384, 3), (16_388, 17), (33_001, 40), (20_000, 4200)])
def test_duality_gap_of_dense_data_of_every_shape(n, d, loss):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + d)
    A = torch.randn(d, n, generator=g, device=DEV)
    y = torch.randn(n, generator=g, device=DEV)
    if loss == "logistic":
        y = torch.where(y >= 0, 1.0, -1.0)
    w = torch.randn(d, generator=g, device=DEV) * 0.1 / d ** 0.5
    lam = 1e-2
    s = snap.Solver("dense_colmajor", n, d, None, None, A.view(-1), y, loss, lam)
    s.set_model(w.cpu().numpy())
    v = torch.from_numpy(s.shared()).to(DEV).double()
    u = v - y.double() if loss == "ridge" else -y.double() * torch.sigmoid(-y.double() * v)
    grad = torch.stack([torch.dot(A[j].double(), u) for j in range(d)]) / n + lam * w.double()
    want = float(grad.square().sum()) / (2 * lam)
    assert abs(s.duality_gap() - want) <= 1e-9 * want      # fp64 throughout: the order of the sums


@pytest.mark.parametrize("slots", [256, 50, 1])           # buckets that hold everything, some of it, almost nothing
@pytest.mark.parametrize("m", [1, 2, 127, 128, 129, 1000, 4097, 60_013, 262_145])
def test_epoch_order_by_buckets(m, slots, monkeypatch):
    if slots < 256:
        monkeypatch.setenv("SNAP_SORT_SLOTS", str(slots))
        m = min(m, 4097 if slots == 1 else 20_011)         # (the list of a full bucket is searched linearly)
    n = 8
    s = snap.Solver("csc", n, m, np.arange(m + 1, dtype=np.int64), (np.arange(m) % n).astype(np.int32), np.ones(m, dtype=np.float32),
                    np.ones(n, dtype=np.float32), "ridge", 1.0, auto_groups=False)
    for seed in (0, 1, 12345, 2 ** 63 + 5):
        s.epoch(seed)
        assert np.array_equal(s.perm(), oracle.permutation(seed, m))


@pytest.mark.parametrize("host_keys", [False, True])
def test_epoch_order_of_two_classes_and_of_more_coordinates_than_buckets_take(host_keys, monkeypatch):
    monkeypatch.setenv("SNAP_SMALL_MAX", "2")
    m, n = 5_003, 64
    k = np.where(np.arange(m) % 3 == 0, 3, 1)
    ptr = np.concatenate([[0], np.cumsum(k)]).astype(np.int64)
    idx = np.concatenate([np.arange(q) * 7 for q in k]).astype(np.int32)
    s = snap.Solver("csc", n, m, ptr, idx, np.ones(idx.size, dtype=np.float32), np.ones(n, dtype=np.float32), "ridge", 1.0,
                    auto_groups=False, host_keys=host_keys)
    for seed in (3, 4):
        s.epoch(seed)
        p = oracle.permutation(seed, m)
        assert np.array_equal(s.perm(), np.concatenate([p[k[p] > 2], p[k[p] <= 2]]))
    monkeypatch.delenv("SNAP_SMALL_MAX")
    m = (1 << 21) + 1
    s = snap.Solver("csc", 4, m, np.arange(m + 1, dtype=np.int64), (np.arange(m) % 4).astype(np.int32), np.ones(m, dtype=np.float32),
                    np.ones(4, dtype=np.float32), "ridge", 1.0, auto_groups=False, host_keys=host_keys)
    s.epoch(9)
    assert np.array_equal(s.perm(), oracle.permutation(9, m))


@pytest.mark.parametrize("loss", ["ridge", "logistic", "elastic"])
@pytest.mark.parametrize("n,d,top", [(300, 40, 32), (300, 40, 64), (900, 257, 250), (900, 100, 257), (20_000, 64, 1024), (4_000, 30, 1025), (20_480, 33, 90), (20_481, 33, 90)])
@pytest.mark.parametrize("in_flight", [1, 12])             # coordinates; one: exactly the sequential epoch
def test_primal_epoch_with_the_shared_vector_in_lds(n, d, top, loss, in_flight):
    rng = np.random.default_rng(n + top)
    k = rng.integers(0, min(n, top) + 1, d)
    k[0], k[-1] = min(n, top), 0
    ptr = np.concatenate([[0], np.cumsum(k)]).astype(np.int64)
    idx = np.concatenate([np.sort(rng.choice(n, q, replace=False)) for q in k]).astype(np.int32)
    val = rng.standard_normal(idx.size).astype(np.float32)
    name = "ridge" if loss == "elastic" else loss
    y = rng.standard_normal(n).astype(np.float32)
    if loss == "logistic":
        y = np.where(y >= 0, 1.0, -1.0).astype(np.float32)
    lam1 = 1e-3 if loss == "elastic" else 0.0
    s = snap.Solver("csc", n, d, ptr, idx, val, y, name, 1e-2, lam1=lam1, auto_groups=False, adaptive=False,
                    max_inflight_nnz=1 if in_flight == 1 else int(in_flight * max(1.0, idx.size / d)))
    o = oracle.Solver(oracle.Matrix("csc", n, d, ptr, idx, val), y, name, 1e-2, lam1=lam1)
    for e in range(12):
        s.epoch(e)
        o.epoch(e)
        x = s.model()[1].astype(np.float64)
        want = np.zeros(n)
        np.add.at(want, idx, val.astype(np.float64) * np.repeat(x, k))
        assert np.linalg.norm(s.shared() - want) <= 1e-5 * max(np.linalg.norm(want), 1e-6)
        if in_flight == 1:                                 # fp32 steps against the fp64 oracle's, the same order
            assert np.linalg.norm(x - o.x) <= 1e-4 * max(np.linalg.norm(o.x), 1e-6)
    P, Po = s.objective(), o.primal()
    assert abs(P - Po) <= 1e-4 * abs(Po)


@pytest.mark.parametrize("loss", ["hinge", "logistic"])
@pytest.mark.parametrize("top,d", [(1, 40), (32, 700), (33, 700), (64, 5_000), (65, 20_480), (256, 20_480), (300, 3_000), (40, 20_481)])
@pytest.mark.parametrize("in_flight", [1, 20, 90])
def test_dual_epoch_with_the_shared_vector_in_lds(top, d, loss, in_flight):
    n = 403
    lam = 60.0 / n
    rng = np.random.default_rng(top)
    k = rng.integers(0, top + 1, n)
    k[3] = top
    ptr, idx, val = zipf_rows(k, d, 14)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    s = snap.Solver("csr", n, d, ptr, idx, val, y, loss, lam, max_inflight_nnz=1 if in_flight == 1 else int(in_flight * max(1.0, idx.size / n)))
    o = oracle.Solver(oracle.Matrix("csr", n, d, ptr, idx, val), y, loss, lam)
    for e in range(30):
        s.epoch(e)
        o.epoch(e)
        if e < 3:
            alpha = s.model()[1].astype(np.float64)
            want = np.zeros(d)
            np.add.at(want, idx, val.astype(np.float64) * np.repeat(y * alpha, np.diff(ptr)))
            assert np.linalg.norm(s.shared() - want) <= 1e-5 * np.linalg.norm(want)
            if in_flight == 1:
                assert np.linalg.norm(alpha - o.x) <= 1e-4 * np.linalg.norm(o.x)
    assert abs(s.objective(want_dual=True)[1] - o.dual()) <= 1e-4 * abs(o.dual())


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n", [2041, 2049, 40_009, 524_285, 524_293, 1_048_583])      # workgroups of 256, 512 and 1024 threads, their edges
def test_group_sweeps_of_every_launch_shape(n, weighted):
    ptr, idx, val, bounds = one_hot_columns(n, [64, 300, 5], 9, 0.05, weighted)
    d, rng = bounds[-1], np.random.default_rng(10)
    y = np.where(rng.random(n) < 0.3, 1.0, -1.0).astype(np.float32)
    s = snap.Solver("csc", n, d, ptr, idx, val, y, "logistic", 1e-3, group_bounds=bounds)
    o = oracle.Solver(oracle.Matrix("csc", n, d, ptr, idx, val), y, "logistic", 1e-3, chunk_bounds=bounds, shuffle_chunks=True)
    for e in range(3):
        s.epoch(e)
        o.epoch(e)
    x = s.model()[1]
    assert np.linalg.norm(x - o.x) <= 2e-5 * np.linalg.norm(o.x)
    P, D = s.objective(want_dual=True)
    assert abs(P - o.primal()) <= 1e-5 * o.primal() and P >= D
