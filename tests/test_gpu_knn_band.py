"""The exact kNN of data whose nearest neighbours one product cannot tell
apart: tight clusters far from each other, many equal distances, duplicates.
Their answers come from the exact distances of all candidates that may be
among them, and of every candidate where those are too many."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ivhd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as m
    return m


def _data(kind, M, N):
    rng = np.random.default_rng(M + N)
    centres = 4 * rng.normal(size=(20, N))[rng.integers(0, 20, M)]
    if kind == "tight":         # distances 1/60 of the offsets
        x = 0.05 * rng.normal(size=(M, N)) + centres
    elif kind == "tighter":     # 1/3000: every point of the cluster may be the nearest
        x = 1e-3 * rng.normal(size=(M, N)) + centres
    elif kind == "onehot":
        x = np.zeros((M, N))
        for b in range(4):
            x[np.arange(M), b * (N // 4) + rng.integers(0, N // 4, M)] = 1
    elif kind == "binary":      # standardised: 64 different rows, in no power of two
        x = np.zeros((M, N))
        x[:, :6] = (rng.integers(0, 2, size=(M, 6)) - 0.3) / 0.4583 * np.linspace(0.5, 1.7, 6)
    elif kind == "two":         # half of the rows equal, the others too
        x = np.where(rng.random((M, 1)) < 0.5, 0.1, 0.7) * np.ones((1, N))
    return x.astype(np.float32)


# 3,000 rows are "few"; 8,300 x 260 has a pilot; of 40,000 equal rows a query keeps no list of hits
@pytest.mark.parametrize("kind,M,N,k", [
    ("tight", 3000, 20, 5), ("tight", 8300, 24, 12), ("tight", 8300, 260, 2), ("tight", 20000, 33, 28),
    ("tighter", 3000, 20, 5), ("tighter", 8300, 24, 12), ("tighter", 8300, 260, 2), ("onehot", 3000, 40, 3),
    ("onehot", 9000, 40, 28), ("binary", 3000, 8, 28), ("binary", 30000, 100, 4), ("two", 3000, 5, 4),
    ("two", 40000, 5, 4), ("two", 40000, 36, 28)])
def test_against_every_candidate(ivhd, kind, M, N, k):
    X = _data(kind, M, N)
    rows = np.random.default_rng(1).choice(M, 120, replace=False)
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()[rows]
    want = oracle.knn(X, k, queries=rows)
    if kind in ("onehot", "binary", "two"):   # equal rows or integer distances: FP32 has the same ties
        pure = kind != "binary"
        for g, w, q in zip(got, want, rows):
            dw = ((X[w].astype(np.float64) - X[q]) ** 2).sum(1)
            assert np.array_equal(g, w) if pure or dw.max() == 0 else set(g[dw == 0]) == set(w[dw == 0])
        return
    tol = N * 2.0 ** -23   # FP32 sums of N squares in order, both roundings of each term
    for q, g, w in zip(rows, got, want):
        assert len(set(g.tolist())) == len(g) and q not in g and g.min() >= 0
        if not np.array_equal(g, w):
            dg = ((X[g].astype(np.float64) - X[q]) ** 2).sum(1)
            dw = ((X[w].astype(np.float64) - X[q]) ** 2).sum(1)
            np.testing.assert_allclose(dg, dw, rtol=tol, atol=0)


@pytest.mark.parametrize("Q,self_rows", [(1, False), (300, True), (5000, True)])
def test_queries_and_distances(ivhd, Q, self_rows):
    X = _data("tight", 9000, 40)
    rows = np.random.default_rng(Q).integers(0, 9000, Q)
    dX = torch.from_numpy(X).cuda()
    own = torch.from_numpy(np.where(np.arange(Q) % 3 == 0, -1, rows).astype(np.int32)).cuda() if self_rows else None
    idx, dist = ivhd.ivhd_knn_query(dX, dX[torch.from_numpy(rows).cuda()].contiguous(), 3, self_idx=own, with_dist=True)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    for i in range(0, Q, max(1, Q // 100)):
        d = ((X.astype(np.float64) - X[rows[i]]) ** 2).sum(1)
        if self_rows and i % 3:
            assert rows[i] not in idx[i]
            d[rows[i]] = np.inf
        else:
            assert idx[i, 0] == rows[i] and dist[i, 0] == 0
        np.testing.assert_allclose(dist[i], np.sort(d)[:3], rtol=40 * 2.0 ** -23)


@pytest.mark.parametrize("kind", ["tight", "two"])
def test_time_does_not_follow_the_data(ivhd, kind):
    rng = np.random.default_rng(3)

    def best(X):
        X = torch.from_numpy(X.astype(np.float32)).cuda()

        def once():
            torch.cuda.synchronize()
            t = time.perf_counter()
            ivhd.ivhd_knn_build(X, 2)
            return time.perf_counter() - t

        once()
        return min(once() for _ in range(4))

    M, N = 100000, 100
    plain = best(rng.normal(size=(M, N)) + 4 * rng.normal(size=(20, N))[rng.integers(0, 20, M)])
    # every query over every candidate takes some forty times as long
    assert best(_data(kind, M, N)) < 12 * plain
