"""The exact kNN of rows that lie along a path in their order: answers against
the oracle, and a time that does not depend on the order."""
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


def _line(M, N):
    rng = np.random.default_rng(M)
    return (np.arange(M)[:, None] / M * 50 * rng.normal(size=(1, N)) + 0.3 * rng.normal(size=(M, N))).astype(np.float32)


@pytest.mark.parametrize("M,N,k", [(3900, 12, 3), (8300, 24, 28), (8191, 260, 2)])
def test_along_a_line(ivhd, M, N, k):
    X = _line(M, N)
    rows = np.random.default_rng(k).choice(M, 150, replace=False)
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()[rows]
    tol = N * 2.0 ** -23   # FP32 sums of N squares in order, both roundings of each term
    for q, g, w in zip(rows, got, oracle.knn(X, k, queries=rows)):
        assert len(set(g.tolist())) == len(g) and q not in g and g.min() >= 0
        if not np.array_equal(g, w):
            dg = ((X[g].astype(np.float64) - X[q]) ** 2).sum(1)
            dw = ((X[w].astype(np.float64) - X[q]) ** 2).sum(1)
            np.testing.assert_allclose(dg, dw, rtol=tol, atol=0)


def test_time_does_not_follow_the_order(ivhd):
    X = torch.from_numpy(_line(100000, 100)).cuda()

    def best(x):
        ivhd.ivhd_knn_build(x, 2)
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ivhd.ivhd_knn_build(x, 2)
            t.append(time.perf_counter() - t0)
        return min(t)

    shuffled = best(X[torch.randperm(len(X), generator=torch.Generator().manual_seed(1)).cuda()].contiguous())
    assert best(X) < 6 * shuffled   # some thirty times as long when swept in the rows' order


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("M,k", [(500, 1), (2000, 5), (3000, 28)])
def test_few_points_along_a_line(ivhd, M, k, reverse):
    # every point nearer than the one before it, on the way to the query
    X = (np.arange(M, dtype=np.float32)[:, None] * np.float32([1, 2, -1]))
    if reverse:
        X = X[::-1].copy()
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()
    i = np.arange(M)
    for q in (0, 1, M // 2, M - 1):
        d = (i - q).astype(np.float64) ** 2
        d[q] = np.inf
        assert np.array_equal(got[q], np.lexsort((i, d))[:k])
