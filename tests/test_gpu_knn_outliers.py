"""The exact kNN of data with rows far from all others (a missing-value code, a
heavy tail, a column of another size): such a row may spoil no error bound but
its own, neither the answers' nor, by way of repeated queries, the time's."""
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


def _mixture(M, N, seed):
    rng = np.random.default_rng(seed)
    return rng, rng.normal(size=(M, N)) + 4 * rng.normal(size=(20, N))[rng.integers(0, 20, M)]


def _check(ivhd, X, k, rows):
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()[rows]
    tol = X.shape[1] * 2.0 ** -23   # FP32 sums of N squares in order, both roundings of each term
    for q, g, w in zip(rows, got, oracle.knn(X, k, queries=rows)):
        assert len(set(g.tolist())) == len(g) and q not in g and g.min() >= 0
        if not np.array_equal(g, w):
            dg = ((X[g].astype(np.float64) - X[q]) ** 2).sum(1)
            dw = ((X[w].astype(np.float64) - X[q]) ** 2).sum(1)
            np.testing.assert_allclose(dg, dw, rtol=tol, atol=0)


# 8,300 rows of more than 256 features go through the pilot; 3,000 rows are "few"
@pytest.mark.parametrize("M,N", [(3000, 20), (8300, 24), (8300, 260)])
@pytest.mark.parametrize("kind", ["1e3", "9999", "1e12", "1e18", "column", "sparse", "codes", "cauchy", "tiny", "large"])
def test_rows_far_off(ivhd, M, N, kind):
    rng, X = _mixture(M, N, M + N)
    if kind[0].isdigit():
        X[M // 3, N // 2] = float(kind)
    elif kind == "column":      # one feature a thousand times the others
        X[:, 3] *= 1e3
    elif kind == "sparse":      # mostly zeros, values of two sizes
        X = X * (rng.random((M, N)) < 0.02) * 10.0 ** rng.integers(0, 4, size=(M, 1))
    elif kind == "codes":       # a missing-value code in one row of twenty
        X[rng.permutation(M)[: M // 20], 5] = 9999.0
    elif kind == "cauchy":
        X = X * np.abs(rng.standard_cauchy(size=(M, 1)))
    elif kind == "tiny":        # squares stay normal FP32
        X = X * 1e-17
    elif kind == "large":       # and here too
        X = X * 1e16
    X = X.astype(np.float32)
    rows = np.unique(np.concatenate([rng.choice(M, 150, replace=False), [M // 3]]))
    _check(ivhd, X, 5, rows)


def test_one_row_does_not_slow_the_others(ivhd):
    _, X = _mixture(60000, 100, 1)
    X = torch.from_numpy(X.astype(np.float32)).cuda()

    def once():
        torch.cuda.synchronize()
        t = time.perf_counter()
        ivhd.ivhd_knn_build(X, 5)
        return time.perf_counter() - t

    once()
    plain = min(once() for _ in range(5))
    X[12345, 6] = 9999.0
    once()
    # repeating every query over all candidates takes more than ten times as long
    assert min(once() for _ in range(5)) < 3 * plain
