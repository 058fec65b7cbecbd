"""The exact kNN's band where its steps meet: more hits than one segment keeps,
than three keep, all points at one distance; tiles of like queries that are full,
ragged or single; queries apart from the points."""
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


def _near_ties_only(X, q, got, want, N):
    if not np.array_equal(got, want):
        dg = ((X[got].astype(np.float64) - q) ** 2).sum(1)
        dw = ((X[want].astype(np.float64) - q) ** 2).sum(1)
        np.testing.assert_allclose(dg, dw, rtol=N * 2.0 ** -23, atol=0)   # FP32 sums, both roundings of each term


# clusters of 20,000 and of 600 points, every one of which may be the nearest
@pytest.mark.parametrize("M,N,clusters,spread,k", [(60000, 16, 3, 1e-4, 3), (60000, 16, 100, 1e-4, 10),
                                                  (25000, 130, 1, 1e-5, 28), (33000, 7, 2000, 1e-3, 2)])
def test_tight_clusters(ivhd, M, N, clusters, spread, k):
    rng = np.random.default_rng(clusters)
    X = (4 * rng.normal(size=(clusters, N))[rng.integers(0, clusters, M)] + spread * rng.normal(size=(M, N))).astype(np.float32)
    rows = rng.choice(M, 60, replace=False)
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()[rows]
    for q, g, w in zip(rows, got, oracle.knn(X, k, queries=rows)):
        assert len(set(g.tolist())) == k and q not in g and g.min() >= 0
        _near_ties_only(X, X[q], g, w, N)


@pytest.mark.parametrize("M,Q", [(5000, 40), (20000, 1500), (40000, 5000)])
def test_all_points_at_one_distance(ivhd, M, Q):
    # +-unit vectors seen from the origin: every row is as near, and the lowest win
    rng = np.random.default_rng(M)
    X = np.zeros((M, 24), np.float32)
    X[np.arange(M), rng.integers(0, 24, M)] = rng.choice([-1.0, 1.0], M)
    q = np.zeros((Q, 24), np.float32)
    own = torch.arange(Q, device="cuda", dtype=torch.int32) % 3
    got, dist = ivhd.ivhd_knn_query(torch.from_numpy(X).cuda(), torch.from_numpy(q).cuda(), 4, self_idx=own, with_dist=True)
    got = got.cpu().numpy()
    assert bool((dist == 1).all())
    for r in range(3):
        want = [i for i in range(5) if i != r][:4]
        assert (got[r::3] == want).all()


@pytest.mark.parametrize("Q", [300, 4100, 20000])
def test_queries_among_tight_clusters(ivhd, Q):
    rng = np.random.default_rng(Q)
    M, N = 30000, 20
    centres = 5 * rng.normal(size=(40, N))
    X = (centres[rng.integers(0, 40, M)] + 1e-3 * rng.normal(size=(M, N))).astype(np.float32)
    q = (centres[rng.integers(0, 40, Q)] + 1e-3 * rng.normal(size=(Q, N))).astype(np.float32)
    q[:5] += 100   # and some from elsewhere
    got = ivhd.ivhd_knn_query(torch.from_numpy(X).cuda(), torch.from_numpy(q).cuda(), 5).cpu().numpy()
    for i in list(range(5)) + list(range(5, Q, max(1, Q // 50))):
        d = ((X.astype(np.float64) - q[i]) ** 2).sum(1)
        _near_ties_only(X, q[i], got[i], np.lexsort((np.arange(M), d))[:5], N)
