"""The exact kNN of calls that are answered from the exact distances at once (few
candidates, or few queries): edges of the tiles of 256 candidates, of the groups
of eight queries, of the chunks of features, of the ranges, aligned and not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ivhd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as m
    return m


def _ranked(X, q, k, own):
    d = ((X.astype(np.float64) - q) ** 2).sum(1)   # integers: exact, in FP32 too
    if own >= 0:
        d[own] = np.inf
    return np.lexsort((np.arange(len(X)), d))[:k]


@pytest.mark.parametrize("M,N,k", [(2, 1, 1), (5, 3, 4), (255, 4, 3), (256, 31, 28), (257, 32, 28), (300, 37, 2),
                                   (1000, 100, 5)])
def test_graph_of_few_points(ivhd, M, N, k):
    X = np.random.default_rng(M).integers(-3, 4, size=(M, N)).astype(np.float32)
    got = ivhd.ivhd_knn_build(torch.from_numpy(X).cuda(), k).cpu().numpy()
    for i in range(M):
        assert np.array_equal(got[i], _ranked(X, X[i], k, i))


# 70,000 candidates in up to 256 ranges; rows at any 4-byte boundary
@pytest.mark.parametrize("M,N,Q,k,shift", [(70000, 8, 1, 28, 0), (70000, 8, 9, 4, 1), (513, 45, 17, 7, 0),
                                           (512, 36, 4000, 1, 2), (100, 64, 20000, 3, 0)])
def test_queries(ivhd, M, N, Q, k, shift):
    rng = np.random.default_rng(M + Q)
    flat = torch.from_numpy(rng.integers(-9, 10, size=M * N + shift).astype(np.float32)).cuda()
    X = flat[shift:].reshape(M, N)
    q = torch.from_numpy(rng.integers(-9, 10, size=(Q, N)).astype(np.float32)).cuda()
    own = torch.from_numpy(np.where(np.arange(Q) % 2 == 0, rng.integers(0, M, Q), -1).astype(np.int32)).cuda()
    idx, dist = ivhd.ivhd_knn_query(X, q, k, self_idx=own, with_dist=True)
    Xh, qh, oh = X.cpu().numpy(), q.cpu().numpy(), own.cpu().numpy()
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    for i in range(0, Q, max(1, Q // 60)):
        want = _ranked(Xh, qh[i], k, oh[i])
        assert np.array_equal(idx[i], want)
        assert np.array_equal(dist[i], ((Xh[want] - qh[i]) ** 2).sum(1))


def test_small_calls_take_a_few_launches(ivhd):
    """300 x 3, k 2, beside a scan of the same points for their neighbours in FP64
    (72 us): 99 us, 273 with the filter's lists."""
    import time
    X = torch.randn((300, 3), device="cuda")
    rows = torch.arange(300, device="cuda", dtype=torch.int32)

    def best(f):
        f()
        t = []
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(lambda: ivhd.ivhd_knn_build(X, 2)) < 2.5 * best(lambda: ivhd.ivhd_eval_neighbours(X, rows, 10))
