"""The exact kNN of a few queries: every query's candidates are split into up
to 64 ranges, whose lists one wavefront merges through LDS."""
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


# lists of 8, 16 and 32; the candidates nearest to a query spread over all
# ranges (random order), or all in one (sorted by distance from it)
@pytest.mark.parametrize("in_order", [False, True])
@pytest.mark.parametrize("Q,k", [(1, 1), (3, 4), (7, 12), (260, 28)])
def test_lists_of_many_ranges_merge(ivhd, Q, k, in_order):
    rng = np.random.default_rng(Q + k)
    M, N = 70000, 12
    X = rng.integers(-512, 512, size=(M, N)).astype(np.float32)   # FP32 distances are exact
    q = rng.integers(-512, 512, size=(Q, N)).astype(np.float32)
    if in_order:
        X = X[np.argsort(((X - q[0]) ** 2).sum(1))]
    got = ivhd.ivhd_knn_query(torch.from_numpy(X).cuda(), torch.from_numpy(q).cuda(), k).cpu().numpy()
    for i in range(Q):
        d = ((X - q[i]) ** 2).sum(1)
        assert np.array_equal(got[i], np.lexsort((np.arange(M), d))[:k])
