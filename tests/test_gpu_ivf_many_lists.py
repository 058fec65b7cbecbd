"""k-means training with so many lists that the search over the centroids is
run again and again by one object and repeats the queries that it could not
certify: every assignment must come out as if it were a search of its own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def p():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_05455_amd as pkg
    return pkg


def _points(M, N, near):
    """A mixture, and a share `near` of the points in one small spot: the
    centroids that start there are too close for one product to tell apart."""
    rng = np.random.default_rng(M + N)
    x = rng.normal(size=(M, N)) + 4 * rng.normal(size=(20, N))[rng.integers(0, 20, M)]
    n = int(near * M)
    x[:n] = x[0] + 1e-3 * rng.normal(size=(n, N))
    return x[rng.permutation(M)].astype(np.float32)


# 3,841 lists are the fewest that are not "few"; 65,536 rows the fewest with a pilot
@pytest.mark.parametrize("M,N,nlist,n_iter,near", [(12000, 40, 4096, 3, 0.05), (12000, 40, 4096, 3, 0.8),
                                                  (9000, 33, 3841, 4, 0.02), (66000, 100, 4096, 3, 0.02)])
def test_assignments_of_repeated_searches(p, M, N, nlist, n_iter, near):
    x = torch.from_numpy(_points(M, N, near)).cuda()
    c, assign = p.ivhd_ivf_train(x, nlist, n_iter)
    again = p.ivhd_ivf_train(x, nlist, n_iter)
    assert torch.equal(c, again[0]) and torch.equal(assign, again[1])
    assert torch.equal(assign, p.ivhd_knn_query(c, x, 1)[:, 0])
    x64, c64 = x.double(), c.double()
    n2 = (x64 ** 2).sum(1, keepdim=True) + (c64 ** 2).sum(1)
    d = n2 - 2 * (x64 @ c64.T)   # FP64: 2^-50 of n2
    least = d.min(1).values
    got = ((x64 - c64[assign.long()]) ** 2).sum(1)
    # FP32 sums of N squares, both roundings of each term
    assert bool((got <= least * (1 + N * 2.0 ** -23) + 2.0 ** -45 * n2.max()).all())
